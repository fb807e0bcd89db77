"""Which kernel an attention call runs on, asked of the library's own rule (no GPU needed): tests that
aim at one kernel assert it, so that a change of the rule cannot move them to another unnoticed."""
import ctypes

from paper_2606_05875_amd import qcf

NAMES = ("f32", "keysplit", "stream", "queue", "w4", "pos", "plain")


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("batch", "max_rows", "max_kv", "hq", "hkv", "d")]


def attn_route(batch, max_rows, max_kv, hq, hkv, d, n_rows, n_kv_rows, bf16=True, kv_pos=False, ws=True):
    fn = qcf.lib()["_ZN3qcf10attn_routeERKNS_9AttnShapeEllbbb"]
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.POINTER(_Shape), ctypes.c_long, ctypes.c_long] + [ctypes.c_bool] * 3
    return NAMES[fn(_Shape(batch, max_rows, max_kv, hq, hkv, d), n_rows, n_kv_rows, bf16, kv_pos, ws)]


def keysplit_waves(n_rows, n_kv, hq, hkv, d):
    """Waves per block of the key-split kernel for such a batch."""
    fn = qcf.lib()["_ZN3qcf14keysplit_wavesERKNS_9AttnShapeEll"]
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.POINTER(_Shape), ctypes.c_long, ctypes.c_long]
    return fn(_Shape(len(n_kv), max(n_rows), max(n_kv), hq, hkv, d), sum(n_rows), sum(n_kv))


def batch_route(n_rows, n_kv, hq, hkv, d, **kw):
    """The route of a batch of requests with n_rows[b] rows over n_kv[b] keys each."""
    return attn_route(len(n_kv), max(n_rows), max(n_kv), hq, hkv, d, sum(n_rows), sum(n_kv), **kw)
