"""Prepared calls hand every argument and the stream to the entry point whole (no GPU: the entry
point is replaced by a recorder that is called through ctypes the same way)."""
import ctypes
import os
from types import SimpleNamespace

import pytest

from paper_2606_05875_amd import qcf

HANDLE = 0x7F1234567890          # an address as a runtime hands it out: more than 32 bits


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(qcf.lib_path()):
        from paper_2606_05875_amd.build import build
        build(verbose=False)


def recorded(name, args, monkeypatch):
    """A Prepared call of `name` whose entry point, on both handles, records what arrives."""
    seen = []
    types = qcf.EXPORTS[name][1]
    callback = ctypes.CFUNCTYPE(ctypes.c_int, *types)(lambda *a: seen.append(a) or 0)
    address = ctypes.cast(callback, ctypes.c_void_p).value
    typed, untyped = ctypes.CDLL(None)._FuncPtr(address), ctypes.CDLL(None)._FuncPtr(address)
    typed.restype, typed.argtypes = qcf.EXPORTS[name]
    monkeypatch.setattr(qcf, "lib", lambda: SimpleNamespace(**{name: typed}))
    monkeypatch.setattr(qcf, "_untyped", lambda: SimpleNamespace(**{name: untyped}))
    return qcf.Prepared(name, args, callback), seen


class Holder:                    # what torch.cuda.Stream offers ctypes
    _as_parameter_ = ctypes.c_void_p(HANDLE)


# the stream is passed in a register by the first entry point and on the stack by the second
@pytest.mark.parametrize("name,args", [
    ("qcf_rope_table", (ctypes.c_void_p(HANDLE + 16), ctypes.c_void_p(HANDLE + 32), 2 ** 31 - 1, 128, 1e6)),
    ("qcf_gather_rows", (ctypes.c_void_p(HANDLE + 16), None, HANDLE + 48, 2 ** 40, 5, 64, 2 ** 33, 64)),
])
def test_arguments_and_stream_arrive_whole(name, args, monkeypatch):
    monkeypatch.setattr(qcf, "_stream", lambda: ctypes.c_void_p(HANDLE + 8))
    p, seen = recorded(name, args, monkeypatch)
    plain = lambda a: a.value if isinstance(a, ctypes.c_void_p) else a
    # the first call takes the declared entry point, the others the one without declared types
    for given, want in ((HANDLE, HANDLE), (HANDLE, HANDLE), (ctypes.c_void_p(HANDLE), HANDLE),
                        (Holder(), HANDLE), (None, HANDLE + 8), (0, None), (2 ** 63 + 5, 2 ** 63 + 5)):
        p(given)
        assert seen[-1][-1] == want, given
        assert seen[-1][:-1] == tuple(plain(a) for a in args)


def test_a_wrong_number_of_arguments_is_refused():
    args = (ctypes.c_void_p(HANDLE), ctypes.c_void_p(HANDLE), 1, 128, 1e6)
    for bad in (args[:-1], args + (0,)):
        with pytest.raises(qcf.QcfError):
            qcf.Prepared("qcf_rope_table", bad, None)


def test_a_call_with_nothing_to_launch_is_a_prepared_call():
    p = qcf.prepare(lambda: None)
    assert isinstance(p, qcf.Prepared)
    assert p.name == "<lambda>" and p.args == () and p.keep is None and p.fn() == 0
    assert p() is None and p(HANDLE) is None


def test_a_call_made_once_converts_nothing(monkeypatch):
    """A new step prepares and calls each of its calls once: its first pass must not pay for the
    conversion that makes the later ones cheap."""
    monkeypatch.setattr(qcf, "_stream", lambda: ctypes.c_void_p(HANDLE))
    args = (ctypes.c_void_p(HANDLE + 16), ctypes.c_void_p(HANDLE + 32), 5, 128, 1e6)
    p, seen = recorded("qcf_rope_table", args, monkeypatch)
    p()
    assert p.args is args
    p()
    assert isinstance(p.args[2], ctypes.c_int64) and isinstance(p.args[4], ctypes.c_double)
    p()
    assert seen[0] == seen[1] == seen[2] and len(seen) == 3
