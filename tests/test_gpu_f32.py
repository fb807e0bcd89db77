"""float32 attention and scores at the edges of their tiles (16 query vectors, 16 keys, 8 waves
taking the key tiles in turn), against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import qcfuse as Q
from paper_2606_05875_amd import qcf
from parity import assert_close, assert_scores
from test_gpu_kernels import dev, draw, host, padded, say

pytestmark = pytest.mark.gpu


def _batch(n_kv, n_rows):
    cu = lambda x: np.concatenate([[0], np.cumsum(x)]).astype(np.int32)
    return cu(n_kv), cu(n_rows)


# head groups 1, 2, 4 and 32 (two tiles per row); fewer, exactly and one more than a tile of
# keys and of query vectors; one to many tiles per wave; a request without rows; padded rows
@pytest.mark.parametrize("kpos", [False, True])
@pytest.mark.parametrize("hq,hkv,d,n_kv,n_rows,pad", [
    (8, 2, 64, [1, 15, 16, 17, 130], [1, 3, 4, 5, 33], 0),
    (4, 4, 128, [127, 128, 129], [16, 15, 17], 64),
    (32, 1, 64, [300, 40], [2, 0], 4),
    (6, 3, 128, [1500], [260], 0),
])
def test_attention_f32_edges(hq, hkv, d, n_kv, n_rows, pad, kpos):
    say("attention f32", hq, hkv, d, n_kv, n_rows, pad, kpos)
    rng = np.random.default_rng(31)
    cu_kv, cu_r = _batch(n_kv, n_rows)
    k = draw(rng, (cu_kv[-1], hkv, d), "f32", 1 / math.sqrt(d))
    v = draw(rng, (cu_kv[-1], hkv, d), "f32", 1 / math.sqrt(d))
    q = draw(rng, (cu_r[-1], hq, d), "f32", math.sqrt(d))
    pos = np.concatenate([np.sort(rng.integers(0, n, m)) for n, m in zip(n_kv, n_rows)]).astype(np.int32)
    kp = None                                        # explicit positions: ascending, with gaps
    if kpos:
        kp = np.concatenate([np.sort(rng.choice(2 * n, n, replace=False)) for n in n_kv]).astype(np.int32)
        pos *= 2
    out = torch.full((cu_r[-1], hq, d), float("nan"), device="cuda")
    lse = torch.empty((cu_r[-1], hq), device="cuda")
    scale = 1 / math.sqrt(d)
    qcf.qcf_sparse_prefill_attn(out, dev(q), dev(pos), dev(cu_r), padded(k, pad, torch.float32),
                                padded(v, pad, torch.float32), dev(cu_kv), max(n_rows), max(n_kv), scale,
                                kv_pos=dev(kp) if kpos else None, lse=lse)
    for b in range(len(n_kv)):
        a, e, ka, ke = cu_r[b], cu_r[b + 1], cu_kv[b], cu_kv[b + 1]
        if e == a:
            continue
        kpb = kp[ka:ke] if kpos else np.arange(ke - ka)
        want = Q.attention(q[a:e], pos[a:e], k[ka:ke], v[ka:ke], kpb, scale, hkv)
        assert_close(host(out)[a:e], want, "f32", f"request {b}")
        vis = kpb <= pos[e - 1]
        if not vis.any():
            continue
        lg = (k[ka:ke][vis, hkv - 1].astype(np.float64) @ q[e - 1, hq - 1].astype(np.float64)) * scale
        assert abs(float(lse[e - 1, hq - 1]) - np.log(np.exp(lg - lg.max()).sum()) - lg.max()) < 1e-4


def test_attention_f32_masked_values_stay_out():
    """Values of keys that a row does not see never reach it, finite or not (rows of a cache past
    a request position may hold anything), and a row that sees no key is zero."""
    say("attention f32, masked rows that are not finite")
    rng = np.random.default_rng(32)
    hq, hkv, d, n = 8, 2, 64, 90
    k, v = (draw(rng, (n, hkv, d), "f32", 1 / math.sqrt(d)) for _ in range(2))
    q = draw(rng, (5, hq, d), "f32", math.sqrt(d))
    pos = np.array([20, 20, 21, 21, 21], np.int32)
    kp = np.arange(n, dtype=np.int32) + 3           # explicit positions: three fewer keys
    bad_v, bad_k = v.copy(), k.copy()
    bad_v[22:, :, ::3], bad_k[22:] = np.nan, np.inf
    cu = dev(np.array([0, 5], np.int32)), dev(np.array([0, n], np.int32))
    for kv_pos in (None, dev(kp)):
        got = []
        for kk, vv in ((k, v), (bad_k, bad_v)):
            out = torch.empty((5, hq, d), device="cuda")
            qcf.qcf_sparse_prefill_attn(out, dev(q), dev(pos), cu[0], dev(kk), dev(vv), cu[1], 5, n,
                                        1 / math.sqrt(d), kv_pos=kv_pos)
            got.append(host(out))
        assert np.isfinite(got[1]).all()
        np.testing.assert_allclose(got[1], got[0], rtol=0, atol=1e-5)
    bad_v[21, 0, 0] = np.inf                        # seen by rows 2-4 only
    out = torch.empty((5, hq, d), device="cuda")
    qcf.qcf_sparse_prefill_attn(out, dev(q), dev(pos), cu[0], dev(k), dev(bad_v), cu[1], 5, n, 1 / math.sqrt(d))
    inf = ~np.isfinite(host(out))
    assert not inf[:2].any() and inf[2:, :hq // hkv, 0].all() and inf.sum() == 3 * hq // hkv
    none = torch.full((5, hq, d), 7.0, device="cuda")
    qcf.qcf_sparse_prefill_attn(none, dev(q), dev(np.full(5, -1, np.int32)), cu[0], dev(k), dev(v), cu[1], 5, n,
                                1 / math.sqrt(d))
    assert not host(none).any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kpos", [False, True])
def test_attention_f32_very_negative_logits(d, kpos):
    """Logits far below -1e30 are logits like any others: two equal largest keys share the weight."""
    say("attention f32, very negative logits", d, kpos)
    n, hq, hkv, scale = 300, 4, 2, 0.25
    rng = np.random.default_rng(34)
    v = draw(rng, (n, hkv, d), "f32")
    k, q = np.zeros((n, hkv, d), np.float32), np.zeros((40, hq, d), np.float32)
    q[..., 0] = 2.0 ** 57
    k[..., 0] = -(2.0 ** 58)
    k[[5, 150], :, 0] = -(2.0 ** 57)                # logits -2^112 for the two, -2^113 for the others
    pos = np.full(40, n - 1, np.int32)
    out, lse = torch.empty((40, hq, d), device="cuda"), torch.empty((40, hq), device="cuda")
    qcf.qcf_sparse_prefill_attn(out, dev(q), dev(pos), dev(np.array([0, 40], np.int32)), dev(k), dev(v),
                                dev(np.array([0, n], np.int32)), 40, n, scale, lse=lse,
                                kv_pos=dev(np.arange(n, dtype=np.int32)) if kpos else None)
    want = np.repeat((v[5].astype(np.float64) + v[150]) / 2, hq // hkv, 0)
    np.testing.assert_allclose(host(out), np.broadcast_to(want, (40, hq, d)), rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(lse.cpu().numpy(), -(2.0 ** 112), rtol=1e-6)


@pytest.mark.parametrize("hq,hkv,d,ctxs,nqs,pad", [
    (8, 2, 64, [1, 15, 17, 129], [1, 4, 5, 33], 0),
    (4, 4, 128, [128, 127], [16, 17], 64),
    (32, 1, 64, [300], [1], 4),
    (16, 4, 128, [2100], [40], 0),
])
def test_scores_f32_edges(hq, hkv, d, ctxs, nqs, pad):
    say("scores f32", hq, hkv, d, ctxs, nqs, pad)
    rng = np.random.default_rng(33)
    cu_kv, cu_q = _batch([c + n for c, n in zip(ctxs, nqs)], nqs)
    k = draw(rng, (cu_kv[-1], hkv, d), "f32", 1 / math.sqrt(d))
    q = draw(rng, (cu_q[-1], hq, d), "f32", 1.5 * math.sqrt(d))
    sc = torch.full((int(cu_kv[-1]),), -5.0, device="cuda")
    qcf.qcf_probe_scores(sc, dev(q), padded(k, pad, torch.float32), dev(cu_q), dev(cu_kv),
                         dev(np.array(ctxs, np.int32)), max(nqs), max(ctxs), 1 / math.sqrt(d))
    got = sc.double().cpu().numpy()
    for b in range(len(ctxs)):
        a, n = int(cu_kv[b]), ctxs[b]
        want = Q.critical_scores(q[cu_q[b]:cu_q[b + 1]], k[a:a + n], 1 / math.sqrt(d), hkv)
        assert_scores(got[a:a + n], want, f"request {b}")
        assert np.all(got[a + n:cu_kv[b + 1]] == -5.0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("pic", [False, True])
def test_scores_f32_very_negative_logits(d, pic):
    """Logits far below -1e30 are logits like any others: two equal largest keys share the weight."""
    say("scores f32, very negative logits", d, pic)
    n, nq, hq, hkv = 300, 9, 4, 2
    k, q = np.zeros((n + nq, hkv, d), np.float32), np.zeros((nq, hq, d), np.float32)
    q[..., 0] = 2.0 ** 57
    k[..., 0] = -(2.0 ** 58)
    k[[5, 150], :, 0] = -(2.0 ** 57)
    sc = torch.full((n + nq,), -5.0, device="cuda")
    i32 = lambda *x: dev(np.array(x, np.int32))
    geo = (i32(0, nq), i32(0, n + nq), i32(n), nq, n, 0.25)
    if pic:
        table = torch.empty((1, d // 2, 2), device="cuda")
        qcf.qcf_rope_table(table, i32(0), 1e4)
        qcf.qcf_probe_scores_pic(sc, dev(q), dev(k), dev(np.zeros(n + nq, np.int32)), table, *geo)
    else:
        qcf.qcf_probe_scores(sc, dev(q), dev(k), *geo)
    want = np.zeros(n)
    want[[5, 150]] = nq * hq / 2
    np.testing.assert_allclose(sc.cpu().numpy()[:n], want, rtol=1e-6)
    assert (sc[n:] == -5.0).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("big", [0, 37, 299])
def test_f32_weights_below_the_smallest_normal_number(d, big):
    """A key whose weight is a subnormal number (e^-91 .. e^-100 of the largest) still counts: its scores
    rank such keys, and a large value of it reaches the output."""
    say("f32, subnormal weights", d, big)
    n, hq, hkv = 300, 4, 2
    gap = np.where(np.arange(n) == big, 0.0, 91.0 + np.arange(n) % 10)
    k, q = np.zeros((n, hkv, d), np.float32), np.zeros((8, hq, d), np.float32)
    q[..., 1], k[..., 1] = 1.0, -gap[:, None]
    v = np.zeros((n, hkv, d), np.float32)
    low = (big + 50) % n
    v[low] = 1e30
    i32 = lambda *x: dev(np.array(x, np.int32))
    out = torch.empty((8, hq, d), device="cuda")
    qcf.qcf_sparse_prefill_attn(out, dev(q), dev(np.full(8, n - 1, np.int32)), i32(0, 8), dev(k), dev(v),
                                i32(0, n), 8, n, 1.0)
    # a subnormal weight has fewer digits: at least 37.2e-45 / 1.4e-45 = 26 steps, half a step off
    np.testing.assert_allclose(host(out), 1e30 * np.exp(-gap[low]), rtol=0.02)
    sc = torch.empty(n + 8, device="cuda")
    k2 = np.concatenate([k, np.zeros((8, hkv, d), np.float32)])
    qcf.qcf_probe_scores(sc, dev(q), dev(k2), i32(0, 8), i32(0, n + 8), i32(n), 8, n, 1.0)
    np.testing.assert_allclose(sc.double().cpu().numpy()[:n], 8 * hq * np.exp(-gap), rtol=0.02)


def test_attention_f32_skips_rows_outside_the_tensors():
    """Row offsets that reach before or past the rows of the call (here inside larger buffers) write
    nothing there; the rows inside are computed."""
    say("attention f32, rows outside the tensors")
    rng = np.random.default_rng(35)
    n, hq, hkv, d, rows = 70, 4, 2, 64, 20
    k, v = (draw(rng, (n, hkv, d), "f32", 1 / math.sqrt(d)) for _ in range(2))
    q = draw(rng, (rows + 16, hq, d), "f32", math.sqrt(d))
    pos = rng.integers(0, n, rows + 16).astype(np.int32)
    out, lse = torch.full((rows + 16, hq, d), 7.0, device="cuda"), torch.full((rows + 16, hq), 7.0, device="cuda")
    inner = slice(8, 8 + rows)
    qcf.qcf_sparse_prefill_attn(out[inner], dev(q)[inner], dev(pos)[inner], dev(np.array([-8, rows + 8], np.int32)),
                                dev(k), dev(v), dev(np.array([0, n], np.int32)), rows + 16, n, 1 / math.sqrt(d),
                                lse=lse[inner])
    want = Q.attention(q[inner], pos[inner], k, v, np.arange(n), 1 / math.sqrt(d), hkv)
    got = host(out)
    assert_close(got[inner], want, "f32", "rows inside")
    assert np.all(got[:8] == 7.0) and np.all(got[8 + rows:] == 7.0)
    assert (lse[:8] == 7.0).all() and (lse[8 + rows:] == 7.0).all()
