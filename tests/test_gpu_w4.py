"""Recomputed-row attention on 4-wave blocks (128 query vectors, 64-key tiles in an XOR-permuted LDS
layout) where it can go wrong: tile remainders, key tails, head groups, more requests than the
block order ranks, no workspace, rotated queries read through an index; against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import qcfuse as Q
from paper_2606_05875_amd import qcf
from parity import assert_close
from routes import batch_route
from test_gpu_kernels import dev, draw, host, padded, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_rows,pad,rot", [
    (32, 8, 128, [200] * 70, [180] * 70, 0, False),               # 70 requests: no ranking by length
    (32, 8, 128, [64, 63, 65, 1] * 40, [64, 33, 31, 1] * 40, 128, True),
    (16, 2, 64, [1500, 40, 1300], [1400, 31, 777], 64, False),     # group 8, head size 64
    (8, 8, 64, [700, 129, 690] * 6, [650, 129, 640] * 6, 0, True), # group 1
    (32, 1, 128, [900, 512], [900, 300], 0, True),                 # group 32: 4 rows per block
    (64, 8, 128, [64] * 120, [64] * 120, 0, False),                # 64 keys: no workspace
    (40, 10, 128, [2000], [1700], 128, True),
])
def test_attention_w4(hq, hkv, d, n_kv, n_rows, pad, rot):
    say("attention, 4-wave blocks", hq, hkv, d, len(n_kv), max(n_kv), pad, rot)
    assert batch_route(n_rows, n_kv, hq, hkv, d) == "w4"
    rng = np.random.default_rng(51)
    cu = lambda x: np.concatenate([[0], np.cumsum(x)]).astype(np.int32)
    cu_kv, cu_r = cu(n_kv), cu(n_rows)
    k = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    v = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    pos = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for n, m in zip(n_kv, n_rows)]).astype(np.int32)
    n, src = int(cu_r[-1]), None
    q = draw(rng, (n + 3, hq, d), "bf16", math.sqrt(d))
    out = torch.full((n, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((n, hq), device="cuda")
    geo = (dev(pos), dev(cu_r), padded(k, pad, torch.bfloat16), padded(v, pad, torch.bfloat16), dev(cu_kv),
           max(n_rows), max(n_kv), 1 / math.sqrt(d))
    if rot:
        src = rng.permutation(n + 3)[:n].astype(np.int32)
        qcf.qcf_sparse_prefill_attn_rope(out, dev(q, torch.bfloat16), *geo,
                                         qcf.rope_position_table(max(n_kv), d, 1e6), q_src=dev(src), lse=lse)
        q = Q.round_storage(Q.rope(q[src], pos, 1e6), "bf16")
    else:
        q = q[:n]
        qcf.qcf_sparse_prefill_attn(out, dev(q, torch.bfloat16), *geo, lse=lse)
    got, rpb = host(out), 128 // (hq // hkv)
    assert np.isfinite(got).all()
    for b in range(0, len(n_kv), 1 if len(n_kv) < 8 else 9):
        a, e, ka, ke = cu_r[b], cu_r[b + 1], cu_kv[b], cu_kv[b + 1]
        first = np.arange(a, e, rpb)                # the first and last row of every row tile
        pick = np.unique(np.concatenate([first, np.minimum(first + rpb - 1, e - 1)]))
        want = Q.round_storage(Q.attention(q[pick], pos[pick], k[ka:ke], v[ka:ke], np.arange(ke - ka),
                                           1 / math.sqrt(d), hkv), "bf16")
        assert_close(got[pick], want, "bf16", f"request {b}")
        r, h = pick[-1], hq - 1
        lg = (k[ka:ka + pos[r] + 1, hkv - 1].astype(np.float64) @ q[r, h].astype(np.float64)) / math.sqrt(d)
        assert abs(float(lse[r, h]) - np.log(np.exp(lg - lg.max()).sum()) - lg.max()) < 2e-3


def test_requests_of_one_tile_are_computed_whole():
    """48 requests of one row tile each: every tile is computed whole, so a request's rows have the
    same bits as in a batch of 64 (which fills the 4-wave grid)."""
    hq, hkv, d, n_kv, rows = 32, 8, 128, 1600, 32
    say("attention, one tile per request", n_kv, rows)
    gen = torch.Generator(device="cuda").manual_seed(52)
    new = lambda n, h: torch.randn((n, h, d), generator=gen, device="cuda").to(torch.bfloat16)
    k, v, q = new(64 * n_kv, hkv), new(64 * n_kv, hkv), new(64 * rows, hq)
    pos = torch.arange(n_kv - rows, n_kv, dtype=torch.int32, device="cuda").repeat(64)
    outs = []
    for reqs in (48, 64):
        assert batch_route([rows] * reqs, [n_kv] * reqs, hq, hkv, d) == "w4"
        cu = lambda n: dev(np.arange(reqs + 1, dtype=np.int32) * n)
        out = torch.empty((reqs * rows, hq, d), dtype=torch.bfloat16, device="cuda")
        qcf.qcf_sparse_prefill_attn(out, q[:reqs * rows], pos[:reqs * rows], cu(rows), k[:reqs * n_kv],
                                    v[:reqs * n_kv], cu(n_kv), rows, n_kv, 1 / math.sqrt(d))
        outs.append(out)
    assert torch.equal(outs[0], outs[1][:48 * rows])


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_rows,rot", [
    (32, 8, 128, [1500, 1100, 64, 1300], [900, 20, 0, 21], True),
    (16, 2, 64, [700] + [300] * 31, [180] + [1] * 31, False),      # group 8
    (8, 8, 64, [1400] + [65, 700, 64, 3] * 2, [1300] + [3] * 8, True),   # group 1
])
def test_few_requests_hold_the_rows(hq, hkv, d, n_kv, n_rows, rot):
    """A batch whose rows sit in few of its requests runs on 8-wave blocks, one per row tile: every
    16th row and the last one of every request against the oracle."""
    say("attention, few requests hold the rows", hq, hkv, d, n_kv[:4], n_rows[:4], rot)
    assert batch_route(n_rows, n_kv, hq, hkv, d) == "plain"
    rng = np.random.default_rng(53)
    cu = lambda x: np.concatenate([[0], np.cumsum(x)]).astype(np.int32)
    cu_kv, cu_r = cu(n_kv), cu(n_rows)
    k = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    v = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    q = draw(rng, (cu_r[-1], hq, d), "bf16", math.sqrt(d))
    pos = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for n, m in zip(n_kv, n_rows)]).astype(np.int32)
    out = torch.full((cu_r[-1], hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    geo = (dev(q, torch.bfloat16), dev(pos), dev(cu_r), dev(k, torch.bfloat16), dev(v, torch.bfloat16), dev(cu_kv),
           max(n_rows), max(n_kv), 1 / math.sqrt(d))
    if rot:
        qcf.qcf_sparse_prefill_attn_rope(out, *geo, qcf.rope_position_table(max(n_kv), d, 1e6))
        q = Q.round_storage(Q.rope(q, pos, 1e6), "bf16")
    else:
        qcf.qcf_sparse_prefill_attn(out, *geo)
    got = host(out)
    assert np.isfinite(got).all()
    for b in range(len(n_kv)):
        a, e, ka, ke = cu_r[b], cu_r[b + 1], cu_kv[b], cu_kv[b + 1]
        if e == a:
            continue
        pick = np.unique(np.concatenate([np.arange(a, e, 16), [e - 1]]))
        want = Q.round_storage(Q.attention(q[pick], pos[pick], k[ka:ke], v[ka:ke], np.arange(ke - ka),
                                           1 / math.sqrt(d), hkv), "bf16")
        assert_close(got[pick], want, "bf16", f"request {b}")
