"""Attention calls with few query vectors (blocks whose waves split the keys, long key ranges cut
over blocks) at the edges of their tiles (32 query vectors, 32 keys), against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import qcfuse as Q
from paper_2606_05875_amd import qcf
from parity import assert_close
from routes import batch_route, keysplit_waves
from test_gpu_kernels import dev, draw, host, padded, say

pytestmark = pytest.mark.gpu


def _attn(hq, hkv, d, n_kv, n_rows, pad, kpos, rot):
    rng = np.random.default_rng(41)
    cu = lambda x: np.concatenate([[0], np.cumsum(x)]).astype(np.int32)
    cu_kv, cu_r = cu(n_kv), cu(n_rows)
    k = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    v = draw(rng, (cu_kv[-1], hkv, d), "bf16", 1 / math.sqrt(d))
    q = draw(rng, (cu_r[-1], hq, d), "bf16", math.sqrt(d))
    pos = np.concatenate([np.sort(rng.integers(0, n, m)) for n, m in zip(n_kv, n_rows)]).astype(np.int32)
    kp = None
    if kpos:                                          # ascending positions with gaps
        kp = np.concatenate([np.sort(rng.choice(2 * n, n, replace=False)) for n in n_kv]).astype(np.int32)
        pos *= 2
    out = torch.full((cu_r[-1], hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((cu_r[-1], hq), device="cuda")
    scale = 1 / math.sqrt(d)
    K, V = padded(k, pad, torch.bfloat16), padded(v, pad, torch.bfloat16)
    geo = (dev(pos), dev(cu_r), K, V, dev(cu_kv), max(n_rows), max(n_kv), scale)
    if rot:
        theta = 1e6
        qcf.qcf_sparse_prefill_attn_rope(out, dev(q, torch.bfloat16), *geo,
                                         qcf.rope_position_table(max(n_kv), d, theta), lse=lse)
        q = Q.round_storage(Q.rope(q, pos, theta), "bf16")
    else:
        qcf.qcf_sparse_prefill_attn(out, dev(q, torch.bfloat16), *geo, kv_pos=dev(kp) if kpos else None, lse=lse)
    for b in range(len(n_kv)):
        a, e, ka, ke = cu_r[b], cu_r[b + 1], cu_kv[b], cu_kv[b + 1]
        if e == a:
            continue
        pick = np.arange(a, e)
        kpb = kp[ka:ke] if kpos else np.arange(ke - ka)
        want = Q.round_storage(Q.attention(q[pick], pos[pick], k[ka:ke], v[ka:ke], kpb, scale, hkv), "bf16")
        assert_close(host(out)[pick], want, "bf16", f"request {b}")
        r, h = pick[-1], hq - 1
        vis = kpb <= pos[r]
        if vis.any():
            lg = (k[ka:ke][vis, hkv - 1].astype(np.float64) @ q[r, h].astype(np.float64)) * scale
            assert abs(float(lse[r, h]) - np.log(np.exp(lg - lg.max()).sum()) - lg.max()) < 2e-3


# head groups 1 to 32; one key, one less, exactly and one more than a tile; rows that fill a unit
# partly; a request without rows; 8, 4 and 2 waves per block (long ranges; few units; many short ones)
@pytest.mark.parametrize("mode", ["causal", "rope", "positions"])
@pytest.mark.parametrize("hq,hkv,d,n_kv,n_rows,pad,waves", [
    (8, 2, 64, [1, 31, 32, 33, 300], [1, 7, 8, 9, 20], 0, 4),
    (4, 4, 128, [257, 1100], [31, 64], 64, 8),
    (16, 4, 64, [993, 40], [33, 7], 0, 8),
    (32, 1, 64, [90, 40], [2, 0], 8, 4),
    (32, 8, 128, [100, 70, 33], [65, 33, 3], 128, 4),
    (64, 8, 128, [300, 257, 64, 33, 290], [40, 64, 1, 33, 64], 0, 2),
    (32, 8, 64, [257, 1, 64, 290, 33, 160, 31, 300, 32], [64, 1, 33, 60, 64, 7, 31, 64, 17], 64, 2),
])
def test_keysplit_edges(hq, hkv, d, n_kv, n_rows, pad, waves, mode):
    say("key-split attention", mode, hq, hkv, d, n_kv, n_rows, pad, waves)
    assert batch_route(n_rows, n_kv, hq, hkv, d, kv_pos=mode == "positions") == "keysplit"
    assert keysplit_waves(n_rows, n_kv, hq, hkv, d) == waves
    _attn(hq, hkv, d, n_kv, n_rows, pad, mode == "positions", mode == "rope")


@pytest.mark.parametrize("mode", ["causal", "positions"])
@pytest.mark.parametrize("hq,hkv,d,n_kv,n_rows", [
    (32, 8, 128, [2047, 90], [7, 4]),                   # 16 units, 4 cuts; a short request in the batch
    (8, 8, 64, [5000], [32]),                           # 8 units, 9 cuts
    (4, 1, 128, [9000], [3]),                           # 1 unit, 16 cuts
])
def test_keysplit_cut_key_ranges(hq, hkv, d, n_kv, n_rows, mode):
    """Key ranges cut over blocks: the partials are merged in order, so two calls over a dirty
    workspace agree bit for bit, and the result matches the oracle."""
    say("key-split attention, cut", mode, hq, hkv, d, n_kv, n_rows)
    assert batch_route(n_rows, n_kv, hq, hkv, d, kv_pos=mode == "positions") == "keysplit"
    _attn(hq, hkv, d, n_kv, n_rows, 0, mode == "positions", False)
    rng = np.random.default_rng(42)
    k, v = (dev(draw(rng, (n_kv[0], hkv, d), "bf16", 0.1), torch.bfloat16) for _ in range(2))
    q = dev(draw(rng, (n_rows[0], hq, d), "bf16", 3.0), torch.bfloat16)
    need = qcf.qcf_sparse_prefill_attn_workspace_size(1, n_rows[0], n_kv[0], hq, hkv, d, torch.bfloat16)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    cu = [dev(np.array([0, n], np.int32)) for n in (n_rows[0], n_kv[0])]
    pos = dev(np.full(n_rows[0], n_kv[0] - 1, np.int32))
    outs = []
    for w in (ws, ws, None):
        o = torch.empty_like(q)
        qcf.qcf_sparse_prefill_attn(o, q, pos, cu[0], k, v, cu[1], n_rows[0], n_kv[0], 0.1, workspace=w)
        outs.append(o)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("mode", ["causal", "rope"])
@pytest.mark.parametrize("d,n", [(64, 1), (64, 33), (128, 40), (128, 290)])
def test_keysplit_infinite_last_value(d, n, mode):
    """An infinite value of the last key gives infinity, and nothing else, to the rows that see it: the
    rest of its tile holds no key."""
    say("key-split attention, infinite last value", mode, d, n)
    rng = np.random.default_rng(43)
    hq, hkv, rows = 8, 2, 9
    k, v = (draw(rng, (n, hkv, d), "bf16", 0.1) for _ in range(2))
    v[n - 1, 1, 5] = np.inf
    q = dev(draw(rng, (rows, hq, d), "bf16", 1.0), torch.bfloat16)
    out = torch.empty_like(q)
    assert batch_route([rows], [n], hq, hkv, d) == "keysplit"
    geo = (dev(np.full(rows, n - 1, np.int32)), dev(np.array([0, rows], np.int32)), dev(k, torch.bfloat16),
           dev(v, torch.bfloat16), dev(np.array([0, n], np.int32)), rows, n, 0.1)
    if mode == "rope":
        qcf.qcf_sparse_prefill_attn_rope(out, q, *geo, qcf.rope_position_table(n, d, 1e6))
    else:
        qcf.qcf_sparse_prefill_attn(out, q, *geo)
    got = host(out)
    assert np.all(got[:, hq // 2:, 5] == np.inf)
    got[:, hq // 2:, 5] = 0
    assert np.isfinite(got).all()
