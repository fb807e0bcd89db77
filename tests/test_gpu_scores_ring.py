"""Probe scores over long key splits (512 keys and more per block, keys through an LDS ring), against
the CPU oracle and, bit for bit, against the pass for keys rotated on the fly (which stages keys
another way: a table of zero angles leaves them as they are)."""
import math

import numpy as np
import pytest
import torch

from oracle import qcfuse as Q
from paper_2606_05875_amd import qcf
from parity import assert_scores
from test_gpu_kernels import dev, draw, padded, say

pytestmark = pytest.mark.gpu


# With r query rows and g heads per KV head a request has ceil(r g / 256) tiles; the splits are
# cut from the longest context for 512 (batches: 2048) blocks or half as many.
@pytest.mark.parametrize("hq,hkv,d,nqs,ctxs,pad", [
    (64, 8, 128, [128], [8300], 0),                       # 4 tiles, splits of 544: a ragged last one
    (32, 8, 64, [65], [33000], 8),                        # a tile of 4 vectors: 7 waves without any
    (64, 8, 64, [256, 1, 40, 7], [4200, 64, 1, 2500], 0), # short requests leave splits empty
    (64, 8, 128, [256, 4] + [5, 33] * 7,                  # edges of chunks, groups and splits
     [1090, 1023, 31, 33, 65, 700, 512, 513, 1, 575, 576, 577, 640, 2, 1056, 32], 128),
    (16, 16, 128, [300, 290, 280, 17] * 4, [2200, 2000, 545, 543] * 4, 0),   # one head per group
])
def test_long_splits(hq, hkv, d, nqs, ctxs, pad):
    say("probe scores, long splits", hq, hkv, d, nqs, ctxs, pad)
    rng = np.random.default_rng(61)
    n_qt = -(-max(nqs) * (hq // hkv) // 256)
    blocks = n_qt * hkv * len(nqs)
    n_splits = max(1, -(-(512 if len(nqs) == 1 else 2048) // blocks))
    assert max(ctxs) / n_splits > 480, "the shape no longer gives long splits"
    cu_kv = np.concatenate([[0], np.cumsum([c + q for c, q in zip(ctxs, nqs)])]).astype(np.int32)
    cu_q = np.concatenate([[0], np.cumsum(nqs)]).astype(np.int32)
    T = int(cu_kv[-1])
    k = draw(rng, (T, hkv, d), "bf16", 1 / math.sqrt(d))
    q = draw(rng, (int(cu_q[-1]), hq, d), "bf16", 1.5 * math.sqrt(d))
    scale = 1 / math.sqrt(d)
    kd, qd = padded(k, pad, torch.bfloat16), dev(q, torch.bfloat16)
    geo = (dev(cu_q), dev(cu_kv), dev(np.array(ctxs, np.int32)), max(nqs), max(ctxs), scale)
    ws = torch.full((qcf.qcf_probe_scores_workspace_size(len(nqs), max(nqs), max(ctxs), hq, hkv, d),),
                    0xFF, dtype=torch.uint8, device="cuda")
    got = torch.full((T,), -5.0, device="cuda")
    qcf.qcf_probe_scores(got, qd, kd, *geo, workspace=ws)
    table = torch.empty((1, d // 2, 2), device="cuda")
    qcf.qcf_rope_table(table, dev(np.zeros(1, np.int32)), 1e6)
    ref = torch.full((T,), -5.0, device="cuda")
    qcf.qcf_probe_scores_pic(ref, qd, kd, dev(np.zeros(T, np.int32)), table, *geo)
    assert torch.equal(got, ref)
    qcf.qcf_probe_scores(got, qd, kd, *geo, accumulate=True, workspace=ws)
    host, first = got.double().cpu().numpy(), ref.double().cpu().numpy()
    for b in range(len(nqs)):
        a, e = int(cu_kv[b]), int(cu_kv[b]) + ctxs[b]
        want = Q.critical_scores(q[cu_q[b]:cu_q[b + 1]], k[a:e], scale, hkv)
        assert_scores(first[a:e], want, f"request {b}")
        np.testing.assert_array_equal(host[a:e], 2 * first[a:e])
        assert np.all(host[e:cu_kv[b + 1]] == -5.0)               # query slots untouched
