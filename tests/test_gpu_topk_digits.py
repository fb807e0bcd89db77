"""Selection where the digits of the radix select begin and end elsewhere: scores that share few, many
or all leading bits, signs and exponents mixed, infinities, NaN, ties at the boundary, at the edges of
the register kernels' sizes.  Exact, against a stable sort of the order-preserving integer keys."""
import numpy as np
import pytest
import torch

from paper_2606_05875_amd import qcf
from test_gpu_kernels import dev, say

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    x = {"equal": lambda: np.full(n, -3.5), "last bit": lambda: np.ones(n),
         "two": lambda: rng.choice([-1.0, 2.0], n), "narrow": lambda: 1 + rng.random(n) * 1e-3,
         "wide": lambda: np.exp(rng.normal(0, 15, n)), "signs": lambda: rng.normal(0, 1, n),
         "negative": lambda: -np.exp(rng.normal(0, 5, n)),
         "special": lambda: rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-45, -1e-45, 3e38, 1.0], n),
         "lowest": lambda: np.where(rng.random(n) < 0.5, np.float32(-3.4028235e38), -np.inf)}[kind]().astype(np.float32)
    if kind == "last bit":
        x = np.where(rng.random(n) < 0.3, np.nextafter(np.float32(1), np.float32(2)), x)
    if kind == "lowest" and n > 2:
        x.view(np.uint32)[:2] = 0xFFFFFFFF           # the smallest key of all: a negative NaN
    return x


@pytest.mark.parametrize("kind", ["equal", "last bit", "two", "narrow", "wide", "signs", "negative", "special", "lowest"])
@pytest.mark.parametrize("top", [1024, 4096, 8192, 16384, 32768, 65536])
def test_select_any_leading_bits(kind, top):
    say("topk digits", kind, top)
    rng = np.random.default_rng(71)
    lens, ks = [], []
    for n in (1, 2, 63, 64, 65, 257, top - 1, top):
        for k in sorted({1, max(1, n // 3), max(1, n - 1)}):
            lens.append(n)
            ks.append(k)
    s = _scores(kind, sum(lens), rng)
    if kind == "lowest":
        s = np.concatenate([_scores(kind, n, rng) for n in lens])
    cum = lambda v: np.concatenate([[0], np.cumsum(v)[:-1]]).astype(np.int32)
    out = torch.full((sum(ks),), -7, dtype=torch.int32, device="cuda")
    i32 = lambda v: dev(np.array(v, np.int32))
    qcf.qcf_select_topk(out, dev(s), i32(cum(lens)), i32(lens), i32(ks), i32(cum(ks)), top)
    bits = np.where(s == 0, np.float32(0), s).view(np.uint32)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.int64)
    got = out.cpu().numpy()
    for a, n, k, o in zip(cum(lens), lens, ks, cum(ks)):
        want = a + np.sort(np.argsort(-key[a:a + n], kind="stable")[:k])
        np.testing.assert_array_equal(got[o:o + k], want, f"{n} scores, k {k}")
