"""The rule that gives an attention call its kernel (no GPU)."""
import os

import pytest

from paper_2606_05875_amd import qcf
from routes import attn_route, batch_route


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(qcf.lib_path()):
        from paper_2606_05875_amd.build import build
        build(verbose=False)


def test_tiles_that_fill_the_chip_are_not_cut():
    """Cut tiles round their partial sums to bf16: only calls whose row tiles of 256 query vectors
    number fewer than 384 -- by the caller's bounds -- go to the persistent grid."""
    for reqs in range(1, 70):                        # one tile per request and KV head, of either size
        for max_kv in (1600, 4096):
            got = batch_route([32] * reqs, [max_kv] * reqs, 32, 8, 128)
            assert got != "stream" or reqs * 8 < 384, (reqs, max_kv, got)
    assert batch_route([32] * 47, [4096] * 47, 32, 8, 128) == "stream"
    assert [batch_route([32] * r, [4096] * r, 32, 8, 128) for r in (48, 63, 64)] == ["w4"] * 3
    # a loose bound of the rows per request had given the whole-tile grid, and does
    args = dict(batch=4, max_kv=4096, hq=32, hkv=8, d=128, n_rows=450, n_kv_rows=4 * 4096)
    assert attn_route(max_rows=450, **args) == "stream"
    assert attn_route(max_rows=800, **args) == "w4"
    assert attn_route(max_rows=2 ** 31 - 1, **args) == "w4"
