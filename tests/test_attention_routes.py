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
    assert attn_route(max_rows=800, **args) == "plain"
    assert attn_route(max_rows=2 ** 31 - 1, **args) == "plain"
    args = dict(batch=1, max_kv=8192, hq=32, hkv=8, d=128, n_rows=1200, n_kv_rows=8192)
    assert attn_route(max_rows=1200, **args) == "stream"
    assert attn_route(max_rows=4000, **args) == "w4"


def test_tiles_are_counted_by_the_rows_there_are():
    """A batch whose rows sit in few of its requests has far fewer row tiles than its longest request
    would give: padding is no reason to leave the persistent grid or the 8-wave blocks."""
    route = lambda rows, kv, d=128: batch_route(rows, [kv] * len(rows), 32, 8, d)
    for d in (64, 128):
        assert route([1000, 32], 4096, d) == "stream"              # 512 tiles of 128 padded, 272 at most
        assert route([700, 10, 10], 2048, d) == "stream"
        assert route([1000, 1000], 4096, d) == "w4"                # 512 of them real
        assert route([600] * 4, 2000, d) == "w4"
        assert route([900, 20, 20, 20], 1500, d) == "plain"        # whole tiles, few of them
        assert route([900, 20, 20, 20], 8192, d) == "plain"
        assert route([2000, 16], 8000, d) == "plain"
        assert route([600] * 3 + [10] * 4, 3000, d) == "w4"        # more tiles than fit the chip at once
        assert route([3000, 30, 30, 30], 4000, d) == "w4"
        assert route([1000] * 3 + [40], 6000, d) == "w4"
        assert route([1250], 1536, d) == "w4"                      # short ranges
        assert route([700, 10], 1400, d) == ("stream" if d == 64 else "w4")
        assert route([1400, 10], 1536, d) == "w4"


def test_large_probes_keep_the_shared_tile_kernel():
    """Long probes of more than 1792 units of 32 query vectors (head size 128) fill the chip with the
    blocks that share key tiles."""
    route = lambda nq, kv, d: batch_route([nq] * 16, [kv] * 16, 32, 8, d, kv_pos=True)
    assert [route(nq, 4000, 128) for nq in (64, 112, 113, 120, 128, 129)] == ["keysplit"] * 2 + ["pos"] * 4
    assert [route(nq, 4000, 64) for nq in (128, 129)] == ["keysplit", "pos"]
    assert route(112, 2016, 128) == "pos" and route(64, 2016, 128) == "keysplit"


def test_work_queues_need_a_workspace_that_was_asked_for():
    """The counters of the work queues lie in the workspace: a call that needs none (at most 64 keys)
    may come with a smaller one, so it never takes them."""
    for rows in (8000, 20000):
        args = dict(batch=1, max_rows=rows, hq=64, hkv=8, d=128, n_rows=rows)
        assert qcf.qcf_sparse_prefill_attn_workspace_size(1, rows, 64, 64, 8, 128) == 0
        assert attn_route(max_kv=64, n_kv_rows=64, **args) == "w4"
        assert qcf.qcf_sparse_prefill_attn_workspace_size(1, rows, 129, 64, 8, 128) > 0
        assert attn_route(max_kv=129, n_kv_rows=129, **args) == "queue"
        assert attn_route(max_kv=129, n_kv_rows=129, ws=False, **args) == "w4"


def test_workspace_holds_the_partials_of_cut_key_ranges():
    """Key ranges are cut into at most 256 partials of 32 query vectors (float32, and two floats each);
    every call long enough to be cut (2017 keys and more) needs a workspace that holds them."""
    for hkv in list(range(1, 260)) + [1000, 65535]:
        for d in (64, 128):
            need = qcf.qcf_sparse_prefill_attn_workspace_size(1, 1, 2017, hkv, hkv, d)
            assert need >= 256 * 32 * (4 * d + 8), (hkv, d)
