"""The graph drivers' kernels at the edges of their tiles (8 vertices per
thread, 32 per bitvector word, 4096 rows per workgroup of the pull), and rows
that the pull has to scan past its first entries, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _graph(n, seed):
    """Random edges, and vertices 1 and n - 2 with edges from every third
    vertex and from a late one only, so that a pull meets long rows with and
    without an early hit."""
    rng = np.random.default_rng(seed)
    e = 4 * n
    src, dst = rng.integers(0, n, e), rng.integers(0, max(1, n - 5), e)
    src = np.concatenate([src, np.arange(0, n, 3), np.arange(n // 2, n)])
    dst = np.concatenate([dst, np.full(len(range(0, n, 3)), min(1, n - 1)), np.full(n - n // 2, max(0, n - 2))])
    key = np.unique(dst.astype(np.int64) * n + src)
    return synth._coo_to_csr(n, n, key // n, key % n, None)


@pytest.mark.parametrize("n", [1, 7, 8, 33, 4095, 4096, 4097, 8200, 20001])
def test_bfs_tile_edges(n):
    torch = _torch()
    A = _graph(n, n)
    M = spx.Matrix.from_host(A, dtype=spx.BOOL)
    s = int(A.col_idx[0])
    dst = np.repeat(np.arange(n), np.diff(A.row_ptr)).astype(np.int32)
    want = oracle.bfs_levels(A.col_idx, dst, n, s)
    for push_only in (False, True):
        level, _ = M.bfs(s, push_only=push_only)
        assert np.array_equal(level.cpu().numpy(), want), f"n={n} push_only={push_only}"
    # levels at an address that is only 4-byte aligned
    import ctypes as C
    from paper_2006_16767_amd import _lib
    buf = torch.full((n + 1,), 77, dtype=torch.int32, device="cuda")
    nl = C.c_int32(0)
    _lib.call("spx_bfs", M._h, s, C.c_void_p(buf.data_ptr() + 4), 1 << 30, None, 0, C.byref(nl), None, 0, None)
    torch.cuda.synchronize()
    assert np.array_equal(buf[1:].cpu().numpy(), want) and int(buf[0]) == 77


@pytest.mark.parametrize("bucket_rows", [0, 64, 128, 4096, 16384])
@pytest.mark.parametrize("lanes", [0, 1, 64])
def test_bfs_levels_on_the_bucket_walk(bucket_rows, lanes):
    """Every level on a direct bucket plan: a short frontier runs as one walk
    per bucket of rows (buckets of whole bitvector words), a long one as the
    product and the update; the last bucket is ragged."""
    _torch()
    n = 20001
    A = _graph(n, 77)
    M = spx.Matrix.from_host(A, dtype=spx.BOOL)
    s = int(A.col_idx[0])
    want = oracle.bfs_levels(A.col_idx, np.repeat(np.arange(n), np.diff(A.row_ptr)).astype(np.int32), n, s)
    plan = spx.Plan()
    plan.pattern, plan.distribution, plan.writeback = spx.PAT_CSC_SPMSPV, spx.DIST_DIRECT, spx.WB_BUCKET
    plan.bucket_rows, plan.lanes = bucket_rows, lanes
    level, plans = M.bfs(s, plan=plan)
    assert np.array_equal(level.cpu().numpy(), want)
    assert len(plans) == M.bfs_levels and all(p.lanes == lanes and p.bucket_rows == bucket_rows for p in plans)


@pytest.mark.parametrize("pattern", [spx.PAT_SPMV, spx.PAT_CSR_SPMSPV])
@pytest.mark.parametrize("n", [1, 5, 4095, 4096, 4097, 12289, 40003])
def test_pagerank_rows_across_tiles(n, pattern):
    """Balanced row-major products leave the rows that span merge tiles (a
    third of the vertices point at vertex 1) to the next select, which adds
    what its chunk of rows lacks; stopped early, to the fold."""
    _torch()
    A = _graph(n, n + 1)
    A = A.with_vals(np.random.default_rng(n).uniform(0.1, 1.0, A.nnz))
    M = spx.Matrix.from_host(A)
    plan = spx.Plan()
    plan.pattern, plan.distribution, plan.writeback = pattern, spx.DIST_BALANCED, 0
    eps = 1e-3 * 0.15 / n
    for limit in (2, 10 ** 6):
        rank, res, _ = M.pagerank(0.85, eps, max_iters=limit, plan=plan, want_residual=True)
        p, r, k = oracle.pagerank_incremental(A, 0.85, eps, limit)
        assert M.pr_iters == k
        # the two add a row's products in different orders: a relative 1e-16
        # times the products per row and rounds, far below 1e-11
        for got, want in ((rank, p), (res, r)):
            assert np.abs(got.cpu().numpy() - want).max() <= 1e-11 * np.abs(want).max(), f"n={n} limit={limit}"
