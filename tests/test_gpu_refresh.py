"""The refresh of the column-major values after an in-place update: by blocks of
64 KB of the row-major ones from 64 blocks on, against a handle made from the
new values (the same values in the same places give the same bits)."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx

pytestmark = pytest.mark.gpu


def _csr(m, n, nnz, seed):
    """nnz distinct cells of an m x n matrix, row-major."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cells = torch.randperm(m * n, generator=g, device="cuda")[:nnz].sort()[0]
    rows, cols = cells // n, (cells % n).to(torch.int32)
    ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.bincount(rows, minlength=m).cumsum(0)
    return ptr.to(torch.int32), cols


@pytest.mark.parametrize("dtype", ["float32", "float64", "int32"])
@pytest.mark.parametrize("n", [1, 37, 4096, 16384])
@pytest.mark.parametrize("extra", [-1, 0, 4099])  # below, at and past 64 blocks
def test_refresh_matches_a_new_handle(dtype, n, extra):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = getattr(torch, dtype)
    nnz = 64 * (8192 if dtype == "float64" else 16384) + extra
    m = -(-nnz * (1 if n < 40 else 3) // n) + 5
    ptr, cols = _csr(m, n, nnz, n + extra)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    draw = lambda k: (torch.randint(-4, 5, (k,), generator=g, device="cuda", dtype=torch.int32) if dtype == "int32"
                      else torch.randn(k, generator=g, device="cuda", dtype=dt))
    vals, x = draw(nnz), draw(n)
    M = spx.Matrix(ptr, cols, vals, m, n)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    plan = spx.Plan()  # column-major, one writer per row and sum: bits repeat
    plan.pattern, plan.distribution, plan.writeback = spx.PAT_CSC_SPMSPV, spx.DIST_BALANCED, spx.WB_SORT
    for step in range(3):
        with torch.no_grad():
            M.vals.copy_(draw(nnz))
        M.sync_values()
        fresh = spx.Matrix(ptr, cols, M.vals.clone(), m, n)
        a, b = M.run_plan((idx, x), plan), fresh.run_plan((idx, x), plan)
        assert torch.equal(a, b), f"{dtype} n={n} extra={extra} step={step}"
        if dtype != "int32":
            G = torch.randn((2, m), generator=g, device="cuda", dtype=dt)
            assert torch.equal(M.transpose_matvec(G), fresh.transpose_matvec(G))
