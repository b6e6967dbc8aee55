"""The refresh by blocks of 64 KB at its smallest size, 96 blocks: the calls
that gather and the calls by blocks leave the same column-major values, and
those of a handle made from the new values."""
import pytest

import paper_2006_16767_amd as spx
from test_gpu_refresh import _csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("n", [1, 4096, 8192])
@pytest.mark.parametrize("extra", [-1, 0, 4099])  # below, at and past 96 blocks
def test_refresh_by_blocks_matches_a_new_handle(dtype, n, extra):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = getattr(torch, dtype)
    nnz = 96 * (8192 if dtype == "float64" else 16384) + extra
    m = -(-nnz * (1 if n == 1 else 3) // n) + 5
    ptr, cols = _csr(m, n, nnz, n + extra)
    M = spx.Matrix(ptr, cols, torch.randn(nnz, device="cuda", dtype=dt), m, n)
    G = torch.randn((2, m), device="cuda", dtype=dt)
    for step in range(4):
        with torch.no_grad():
            M.vals.copy_(torch.randn(nnz, device="cuda", dtype=dt))
        M.sync_values()
        fresh = spx.Matrix(ptr, cols, M.vals.clone(), m, n)
        assert torch.equal(M.transpose_matvec(G), fresh.transpose_matvec(G)), step
