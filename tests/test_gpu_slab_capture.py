"""A handle's first gradients captured into a HIP graph: the slab kernels search
for the bounds that no table holds yet. Replays, with eager calls (which build
the tables) between them, give the bits that the eager calls give."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("m,n,p,B", [
    (8200, 600, 0.3, 3),      # 16-byte columns of G: dX over three slabs, the last of 10 rows
    (8200, 600, 0.3, 70),
    (300, 8192, 0.2, 64),     # dvals over 16 (32) blocks of columns
    (2100, 2049, 0.1, 20),    # the last block of one column
    (2100, 2049, 0.1, 5),     # dvals blocks of 2048 columns (1024 in FP64)
    (300, 8200, 0.1, 3),      # and of 8192
])
def test_captured_first_backward(dtype, m, n, p, B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = getattr(torch, dtype)
    rng = np.random.default_rng(m + B)
    mask = rng.random((m, n)) < p
    mask[:, 0] |= np.arange(m) % 7 == 0
    mask[5] = False    # an empty row, an empty column and a full one
    mask[:, 1] = False
    mask[:, n - 1] = True
    rows, cols = np.nonzero(mask)
    ptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    A = synth.CSR(m, n, ptr, cols.astype(np.int32), rng.standard_normal(cols.size).astype(dtype))
    M, E = spx.Matrix.from_host(A), spx.Matrix.from_host(A)
    G, X = torch.randn(B, m, device="cuda", dtype=dt), torch.randn(B, n, device="cuda", dtype=dt)
    dX, dv = torch.empty_like(X), torch.empty(A.nnz, device="cuda", dtype=dt)
    want = E.backward(G, X)
    M.spmv_batch(X)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        M.transpose_matvec(G, dX)
        M.dvals(G, X, dv)
    for step in range(4):
        dX.zero_()
        dv.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dX, want[0]) and torch.equal(dv, want[1]), step
        if step > 0:
            eager = M.backward(G, X)
            assert torch.equal(eager[0], want[0]) and torch.equal(eager[1], want[1])
        G.normal_()
        X.normal_()
        want = E.backward(G, X)
