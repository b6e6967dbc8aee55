"""The layer's products through LDS slabs, at the sizes where the split can go
wrong: operands of exactly one slab, one column more (several row blocks for
dX, 16-byte columns for the forward), batch rows around a column's 8 FP32 or 4
FP64 values, segments around the 64 groups and the 64-entry step, rows longer
than several steps, empty rows, ascending and shuffled column indices (dvals
blocks of 512, 2048 and 8192 columns). Bounds: a result
is a chain of at most ceil(length / 16) + 4 fused additions per slab (1,100
entries in a column here: 75 roundings of 2^-24, 4.5e-6 of sum |a x|), dvals
one of at most 4 per 64 batch rows and a fold of 4, so the library's 1e-5 and
1e-12 hold. dvals takes the slab path only where the columns ascend within
every row: both kinds run."""
import numpy as np
import pytest

import oracle
import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

from parity_util import assert_close

pytestmark = pytest.mark.gpu

SHAPES = [
    # m, n, entries per row
    (65, 4096, 64),    # one whole slab, a second round of the 64 groups with one segment
    (1030, 4097, 17),  # one column past a slab of 32-byte columns
    (70, 8192, 150),   # one whole slab of 16-byte columns, rows of three steps
    (8195, 65, 9),     # dX over three row blocks of G
    (513, 300, 40),
    (200, 1025, 100),  # dvals over three blocks of columns, the last of one
    (1, 9, 9),
]


def _matrix(m, n, per_row, dtype, seed, ascend=False):
    rng = np.random.default_rng(seed)
    A = synth.uniform_rows(m, n, per_row, seed, dtype=dtype) if per_row < n else synth.random_csr(m, n, 1.0, seed)
    # some rows emptied, and the columns of every row shuffled or ascending
    keep = np.ones(A.nnz, bool)
    rows = np.repeat(np.arange(m), np.diff(A.row_ptr))
    if m > 4:
        keep[np.isin(rows, rng.choice(m, m // 20, replace=False))] = False
    order = np.lexsort((np.asarray(A.col_idx) if ascend else rng.random(A.nnz), rows))
    order = order[keep[order]]
    rows = rows[order]
    ptr = np.zeros(m + 1, np.int32)
    np.cumsum(np.bincount(rows, minlength=m), out=ptr[1:])
    return synth.CSR(m, n, ptr, np.asarray(A.col_idx)[order], np.asarray(A.vals)[order].astype(dtype))


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("B", [1, 4, 5, 9, 64, 70])
@pytest.mark.parametrize("ascend", [False, True])
def test_slab_products_match_oracle(kind, shape, B, ascend):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = np.float32 if kind == "f32" else np.float64
    m, n, per_row = SHAPES[shape]
    A = _matrix(m, n, per_row, dt, 900 + shape, ascend)
    M = spx.Matrix.from_host(A)
    rng = np.random.default_rng(B)
    X = rng.standard_normal((B, n)).astype(dt)
    G = rng.standard_normal((B, m)).astype(dt)
    Xd, Gd = torch.as_tensor(X, device="cuda"), torch.as_tensor(G, device="cuda")
    Y = M.spmv_batch(Xd)
    dX, dv = M.backward(Gd, Xd)
    again = M.backward(Gd, Xd)
    torch.cuda.synchronize()
    # fixed orders of summation: the same bits on every call
    assert torch.equal(dX, again[0]) and torch.equal(dv, again[1]) and torch.equal(Y, M.spmv_batch(Xd))
    Yh, dXh = Y.cpu().numpy(), dX.cpu().numpy()
    dX_ref, S_dx, dv_ref = oracle.grad(A, G, X)
    for b in range(B):
        ref, S = oracle.spmv(A, X[b].astype(np.float64))
        assert_close(Yh[b], ref, S, kind, f"forward {m}x{n} B={B} b={b}")
        assert_close(dXh[b], dX_ref[b], S_dx[b], kind, f"dX {m}x{n} B={B} b={b}")
    S_dv = oracle.grad(A.with_vals(np.ones(A.nnz)), np.abs(G), np.abs(X), want_dx=False)[2]
    assert_close(dv.cpu().numpy(), dv_ref, S_dv, kind, f"dvals {m}x{n} B={B}")


def test_slab_lanes_without_an_entry_take_no_part():
    """Infinities and NaN in the operand reach the rows that hold their
    column and no other row."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, B = 130, 200, 6
    A = _matrix(m, n, 20, np.float32, 77)
    M = spx.Matrix.from_host(A)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((B, n)).astype(np.float32)
    X[2, 0] = np.inf
    X[4, n - 1] = np.nan
    Y = M.spmv_batch(torch.as_tensor(X, device="cuda")).cpu().numpy()
    D = np.zeros((m, n), bool)
    D[np.repeat(np.arange(m), np.diff(A.row_ptr)), A.col_idx] = True
    want = np.ones((B, m), bool)
    want[2, D[:, 0]] = False
    want[4, D[:, n - 1]] = False
    assert np.array_equal(np.isfinite(Y), want)
