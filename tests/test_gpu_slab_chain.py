"""Rows and columns that fill LDS slabs, with products chosen so that one long
FP32 chain per lane loses every small one: the first product of each of a
segment's 16 lanes is 1, all others are 2^-24, and 1 + 2^-24 rounds to 1. In
one chain a slab of 4096 (8192) entries loses 255 (511) of them, 1.5e-5 (3.0e-5)
of the sum; with at most 64 additions before a fold it is at most 64 + 8 + 4
roundings of 2^-24, 4.5e-6, so the library's bound of 1e-5 * sum |a x| holds."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what,length,B", [
    ("forward", 4096, 5),   # 32-byte columns
    ("forward", 4096, 3),   # 16-byte columns
    ("forward", 8192, 8),
    ("dX", 4096, 5),
    ("dX", 12288, 5),       # three slabs
    ("dX", 12288, 2),
])
def test_long_segments_keep_the_bound(what, length, B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    segs = 70  # more than the 64 groups of a workgroup
    vals = np.full((segs, length), 2.0 ** -24, np.float32)
    vals[:, :16] = 1.0
    exact = vals[0].astype(np.float64).sum()
    if what == "dX":
        vals = vals.T
    m, n = vals.shape
    A = synth.CSR(m, n, np.arange(m + 1, dtype=np.int32) * n, np.tile(np.arange(n, dtype=np.int32), m),
                  np.ascontiguousarray(vals).ravel())
    M = spx.Matrix.from_host(A)
    ones = torch.ones((B, length), dtype=torch.float32, device="cuda")
    out = M.spmv_batch(ones) if what == "forward" else M.backward(ones, want_dvals=False)[0]
    assert out.shape == (B, segs)
    worst = float((out.double() - exact).abs().max())
    assert worst <= 1e-5 * exact, worst / exact
