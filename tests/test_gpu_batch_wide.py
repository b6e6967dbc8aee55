"""run_batch over 2^24 columns, where a group's slab (2 GiB and a line) lies
beyond 32-bit buffer offsets and its rows are gathered by plain addresses.
The work units are those of 32 empty rows, of empty rows between two rows
longer than a unit, of a single row and of whole rows: a unit without entries
gathers nothing but the slab's zero row. The vectors hold 2 % of the columns,
enough to join a group."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64, np.int32])
def test_groups_beyond_32_bit_offsets(dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 1 << 24
    lens = [3, 0, 40] + [0] * 100 + [900] + [0] * 5 + [1500, 1] + [0] * 31 + [17] * 60 + [0] * 70
    rng = np.random.default_rng(24)
    m = len(lens)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    nx = n // 50 + 1
    # a row's columns: from the vectors' stride and from anywhere, the last column among them
    cols = [np.unique(np.concatenate([rng.integers(0, nx, k) * 49, rng.integers(0, n, k), [n - 1]]))[-k:] if k else []
            for k in lens]
    idx = np.concatenate(cols).astype(np.int32)
    whole = dtype == np.int32
    vals = rng.integers(-9, 10, idx.size).astype(dtype) if whole else rng.standard_normal(idx.size).astype(dtype)
    xi = [np.arange(nx, dtype=np.int64) * 49, np.append(np.arange(nx - 1, dtype=np.int64) * 50 + 7, n - 1)]
    B = len(xi)
    assert all(v[-1] < n and v.size >= 0.02 * n for v in xi)
    xv = [rng.integers(-9, 10, v.size).astype(dtype) if whole else rng.standard_normal(v.size).astype(dtype)
          for v in xi]
    M = spx.Matrix.from_host(synth.CSR(m, n, ptr, idx, vals))
    vec_ptr = np.concatenate([[0], np.cumsum([v.size for v in xi])]).astype(np.int32)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    Y = M.run_batch(dev(vec_ptr), dev(np.concatenate(xi).astype(np.int32)), dev(np.concatenate(xv)))
    torch.cuda.synchronize()
    assert M.batch_status() == 0
    Y = Y.cpu().numpy()
    rows = np.repeat(np.arange(m), lens)
    for b in range(B):
        x = np.zeros(n, np.float64)
        x[xi[b]] = xv[b]
        terms = vals.astype(np.float64) * x[idx]
        ref = np.bincount(rows, terms, minlength=m)
        bound = {np.float32: 1e-5, np.float64: 1e-12, np.int32: 0.0}[dtype] * np.bincount(rows, np.abs(terms), minlength=m)
        assert np.abs(terms).sum() > 0
        assert np.all(np.abs(Y[b].astype(np.float64) - ref) <= bound), b
