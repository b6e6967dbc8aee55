"""Balanced atomic column-major products whose tile size follows the work: at
one position per thread (65536 items and less over 256 tiles), at the step to
two, and with the full 2048 items per tile, against the oracle."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

from parity_util import assert_close, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f32", "f64", "i32", "bool"])
@pytest.mark.parametrize("items", [16, 272, 65518, 65535, 65552, 131088, 600015,
                                   4080, 4096, 1048544, 1048576])  # 1, 2, 256, 257 runs of 256 lengths
def test_tile_size_follows_the_items(kind, items):
    """Every column has 15 entries, so an entry of x is 16 items of the merge
    (65535 and 600015: one column has 14)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx = -(-items // 16)
    n, m = nx + 40, 30000
    rng = np.random.default_rng(items)
    cols = np.repeat(np.arange(n), 15)
    rows = (np.repeat(rng.integers(0, m, n), 15) + np.tile(np.arange(15) * 1999, n)) % m
    pick = rng.permutation(n)[:nx].astype(np.int32)
    pick.sort()
    short = 16 * nx - items
    if short:  # the first selected column loses entries
        drop = np.nonzero(cols == pick[0])[0][:short]
        rows, cols = np.delete(rows, drop), np.delete(cols, drop)
    npdt = {"f32": np.float32, "f64": np.float64, "i32": np.int32, "bool": None}[kind]
    vals = None
    if npdt is not None:
        vals = (rng.integers(-4, 5, rows.size) if kind == "i32" else rng.uniform(-1, 1, rows.size)).astype(npdt)
    order = np.lexsort((cols, rows))
    A = synth._coo_to_csr(m, n, rows[order], cols[order], None if vals is None else vals[order])
    code = {"f32": spx.F32, "f64": spx.F64, "i32": spx.I32, "bool": spx.BOOL}[kind]
    M = spx.Matrix.from_host(A, dtype=code)
    xv = None
    if npdt is not None:
        xv = (rng.integers(-4, 5, nx) if kind == "i32" else rng.uniform(-1, 1, nx)).astype(npdt)
    t = lambda a: torch.as_tensor(a, device="cuda")
    plan = spx.Plan()
    plan.pattern, plan.distribution, plan.writeback = spx.PAT_CSC_SPMSPV, spx.DIST_BALANCED, spx.WB_ATOMIC
    y = M.run_plan((t(pick), None if xv is None else t(xv)), plan)
    ref, S = reference(A, pick, xv, kind)
    assert_close(y.cpu().numpy(), ref, S, kind, f"{kind} {items} items")
