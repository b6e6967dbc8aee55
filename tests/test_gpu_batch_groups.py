"""run_batch at the edges of its groups (32 vectors of 4-byte values, 16 of
8-byte ones), slab tiles (256 columns), row blocks (64 KB of Y), work units
(768 entries, 512 of 8-byte values, 32 rows) and column segments, against the oracle."""
import numpy as np
import pytest

import paper_2006_16767_amd as spx
from paper_2006_16767_amd import synth

from parity_util import assert_close, reference

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _matrix(m, n, per_row, npdt, seed):
    """per_row entries in a tenth of the rows and 3 in the others (empty rows
    in between); row 5 and column 2 full."""
    rng = np.random.default_rng(seed)
    counts = np.where(rng.random(m) < 0.1, min(per_row, n), min(3, n))
    counts[rng.random(m) < 0.2] = 0
    rows = np.repeat(np.arange(m), counts)
    cols = rng.integers(0, n, rows.size)
    rows = np.concatenate([rows, np.full(n, 5), np.arange(m)])
    cols = np.concatenate([cols, np.arange(n), np.full(m, 2)])
    key = np.unique(rows.astype(np.int64) * n + cols)
    rows, cols = key // n, key % n
    row_ptr = np.zeros(m + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(rows, minlength=m))
    if npdt == np.int32:
        vals = rng.integers(-4, 5, key.size).astype(npdt)
    else:
        vals = rng.uniform(-1, 1, key.size).astype(npdt)
    return synth.CSR(m, n, row_ptr, cols.astype(np.int32), vals)


def _batch(n, counts, npdt, seed, shuffle):
    """Vectors of counts[b] entries; every other one in a random order."""
    rng = np.random.default_rng(seed)
    out = []
    for b, c in enumerate(counts):
        idx = rng.permutation(n)[:c].astype(np.int32)
        if not (shuffle and b % 2):
            idx.sort()
        val = rng.integers(-4, 5, c) if npdt == np.int32 else rng.uniform(-1, 1, c)
        out.append((idx, val.astype(npdt)))
    return out


def _check(M, A, vecs, kind, npdt, what):
    torch = _torch()
    t = lambda a: torch.as_tensor(a, device="cuda")
    ptr = np.zeros(len(vecs) + 1, np.int32)
    ptr[1:] = np.cumsum([len(i) for i, _ in vecs])
    Y = torch.full((len(vecs), A.m), 7, device="cuda", dtype=t(vecs[0][1]).dtype)
    M.run_batch(t(ptr), t(np.concatenate([i for i, _ in vecs])), t(np.concatenate([v for _, v in vecs])), Y)
    torch.cuda.synchronize()
    assert M.batch_status() == 0
    Y = Y.cpu().numpy()
    for b, (idx, val) in enumerate(vecs):
        ref, S = reference(A, idx, val, kind)
        assert_close(Y[b], ref, S, kind, f"{what} b={b} nnz_x={len(idx)}")


@pytest.mark.parametrize("kind,rows", [("f32", 16384), ("i32", 16384), ("f64", 8192)])
def test_edges_of_groups_tiles_and_blocks(kind, rows):
    npdt = {"f32": np.float32, "f64": np.float64, "i32": np.int32}[kind]
    gs = 16 if kind == "f64" else 32
    for case, (m, n, joined) in enumerate([(rows - 1, 255, gs - 1), (rows, 256, gs), (rows + 1, 257, gs + 1),
                                           (2 * rows + 33, 1500, 2 * gs + 1), (37, 700, 1), (40, 300, 0)]):
        A = _matrix(m, n, 40, npdt, case)
        M = spx.Matrix.from_host(A, renumber=False)
        # joined vectors hold at least 2 % of n; the others less, down to none
        counts = [n, n - 1] + [max(1, n // 3 + 5 * i % n) for i in range(joined)]
        counts = [min(c, n) for c in counts[:joined]] + [0, 1, max(1, n // 60), 0, max(1, n // 100)]
        order = np.random.default_rng(case).permutation(len(counts))
        vecs = _batch(n, [counts[i] for i in order], npdt, case, shuffle=True)
        _check(M, A, vecs, kind, npdt, f"{kind} {m}x{n}")


@pytest.mark.parametrize("kind", ["f32", "f64"])
def test_too_few_entries_for_row_blocks(kind):
    """More than eight segments per entry: the persistent phases run the
    sparse vectors, beside a group."""
    npdt = {"f32": np.float32, "f64": np.float64}[kind]
    rng = np.random.default_rng(4)
    m, n = 300_000, 40_000
    rows, cols = np.sort(rng.choice(m, 900, replace=False)), rng.integers(0, n, 900)
    row_ptr = np.zeros(m + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(rows, minlength=m))
    A = synth.CSR(m, n, row_ptr, cols.astype(np.int32), rng.uniform(-1, 1, 900).astype(npdt))
    M = spx.Matrix.from_host(A, renumber=False)
    vecs = _batch(n, [n, 40, 0, n // 3, 1, 700], npdt, 9, shuffle=True)
    _check(M, A, vecs, kind, npdt, f"{kind} sparse rows")


def test_batches_of_changing_size_on_one_handle():
    """A smaller batch after a larger one, and back: what one leaves in the
    workspace does not show in the next."""
    A = _matrix(5000, 900, 20, np.float32, 1)
    M = spx.Matrix.from_host(A, renumber=False)
    for i, counts in enumerate([[900] * 70 + [5] * 20, [300, 4], [0, 3, 900] * 9, [450] * 40]):
        _check(M, A, _batch(900, counts, np.float32, i, shuffle=i == 2), "f32", np.float32, f"batch {i}")
