"""What the library's host code does around its kernels where something fails
or the stream is being captured: which kernels it launches, what it allocates
and when it waits. Runs without a GPU, on a stand-in for the HIP runtime
(hip_stub.cpp) that only writes these calls down; every scenario in a process
of its own."""
import ctypes as C
import importlib.util
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PY = os.path.join(os.path.dirname(HERE), "paper_2006_16767_amd", "_lib.py")
ALLOCATION_REFUSED, ALLOCATION_ALLOWED = 1, 2  # during a capture
TABLE = "Lb1E"  # in the name of a slab kernel that reads a table of bounds


class Stub:
    def __init__(self, path):
        # before libspx, so that its references bind to the stand-in
        self.so = C.CDLL(path, mode=C.RTLD_GLOBAL)
        self.so.stub_log.restype = C.c_char_p
        self.so.stub_fail_sizes.argtypes = [C.c_size_t, C.c_size_t]
        self.so.stub_total.argtypes = [C.c_uint64]
        spec = importlib.util.spec_from_file_location("spx_lib", LIB_PY)
        self.L = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.L)
        self.lib = self.L.load()
        self.keep = []

    def array(self, kind, values):
        a = (kind * max(1, len(values)))(*values)
        self.keep.append(a)
        return C.addressof(a)

    def zeros(self, bytes_):
        a = (C.c_char * bytes_)()
        self.keep.append(a)
        return C.addressof(a)

    def matrix(self, m, n, per_row, dtype=None):
        """per_row entries in the first columns of each row; device memory is
        host memory, so the arrays serve as they are."""
        L = self.L
        nnz = m * per_row
        csr = L.Csr(m, n, nnz, L.F32 if dtype is None else dtype, self.array(C.c_int32, range(0, nnz + 1, per_row)),
                    self.array(C.c_int32, list(range(per_row)) * m), self.zeros(4 * nnz))
        h = C.c_void_p()
        assert self.lib.spx_matrix_create(C.byref(csr), L.NO_RENUMBER | L.FORMAT_CSR, None, C.byref(h)) == 0
        return h

    def calls(self, f, *args):
        """The status of f(*args) and what the library asked of the runtime."""
        self.so.stub_clear_log()
        rc = f(*args)
        return rc, self.so.stub_log().decode().split("\n")[:-1]


def kernels(log):
    return [line for line in log if line.startswith("launch")]


def has(log, name):
    return any(name in line for line in log)


def block_bounds_under_capture(s, mode):
    """The first backward of a handle is a captured one: no table of bounds is
    built (it would be filled when the graph runs) and nothing is allocated;
    the kernels search for the bounds. The next eager call builds the tables
    and reads them, and so does a call captured after it."""
    m, n, B = 8192, 600, 64
    H = s.matrix(m, n, 200)
    X, G, Y, dX, dv = (s.zeros(4 * k) for k in (B * n, B * m, B * m, B * n, m * 200))
    rc, log = s.calls(s.lib.spmv_csr_batch, H, B, X, Y, None)
    assert rc == 0 and kernels(log) == log and has(log, "k_slab_gather")
    s.so.stub_capturing(mode)
    for call, args in ((s.lib.spx_backward, (G, X, dX, dv)), (s.lib.spmv_csr_transpose, (G, dX)),
                       (s.lib.dvals_pattern, (G, X, dv)), (s.lib.spmv_csr_batch, (X, Y))):
        rc, log = s.calls(call, H, B, *args, None)
        assert rc == 0, s.lib.spx_last_error()
        assert kernels(log) == log and not has(log, "k_slab_part") and has(log, "k_slab_"), log
        assert call is s.lib.spmv_csr_batch or not any(TABLE in line for line in log), log
    s.so.stub_capturing(0)
    rc, log = s.calls(s.lib.spx_backward, H, B, G, X, dX, dv, None)
    assert rc == 0 and sum("k_slab_part" in line for line in log) == 2
    assert sum(TABLE in line for line in log) == 2, log
    s.so.stub_capturing(mode)
    rc, log = s.calls(s.lib.spx_backward, H, B, G, X, dX, dv, None)
    assert rc == 0 and kernels(log) == log and sum(TABLE in line for line in log) == 2, log


def workspace_for_a_captured_call(s):
    """A forward through the slabs keeps the workspace where the backward, or a
    smaller batch, needs it: a call captured next cannot allocate. Where the
    slabs take them all it allocates nothing."""
    for m, n, per_row, B, keeps in ((16384, 4096, 205, 64, False), (65536, 4096, 64, 8, False), (65536, 1000, 2, 8, False),
                                    (100000, 4096, 8, 8, True), (16384, 4096, 8, 4, True)):
        H = s.matrix(m, n, per_row)
        rc, log = s.calls(s.lib.spmv_csr_batch, H, B, 1 << 50, 1 << 51, None)
        if not has(log, "k_slab_gather"):  # its own workspace
            assert has(log, "malloc")
            continue
        assert rc == 0 and has(log, "malloc") == keeps, (m, n, per_row, log)
        s.so.stub_capturing(ALLOCATION_REFUSED)
        for b in range(1, B + 1):
            for f, args in ((s.lib.spmv_csr_batch, ()), (s.lib.spmv_csr_transpose, ()), (s.lib.dvals_pattern, (1 << 52,)),
                            (s.lib.spx_backward, (1 << 52, 1 << 53))):
                assert s.calls(f, H, b, 1 << 50, 1 << 51, *args, None)[0] == 0, (m, n, per_row, b, f.__name__)
        s.so.stub_capturing(0)


def block_bounds_without_memory(s):
    """No memory for the tables of bounds: the kernels search for them, and the
    tables are not tried again."""
    m, n, B = 8192, 600, 64
    H = s.matrix(m, n, 200)
    X, G, dX, dv = (s.zeros(4 * k) for k in (B * n, B * m, B * n, m * 200))
    s.so.stub_fail_sizes(2 * n * 4, 2 * m * 4)
    rc, log = s.calls(s.lib.spx_backward, H, B, G, X, dX, dv, None)
    assert rc == 0 and sum("malloc-failed" in line for line in log) == 2
    for _ in range(2):
        assert has(log, "k_slab_gather") and has(log, "k_slab_dots") and not any(TABLE in line for line in log), log
        rc, log = s.calls(s.lib.spx_backward, H, B, G, X, dX, dv, None)
        assert rc == 0 and kernels(log) == log


def layer_products_in_place(s):
    """A result that shares memory with an operand (a square layer in place,
    gradients over G or X): the kernels that copy the operand first, and with
    dX over G both gradients from the one copy of G."""
    n, B = 2048, 64
    H = s.matrix(n, n, 200)
    X, G, dX, dv = (s.zeros(4 * k) for k in (B * n, B * n, B * n, 200 * n))

    def ran(f, *args):
        rc, log = s.calls(f, H, B, *args, None)
        assert rc == 0, s.lib.spx_last_error()
        return [line for line in kernels(log) if "k_slab_part" not in line]

    # apart, through the slabs
    assert all("k_slab" in k for k in ran(s.lib.spmv_csr_batch, X, G) + ran(s.lib.spmv_csr_transpose, G, dX) +
               ran(s.lib.dvals_pattern, G, X, dv) + ran(s.lib.spx_backward, G, X, dX, dv))
    last = 4 * (B * n - 1)
    for f, args in ((s.lib.spmv_csr_batch, (X, X)), (s.lib.spmv_csr_batch, (X, X + last)),
                    (s.lib.spmv_csr_transpose, (G, G)), (s.lib.spmv_csr_transpose, (G + last, G)),
                    (s.lib.dvals_pattern, (dv, X, dv)), (s.lib.dvals_pattern, (G, dv + 4, dv)),
                    (s.lib.spx_backward, (G, None, G, None)), (s.lib.spx_backward, (G, X, G, dv))):
        log = ran(f, *args)
        assert has(log[:1], "k_transpose") and not has(log, "k_slab"), (f.__name__, log)
    # one copy of G, made before dX
    assert sum("k_transpose" in k for k in log) == 2 and has(log[1:2], "k_seg_gather"), log
    # a gradient that is apart goes through the slabs
    log = ran(s.lib.spx_backward, dv, X, dX, dv)
    assert has(log[:1], "k_slab_gather") and has(log[1:], "k_transpose") and has(log[-1:], "k_sddmm"), log


def layer_kernel_by_size(s):
    """Forward and dX go to the faster kernel, where one is much the faster
    on the GPU: few entries per segment and slab, many batch rows, 8-byte
    values and many slabs belong to the gather from L2."""
    L2, SLAB = "k_seg_gather", "k_slab_gather"
    for m, n, per_row, dtype, want in (
            (300000, 4096, 8, s.L.F32, {("fwd", 8): SLAB, ("fwd", 64): L2, ("fwd", 256): L2}),
            (100000, 1024, 16, s.L.F64, {("fwd", 4): SLAB, ("fwd", 64): L2}),
            (100000, 1024, 128, s.L.F64, {("fwd", 64): SLAB}),
            (16384, 8192, 8, s.L.F32, {("fwd", 8): SLAB, ("fwd", 64): L2}),
            (2000, 1024, 8, s.L.F32, {("fwd", 1): SLAB, ("fwd", 64): SLAB, ("fwd", 256): SLAB}),
            (16384, 4096, 205, s.L.F32, {("fwd", 64): SLAB, ("dX", 64): SLAB}),
            (65536, 1000, 2, s.L.F32, {("dX", 1): L2, ("dX", 64): L2}),
            (65536, 1000, 31, s.L.F32, {("dX", 1): SLAB, ("dX", 64): SLAB}),
            (65536, 16384, 32, s.L.F64, {("dX", 1): SLAB, ("dX", 64): L2})):
        H = s.matrix(m, n, per_row, dtype)
        for (what, B), kernel in want.items():
            f = s.lib.spmv_csr_batch if what == "fwd" else s.lib.spmv_csr_transpose
            # (nothing reads or writes the operands here)
            rc, log = s.calls(f, H, B, 1 << 50, 1 << 51, None)
            assert rc == 0 and has(log, kernel) and not has(log, L2 if kernel == SLAB else SLAB), (m, n, per_row, B, log)


def values_gradient_by_size(s):
    """The gradient of the values, likewise: with more batch rows than a slab
    holds it takes workgroups for half the chip and 16 entries per row and
    block of columns."""
    for m, n, per_row, dtype, slabs, gather in (
            (2000, 256, 256, s.L.F32, (1, 64), (65, 256)),   # 32 workgroups
            (2000, 256, 256, s.L.F64, (1, 32), (33, 64)),
            (16384, 1024, 16, s.L.F32, (64,), (256,)),       # 8 entries per row and block
            (16384, 1024, 32, s.L.F32, (64, 256), ()),
            (100000, 256, 16, s.L.F64, (32, 64, 256), ()),
            (2000, 4096, 128, s.L.F32, (64, 256), ())):
        H = s.matrix(m, n, per_row, dtype)
        s.calls(s.lib.dvals_pattern, H, 1, 1 << 50, 1 << 51, 1 << 52, None)
        for B in slabs + gather:
            rc, log = s.calls(s.lib.dvals_pattern, H, B, 1 << 50, 1 << 51, 1 << 52, None)
            assert rc == 0 and has(log, "k_slab_dots") == (B in slabs) and has(log, "k_sddmm") == (B in gather), \
                (m, n, per_row, B, log)


def batch_table(s, without_memory):
    """run_batch's table of column segments: where its memory is refused the
    products go by atomics and it is not tried again; where its build fails
    the next call builds it."""
    m, n, B = 40000, 64, 2  # three blocks of 16384 rows
    H = s.matrix(m, n, 8)
    args = (H, B, 6, s.array(C.c_int32, [0, 3, 6]), s.array(C.c_int32, [0, 1, 2] * 2), s.zeros(24), s.zeros(4 * B * m),
            None)
    if without_memory:
        s.so.stub_fail_sizes(4 * (3 * n + 1), 4 * (3 * n + 1))
        rc, log = s.calls(s.lib.run_batch, *args)
        assert rc == 0 and has(log, "malloc-failed") and has(log, "k_batch_phase"), log
        rc, log = s.calls(s.lib.run_batch, *args)
        assert rc == 0 and kernels(log) == log and has(log, "k_batch_phase"), log
    else:
        s.so.stub_fail_launch(b"k_segs", 0)
        assert s.calls(s.lib.run_batch, *args)[0] == -7
        rc, log = s.calls(s.lib.run_batch, *args)
        assert rc == 0 and has(log, "k_segs") and has(log, "k_batch_rows"), log


def refresh(s):
    """Below 96 blocks of 16384 entries every refresh is a launch. From there
    on the first one is. The second one orders the permutation by
    blocks (it allocates and waits), unless it is being captured; from then on
    a refresh is a launch again."""
    H = s.matrix(1 << 14, 300, 95)
    for _ in range(3):
        rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
        assert rc == 0 and len(log) == 1 and has(log, "k_gather_perm"), log
    H = s.matrix(1 << 14, 300, 96)
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and len(log) == 1 and has(log, "k_gather_perm"), log
    s.so.stub_capturing(ALLOCATION_ALLOWED)
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and len(log) == 1 and has(log, "k_gather_perm"), log
    s.so.stub_capturing(0)
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and has(log, "k_perm_keys") and has(log, "sync") and has(log[-1:], "k_gather_blocks"), log
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and len(log) == 1 and has(log, "k_gather_blocks"), log


def refresh_without_memory(s):
    H = s.matrix(1 << 14, 300, 96)
    assert s.calls(s.lib.spx_matrix_values_updated, H, None)[0] == 0
    s.so.stub_fail_sizes(3 << 20, 3 << 20)  # the 16-bit half of the ordered permutation
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and has(log, "malloc-failed") and has(log[-1:], "k_gather_perm"), log
    rc, log = s.calls(s.lib.spx_matrix_values_updated, H, None)
    assert rc == 0 and len(log) == 1 and has(log, "k_gather_perm"), log


def ranking_that_fails_with_a_count_to_come(s):
    """The product queued behind a round's select fails: the call waits for
    the select, whose total would else reach the word that the next call
    waits on."""
    m = 64
    H = s.matrix(m, m, 16)
    rank = s.zeros(4 * m)
    plan = s.L.Plan(s.L.PAT_SPMV, s.L.DIST_BALANCED, s.L.WB_NONE, 0, 0, 0)
    iters = C.c_int32()
    args = lambda products: (H, 0.85, 1e-6, products, C.byref(plan), rank, None, C.byref(iters), None, 0, None)
    assert s.calls(s.lib.spx_pagerank, *args(0))[0] == 0  # the column sums
    s.so.stub_total(80 << 32 | 5)
    s.so.stub_total(80 << 32 | 5)
    s.so.stub_fail_launch(b"k_csr_merge", 1)
    rc, log = s.calls(s.lib.spx_pagerank, *args(5))
    assert rc == -7 and sum("k_pr_select" in line for line in log) == 2
    select = max(i for i, line in enumerate(log) if "k_pr_select" in line)
    assert has(log[select:], "k_csr_merge") and has(log[select:], "sync"), log
    # and a ranking that ends by itself does not wait for the last product
    s.so.stub_total(0)
    rc, log = s.calls(s.lib.spx_pagerank, *args(5))
    assert rc == 0 and iters.value == 0 and kernels(log) == log


SCENARIOS = {
    "workspace_for_a_captured_call": workspace_for_a_captured_call,
    "values_gradient_by_size": values_gradient_by_size,
    "layer_kernel_by_size": layer_kernel_by_size,
    "layer_products_in_place": layer_products_in_place,
    "batch_table_without_memory": lambda s: batch_table(s, True),
    "batch_table_not_built": lambda s: batch_table(s, False),
    "refresh": refresh,
    "refresh_without_memory": refresh_without_memory,
    "ranking_that_fails_with_a_count_to_come": ranking_that_fails_with_a_count_to_come,
    "block_bounds_captured_no_allocation": lambda s: block_bounds_under_capture(s, ALLOCATION_REFUSED),
    "block_bounds_captured_allocation": lambda s: block_bounds_under_capture(s, ALLOCATION_ALLOWED),
    "block_bounds_without_memory": block_bounds_without_memory,
}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_stub.cpp"), "-o", path],
                   check=True)
    return path


@pytest.mark.parametrize("name", SCENARIOS)
def test_host_calls(name, stub):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), name, stub], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    SCENARIOS[sys.argv[1]](Stub(sys.argv[2]))
