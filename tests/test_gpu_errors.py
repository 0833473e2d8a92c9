"""Error paths of the C ABI, forced from the host: every condition here is one the library detects itself
(on the host, or through its own range checks on the device), so every kernel still runs to its end.
Needs an MI355X."""
import ctypes

import numpy as np
import pytest

from paper_2009_14600_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tsp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_14600_amd import tsp as binding
    binding.load_library()
    return binding


class _FailingHandle:
    """A handle whose allocator callback returns NULL from its k-th call on (k counted from 0), or for blocks larger than
    most_bytes."""

    def __init__(self, tsp, fail_from, most_bytes=1 << 62):
        import torch
        self.calls = 0
        self.refused = 0
        self.fail_from = fail_from
        self.blocks = {}

        def alloc(_user, nbytes, _stream):
            k = self.calls
            self.calls += 1
            if k >= self.fail_from or nbytes > most_bytes:
                self.refused += 1
                return None
            t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
            self.blocks[t.data_ptr()] = t
            return t.data_ptr()

        def free(_user, ptr, _stream):
            self.blocks.pop(ptr, None)

        self._cb = (tsp._ALLOC_FN(alloc), tsp._FREE_FN(free))
        self._allocator = tsp._Allocator(self._cb[0], self._cb[1], None)
        self.lib = tsp.load_library()
        self.h = ctypes.c_void_p()
        assert self.lib.tsp_create(ctypes.byref(self.h), ctypes.byref(self._allocator)) == 0

    def close(self):
        self.lib.tsp_destroy(self.h)


# (WORK_ORDER keeps the tile kernels, whatever the operands)
@pytest.mark.parametrize("maker,tile_edge,work_order,by_rows", [
    (lambda: inputs.config(2, small=True), 0, 0, True),     # rows: small ones, the multiplication launched ahead on a warm handle
    (lambda: inputs.config(4, small=True), 0, 0, True),     # rows: heavy ones too
    (lambda: inputs.config(2, small=True), 0, 2, False),    # list kernel, whole-tile-row multiplication kernel
    (lambda: inputs.config(4, small=True), 0, 1, False),    # general task-list kernel, separate counting kernel, order kept
    (lambda: inputs.config(5, small=True), 0, 0, False),    # list kernel with a block per tile-row, full tiles
    (lambda: inputs.config(1, small=True), 8, 0, False),    # the paper's pipeline (tsp_spgemm_paper) at two tile edges
    (lambda: inputs.config(5, small=True), 32, 0, False),
])
@pytest.mark.parametrize("warm", [False, True])
def test_allocator_returning_null_at_every_call_site(tsp, maker, tile_edge, work_order, by_rows, warm):
    """tsp_spgemm (tile_edge 0) or tsp_spgemm_paper with an allocator that runs dry after k calls, for every k
    up to the number of calls a successful product makes: status -4 (TSP_ERR_ALLOC_FAILED), *C zeroed, nothing
    leaked (after tsp_trim the handle holds no byte and the allocator has every block back), and the handle
    works again once memory is there.  On a new handle, and on one that has multiplied these operands twice and given its
    cached memory back: it sizes arrays and launches kernels by what it remembers."""
    import torch
    A = maker()
    dA = tsp.to_device(A)
    sA = dA._struct()

    def multiply(handle, out):
        if tile_edge:
            return handle.lib.tsp_spgemm_paper(handle.h, tile_edge, ctypes.byref(sA), ctypes.byref(sA), ctypes.byref(out), None)
        return handle.lib.tsp_spgemm(handle.h, ctypes.byref(sA), ctypes.byref(sA), ctypes.byref(out), None)

    def trimmed(handle):
        assert handle.lib.tsp_trim(handle.h, None) == 0
        st = tsp._Stats()
        assert handle.lib.tsp_get_stats(handle.h, ctypes.byref(st)) == 0
        return st

    def good(handle):
        out = tsp._Csr()
        assert multiply(handle, out) == 0
        torch.cuda.synchronize()
        nnz = out.nnz
        assert handle.lib.tsp_csr_free(handle.h, ctypes.byref(out), None) == 0
        return nnz

    def new_handle():
        h = _FailingHandle(tsp, fail_from=1 << 30)
        assert h.lib.tsp_set_option(h.h, tsp.OPT_WORK_ORDER, work_order) == 0
        if warm:
            good(h), good(h), trimmed(h)
        h.calls = 0
        return h

    ok = new_handle()
    want_nnz, calls = good(ok), ok.calls
    # what a handle keeps for its whole life (the slots of its chained prefix sums, an order of the tile-rows), to tell it
    # from a leak
    st = trimmed(ok)
    kept_bytes, kept_blocks = st.workspace_bytes, len(ok.blocks)
    assert kept_blocks <= 1 + (work_order == 1)
    if not tile_edge:
        assert (st.pairs == 0) == by_rows
    ok.close()
    assert calls >= 10
    for k in range(calls):
        h = new_handle()
        h.fail_from = k
        out = tsp._Csr(7, 7, 7, 1, 1, 1, 1, 1)
        status = multiply(h, out)
        torch.cuda.synchronize()
        assert status == -4, (k, status)
        assert (out.rows, out.cols, out.nnz, out.row_ptr, out.col_idx, out.val) == (0, 0, 0, None, None, None), k
        st = trimmed(h)
        assert st.workspace_bytes <= kept_bytes and len(h.blocks) <= kept_blocks, (k, st.workspace_bytes, len(h.blocks))
        # memory comes back: the same handle multiplies
        h.fail_from = 1 << 30
        assert good(h) == want_nnz
        h.close()


@pytest.mark.parametrize("what,most_bytes", [("entries of the small rows", 2 << 20), ("pattern of the heavy rows", 1 << 20)])
def test_row_kernels_without_the_memory_they_ask_for(tsp, oracle, what, most_bytes):
    """An allocator that refuses large blocks: a product by rows whose small rows ask for more goes by tiles, one whose heavy
    rows do takes them some at a time; on a new handle, and on one that knows the product."""
    import torch
    rng = np.random.default_rng(3)
    if what.startswith("entries"):                  # 20000 rows of one entry: 3.8 MB, everything else less than 1 MB
        n = 20000
        A = inputs.from_coo(n, n, np.arange(n), rng.integers(0, n, n), rng.uniform(-1, 1, n))
        B = A
    else:                                           # 400 rows of 17 entries, 70001 columns: a pattern of 3.7 MB
        A = inputs.from_coo(400, 500, np.repeat(np.arange(400), 17), np.concatenate([np.sort(rng.choice(500, 17, replace=False)) for _ in range(400)]),
                            rng.uniform(-1, 1, 400 * 17))
        B = inputs.from_coo(500, 70001, np.repeat(np.arange(500), 2), np.sort(rng.integers(0, 35000, (500, 2)) * 2 + [0, 1], axis=1).ravel(),
                            rng.uniform(-1, 1, 1000))
    want = oracle.spgemm(A, B, threads=2)
    dA = tsp.to_device(A)
    dB = dA if B is A else tsp.to_device(B)
    sA, sB = dA._struct(), dB._struct()

    def multiply(h):
        out, st = tsp._Csr(), tsp._Stats()
        status = h.lib.tsp_spgemm(h.h, ctypes.byref(sA), ctypes.byref(sA if B is A else sB), ctypes.byref(out), None)
        torch.cuda.synchronize()
        assert status == 0 and h.lib.tsp_get_stats(h.h, ctypes.byref(st)) == 0
        got = []
        for ptr, count, dtype in ((out.row_ptr, out.rows + 1, torch.int64), (out.col_idx, out.nnz, torch.int32), (out.val, out.nnz, torch.float32)):
            got.append(h.blocks[ptr].view(dtype)[:count].cpu().numpy())
        assert h.lib.tsp_csr_free(h.h, ctypes.byref(out), None) == 0
        assert np.array_equal(got[0], want.row_ptr) and np.array_equal(got[1], want.col)
        assert np.all(np.abs(got[2].astype(np.float64) - want.val) <= 1e-5 * want.mag + 1e-7)
        return st.pairs

    plenty = _FailingHandle(tsp, fail_from=1 << 30)
    assert multiply(plenty) == 0 and plenty.refused == 0
    plenty.close()
    h = _FailingHandle(tsp, fail_from=1 << 30, most_bytes=most_bytes)
    for _ in range(3):
        refused = h.refused
        assert (multiply(h) == 0) == what.startswith("pattern")
        assert h.refused > refused
    h.close()


def test_index_overflow_and_unsupported_span(tsp):
    """-5 (TSP_ERR_INDEX_OVERFLOW): a matrix with 2^31 rows, refused on the host before any array is
    touched.  -7 (TSP_ERR_UNSUPPORTED): a tile-row of C whose candidates lie more than 131072 tile columns
    apart (here 187500), found by the counting kernel's own range check; the handle works afterwards."""
    import torch
    handle = tsp.Handle(validate=True)
    small = tsp.to_device(inputs.random_sparse(20, 20, 0.2, 1))
    s = small._struct()
    huge = tsp._Csr(1 << 31, s.cols, s.nnz, s.row_ptr, s.col_idx, s.val, s.row_ptr_type, s.val_type)
    out = tsp._Csr()
    assert handle._lib.tsp_spgemm(handle._h, ctypes.byref(huge), ctypes.byref(s), ctypes.byref(out), handle._stream()) == -5
    many = tsp._Csr(s.rows, s.cols, 1 << 31, s.row_ptr, s.col_idx, s.val, s.row_ptr_type, s.val_type)
    assert handle._lib.tsp_spgemm(handle._h, ctypes.byref(many), ctypes.byref(s), ctypes.byref(out), handle._stream()) == -5
    N = 3_000_000
    A = inputs.from_coo(16, 16, [0, 3], [0, 5], [1.0, 2.0])
    B = inputs.from_coo(16, N, [0, 0, 5], [0, N - 1, 77], [1.0, 1.0, 1.0])
    with pytest.raises(tsp.TspError) as e:
        handle.spgemm(tsp.to_device(A), tsp.to_device(B))
    assert e.value.status == -7
    C = handle.spgemm(small, small)
    assert C.nnz > 0
    C.free()
    handle.close()
