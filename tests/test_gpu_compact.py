"""tsp_compact_zeros and tsp_compact_zeros_static against numpy, on row pointers that chunks of entries could get wrong: rows
that begin behind the first entry and end before the last (a slice of a matrix), many more rows than entries, runs of empty
rows either side of what one block finds, and pointers that go down.  Needs an MI355X."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PART, ROWS = 4096, 4096                  # entries of a part and rows of a block in csrc/compact.hip


@pytest.fixture(scope="module")
def tsp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_14600_amd import tsp as binding
    binding.load_library()
    return binding


def _expected(row_ptr, col, val):
    starts = np.maximum.accumulate(np.clip(np.array([int(x) for x in row_ptr], dtype=object), 0, val.size).astype(np.int64))
    keep = ~(val == 0)
    keep[:starts[0]] = keep[starts[-1]:] = False
    before = np.concatenate([[0], np.cumsum(keep)])
    return before[starts], col[keep], val[keep]


def _check(tsp, what, row_ptr, nnz, i64=True, seed=0):
    import torch
    rng = np.random.default_rng(seed)
    print(f"compaction: {what}, {len(row_ptr) - 1} rows, {nnz} entries", flush=True)
    val = np.where(rng.random(nnz) < 0.3, 0.0, rng.uniform(0.5, 1, nnz)).astype(np.float32)
    val[::97] = np.nan
    val[5::101] = -0.0
    col = np.arange(nnz, dtype=np.int32)
    want = _expected(row_ptr, col, val)
    dev = [torch.from_numpy(x).cuda() for x in (np.array([int(x) for x in row_ptr], dtype=np.int64 if i64 else np.int32), col, val)]
    h = tsp.Handle()
    try:
        A = tsp.DeviceCSR(len(row_ptr) - 1, max(nnz, 1), *dev)
        for static in (False, True):
            if static:
                if A.rows < 1:
                    continue
                out = [torch.full((A.rows + 1,), -7, dtype=torch.int64, device="cuda"), torch.zeros(max(nnz, 1), dtype=torch.int32, device="cuda"),
                       torch.zeros(max(nnz, 1), dtype=torch.float32, device="cuda")]
                n = h.compact_zeros_static(A, *out)
                got = [out[0].cpu().numpy(), out[1][:n].cpu().numpy(), out[2][:n].cpu().numpy()]
            else:
                C = h.compact_zeros(A)
                n, got = C.nnz, C.to_host()
                C.free()
            assert n == want[2].size
            for x, y in zip(got, want):
                assert np.array_equal(x, y, equal_nan=x.dtype == np.float32), (what, static)
    finally:
        h.close()


def _pointers(lengths, first=0):
    return first + np.concatenate([[0], np.cumsum(lengths)])


@pytest.mark.parametrize("i64", [False, True])
@pytest.mark.parametrize("first,slack", [(1, 0), (0, 1), (PART, PART), (PART - 1, 3 * PART + 1), (17, 5000), (9 * PART + 5, 0)])
def test_a_slice_of_rows(tsp, i64, first, slack):
    rng = np.random.default_rng(first + slack)
    p = _pointers(rng.integers(0, 30, 700), first)
    _check(tsp, "slice", p, int(p[-1]) + slack, i64)
    _check(tsp, "slice without entries", np.full(9, first), first + slack + 1, i64)


@pytest.mark.parametrize("empty", [900, 3000, ROWS - 1, ROWS, ROWS + 1, 3 * ROWS + 5, 100001])
@pytest.mark.parametrize("entries", [0, 1, PART, 2 * PART + 9])
def test_runs_of_empty_rows(tsp, empty, entries):
    full = np.full(entries, 1)
    none = np.zeros(empty, np.int64)
    for what, lengths in (("behind", [full, none]), ("in front", [none, full]), ("between", [full[:entries // 2], none, full[entries // 2:], none, full])):
        p = _pointers(np.concatenate(lengths).astype(np.int64), 3)
        _check(tsp, f"empty rows {what}", p, int(p[-1]) + 2, seed=entries)
        _check(tsp, f"empty rows {what}, whole parts", p - 3, int(p[-1]) - 3, seed=entries)


@pytest.mark.parametrize("i64", [False, True])
@pytest.mark.parametrize("seed", range(6))
def test_row_pointers_that_go_down(tsp, i64, seed):
    rng = np.random.default_rng(seed)
    p = [int(x) for x in _pointers(rng.integers(0, 30, 1500))]
    nnz = p[-1]
    far = 2 ** 62 if i64 else 2 ** 31 - 1
    for _ in range(1 + 3 * seed):
        p[int(rng.integers(0, len(p)))] = int(rng.choice([-far, far, 0, nnz, int(rng.integers(0, nnz)), -1, nnz + 1]))
    _check(tsp, "pointers that go down", p, nnz, i64, seed)
    _check(tsp, "negative and none", [-5, -7, 0, 0], 2 * PART, i64)


@pytest.mark.parametrize("nnz", [0, 1, PART - 1, PART, PART + 1, 64 * PART, 70 * PART + 3, 200 * PART + 1])
def test_matrices_of_sizes_met_before(tsp, nnz):
    """One handle and one size: few zeros and many, none and nothing else, rows of all kinds, row pointers that go down; each into
    arrays sized after the matrix before it, and without allocation.  As many parts as a group of blocks, fewer and more."""
    import torch
    rows, rng = 2 * ROWS + 77, np.random.default_rng(nnz)

    def pointers(lengths):
        return np.concatenate([[0], np.sort(rng.integers(0, nnz + 1, rows - 1)) if lengths is None else np.minimum(np.cumsum(lengths)[:-1], nnz), [nnz]])

    spread = pointers(None)
    down = spread.copy()
    down[rows // 2] = 0
    run = pointers(np.where(np.arange(rows) < rows // 3, 0, 3 * nnz // rows + 1))
    h = tsp.Handle()
    try:
        for what, share, p in (("first", 0.3, spread), ("as many", 0.3, spread), ("fewer zeros", 0.1, spread), ("more", 0.8, spread), ("none", 0.0, spread),
                               ("none again", 0.0, spread), ("some", 0.2, run), ("a run of empty rows", 0.2, run), ("down", 0.2, down), ("all", 1.0, run),
                               ("after all", 0.5, spread), ("at last", 0.5, spread)):
            val = np.where(rng.random(nnz) < share, 0.0, rng.uniform(0.5, 1, nnz)).astype(np.float32)
            col = np.arange(nnz, dtype=np.int32)
            want = _expected(p, col, val)
            dev = [torch.from_numpy(x).cuda() for x in (p.astype(np.int64), col, val)]
            A = tsp.DeviceCSR(rows, max(nnz, 1), *dev)
            C = h.compact_zeros(A)
            out = [torch.full((rows + 1,), -7, dtype=torch.int64, device="cuda"), torch.full((max(nnz, 1),), -7, dtype=torch.int32, device="cuda"),
                   torch.full((max(nnz, 1),), -7.0, dtype=torch.float32, device="cuda")]
            n = h.compact_zeros_static(A, *out)
            assert n == C.nnz == want[2].size, what
            for got in (C.to_host(), [out[0].cpu().numpy(), out[1][:n].cpu().numpy(), out[2][:n].cpu().numpy()]):
                for x, y in zip(got, want):
                    assert np.array_equal(x, y), what
            assert not nnz or bool((out[1][n:] == -7).all()) and bool((out[2][n:] == -7.0).all()), what    # (nothing behind them)
            C.free()
    finally:
        h.close()


@pytest.mark.parametrize("parts", [16384 - 2, 16384 - 1, 16384])
def test_as_many_parts_as_the_copying_blocks_add_up(tsp, parts):
    """Either side of the number of counts (one of them of the rows) that the copying blocks add up themselves; the second time into
    arrays sized after the first."""
    import torch
    nnz = parts * PART - 7
    col = torch.arange(nnz, dtype=torch.int32, device="cuda")
    row_ptr = torch.tensor([0, nnz // 3, nnz], device="cuda")
    h = tsp.Handle()
    try:
        for every in (3, 3, 2):
            val = (col % every != 0).float()
            keep = torch.nonzero(val).flatten().int()
            C = h.compact_zeros(tsp.DeviceCSR(2, nnz, row_ptr, col, val))
            assert C.nnz == keep.numel()
            assert torch.equal(C.col_idx[:C.nnz], keep) and bool((C.val[:C.nnz] == 1).all())
            assert C.row_ptr.tolist() == [0, int((val[:nnz // 3] != 0).sum()), keep.numel()]
            C.free()
    finally:
        h.close()


@pytest.mark.parametrize("nnz", [20, PART - 1, PART, PART + 1, 3 * PART + 5])
@pytest.mark.parametrize("zero", [0, -1, 7])
def test_nothing_to_drop_after_a_product_that_lost_entries(tsp, nnz, zero):
    """Products with the compaction, one that loses an entry (the first of all, the last, one of a few) or several and one of the same
    sizes that loses none: that one copies nothing into the arrays it was given ahead, and keeps those of the multiplication."""
    import torch
    from paper_2009_14600_amd import inputs
    rows, cols = 97, 300
    rng = np.random.default_rng(nnz)
    key = np.sort(rng.choice(rows * cols, nnz, replace=False))
    A = inputs.from_coo(rows, cols, key // cols, key % cols, rng.uniform(0.5, 1, nnz), "left")
    unit = tsp.to_device(inputs.from_coo(cols, cols, np.arange(cols), np.arange(cols), np.ones(cols), "unit"))
    whole, one, several = tsp.to_device(A), tsp.to_device(A), tsp.to_device(A)
    one.val[zero] = 0
    several.val[::3] = 0
    h = tsp.Handle()
    try:
        h.set_option(tsp.OPT_COMPACT_ZEROS, 1)
        for M in (whole, one, one, whole, whole, several, several, whole, one):
            h.trim()                                           # (no block that holds what an earlier product has left)
            C = h.spgemm(M, unit)
            want = M.val.cpu().numpy().astype(np.float32)
            keep = want != 0
            row_ptr, col, val = C.to_host()
            assert np.array_equal(row_ptr, np.concatenate([[0], np.cumsum(keep)])[A.row_ptr])
            assert np.array_equal(col, A.col_idx[keep]) and np.array_equal(val, want[keep])
            if M is whole:                                     # (ahead there is room for two thirds of it at least)
                bits, n = C.col_idx.view(torch.uint8), 4 * (nnz // 2)
                assert sum(1 for block in h._blocks.values() if block.numel() >= n and bool((block[:n] == bits[:n]).all())) == 1
            C.free()
    finally:
        h.close()


@pytest.mark.parametrize("descends", [False, True])
def test_more_left_than_last_time_again_and_again(tsp, descends):
    """Matrices of the same sizes with many zeros, and with few (or with a row pointer that goes down), in turn: after one that did not
    fit what was launched ahead nothing is, until four have come one behind the other that would have fitted.  (Seen by the bytes that
    a call takes: those of a copy ahead have room for a sixteenth more, and one in vain leaves its arrays.)"""
    import torch
    rng = np.random.default_rng(3)
    rows, n = 500, 3 * PART + 77
    row_ptr = np.sort(np.concatenate([[0, n], rng.integers(0, n, rows - 1)])).astype(np.int64)
    other_ptr = row_ptr.copy()
    if descends:
        other_ptr[200] = 0
    made = []
    for pointers, share in ((row_ptr, 0.5), (other_ptr, 0.5 if descends else 0.1)):
        val = np.where(rng.random(n) < share, 0, rng.uniform(0.5, 1, n)).astype(np.float32)
        col = np.arange(n, dtype=np.int32)
        made.append((tsp.DeviceCSR(rows, n, *(torch.from_numpy(x).cuda() for x in (pointers, col, val))), _expected(pointers, col, val)))
    h = tsp.Handle()
    try:
        def blocks(k):
            C, want = made[k]
            h.trim()
            before = set(h._blocks)
            out = h.compact_zeros(C)
            new = sum(h._blocks[p].numel() for p in set(h._blocks) - before)
            for x, y in zip(out.to_host(), want):
                assert np.array_equal(x, y)
            out.free()
            return new

        plain, few = blocks(0), blocks(0)                      # (the second into arrays for a sixteenth more)
        assert few > plain
        missed = blocks(1)
        assert [blocks(0) for _ in range(3)] == [plain] * 3
        assert blocks(1) < missed
        assert [blocks(0) for _ in range(6)] == [plain] * 4 + [few] * 2
    finally:
        h.close()
