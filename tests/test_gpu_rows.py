"""The row kernels (csrc/rowwise.hip), which tsp_spgemm takes for operands with little in their tiles, against the CPU
oracle at the sizes where they can go wrong: the bounds of merged rows, the windows of columns, the span of one block's
bitmap, workspaces kept from a product of the same sizes.  Needs an MI355X."""
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


def _matrix(rng, rows, cols, per_row, name="", dense=()):
    """About per_row (a number or one per row) entries per row at random columns; the rows in `dense` get 40 times as many."""
    want = np.broadcast_to(np.asarray(per_row), (rows,)).copy()
    for r in dense:
        want[r % rows] *= 40
    r = np.repeat(np.arange(rows), want)
    key = np.unique(r * cols + rng.integers(0, cols, r.size))
    return inputs.from_coo(rows, cols, key // cols, key % cols, rng.uniform(-1, 1, key.size), name)


def _check(h, tsp, oracle, A, B=None, by_rows=True, calls=2, **upload):
    print(f"rows: {A.name} {A.rows}x{A.cols}x{(B or A).cols}, nnz {A.nnz}, {(B or A).nnz}", flush=True)
    dA = tsp.to_device(A, **upload)
    dB = dA if B is None else tsp.to_device(B, **upload)
    ref = oracle.spgemm(A, A if B is None else B, threads=4)
    first = None
    for _ in range(calls):                       # (from the second call on with what the handle kept of the first)
        C = h.spgemm(dA, dB)
        if by_rows is not None:
            assert (h.stats()["pairs"] == 0) == by_rows
        row_ptr, col, val = C.to_host()
        C.free()
        assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
        assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
        if first is not None:
            assert np.array_equal(first.view(np.uint32), val.view(np.uint32))       # runs are bit-identical
        first = val


# entries per row of A and of B either side of the bounds of merged rows (8 and 16 entries, 256 products), of the lanes
# per segment in the sizing pass, and of one load per segment
@pytest.mark.parametrize("a_row,b_row", [(1, 1), (8, 3), (16, 4), (16, 12), (3, 40), (8, 32), (8, 33), (9, 20), (16, 16), (16, 17), (17, 3), (40, 70), (5, 300)])
def test_bounds_of_small_rows(tsp, oracle, a_row, b_row):
    rng = np.random.default_rng(100 * a_row + b_row)
    h = tsp.Handle()
    try:
        A = _matrix(rng, 300, 3001, rng.integers(0, a_row + 1, 300), "ragged left", dense=(7,))
        A2 = _matrix(rng, 300, 3001, a_row, "even left")
        B = _matrix(rng, 3001, 3001, b_row, "right")
        _check(h, tsp, oracle, A, B, value_dtype="f32", row_ptr_dtype="i64")
        _check(h, tsp, oracle, A2, B)
    finally:
        h.close()


@pytest.mark.parametrize("cols", [1, 33, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 16385, 70001, 393216, 393217, 900001])
def test_windows_of_columns(tsp, oracle, cols):
    """Narrow results in one window of 2048 or of 4096 columns, wide ones in many, and beyond the columns whose bits
    one block of the sizing pass holds; light, heavy and very heavy rows (several tasks) side by side."""
    rng = np.random.default_rng(cols)
    h = tsp.Handle()
    try:
        A = _matrix(rng, 259, 900, rng.integers(0, 40, 259), "left", dense=(0, 100, 258))
        B = _matrix(rng, 900, cols, min(60, cols), "right", dense=(3, 899) if cols > 100 else ())
        _check(h, tsp, oracle, A, B, by_rows=None if cols < 100 else True)
    finally:
        h.close()


def test_same_sizes_another_structure(tsp, oracle):
    """Operands of the same sizes as the last product's, with more and with fewer heavy rows than the kept lists hold,
    and some that suit the tile kernels."""
    n, rng = 1600, np.random.default_rng(5)
    even = np.full(n, 6)
    skewed = np.full(n, 2)
    skewed[::40] = 162                            # the same number of entries, 40 heavy rows
    more = np.full(n, 3)
    more[::80] = 243                              # 20 of them
    h = tsp.Handle()
    try:
        def exact(lengths):
            cols = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths])
            return inputs.from_coo(n, n, np.repeat(np.arange(n), lengths), cols, rng.uniform(-1, 1, cols.size))
        for lengths in (even, skewed, more, skewed, even):
            A = exact(lengths)
            assert A.nnz == 6 * n
            _check(h, tsp, oracle, A, calls=1)
        block = inputs.block_clustered(8192, seed=9)
        _check(h, tsp, oracle, block, by_rows=False)
        _check(h, tsp, oracle, exact(even))
    finally:
        h.close()


@pytest.mark.parametrize("cols,kept_rows", [(1600, 0), (1600, 1), (1600, 30), (1600, 64), (9000, 30)])
def test_pattern_of_the_heavy_rows_kept_or_found_again(tsp, oracle, cols, kept_rows):
    """The pattern of the heavy rows within a limit of some rows: products of the same sizes with more heavy rows than that
    and with fewer, in either order (the room for the pattern follows the last product, the pattern the one at hand)."""
    n, rng = 1600, np.random.default_rng(11)
    many, few = np.full(n, 2), np.full(n, 3)
    many[::40] = 162                              # 40 heavy rows
    few[::80] = 243                               # 20, and as many entries
    assert many.sum() == few.sum()
    row_bytes = 256 if cols <= 2048 else 3 * 512  # a bit per column, in whole windows
    B = _matrix(rng, n, cols, 6, "right")
    h = tsp.Handle()
    try:
        h.set_option(tsp.OPT_PATTERN_BYTES, kept_rows * row_bytes)
        for lengths in (many, many, few, few, many, few):
            col = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths])
            A = inputs.from_coo(n, n, np.repeat(np.arange(n), lengths), col, rng.uniform(-1, 1, col.size), "left")
            _check(h, tsp, oracle, A, B, calls=1)
    finally:
        h.close()


def test_more_lanes_for_rows_of_up_to_16_entries(tsp, oracle):
    """The lanes of a small row follow the last product of the same sizes: rows of 9 and of 16 entries, small but for the
    eight lanes of a mean row, come and go."""
    n, rng = 1600, np.random.default_rng(8)
    even, nine, most = np.full(n, 4), np.full(n, 3), np.full(n, 2)
    nine[::6] = 9
    nine[1:3] -= 1
    most[::7] = 16
    most[1:4] -= 2
    assert nine.sum() == most.sum() == even.sum()
    h = tsp.Handle()
    try:
        for lengths in (even, nine, nine, even, most, most, nine):
            cols = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths])
            A = inputs.from_coo(n, n, np.repeat(np.arange(n), lengths), cols, rng.uniform(-1, 1, cols.size))
            B = inputs.random_fixed_per_row(n, 1, seed=4)
            _check(h, tsp, oracle, A, B, calls=1, by_rows=True)
    finally:
        h.close()


def _bits(h, tsp, A, B=None):
    C = h.spgemm(A, A if B is None else B)
    by_rows = h.stats()["pairs"] == 0
    out = [x.view(np.uint32) if x.dtype == np.float32 else x for x in C.to_host()]
    C.free()
    return by_rows, out


def _exact_lengths(rng, cols, lengths, values):
    col = np.concatenate([np.sort(rng.choice(cols, k, replace=False)) for k in lengths])
    return inputs.from_coo(len(lengths), cols, np.repeat(np.arange(len(lengths)), lengths), col, values(col.size), "exact lengths")


def _full_tiles(rng, n):
    """64 entries per row: four full tiles in every tile-row."""
    tile = np.sort(np.argsort(rng.random((n // 16, n // 16)), axis=1)[:, :4], axis=1)
    col = (tile[:, None, :, None] * 16 + np.arange(16)).repeat(16, axis=1).reshape(n, 64)
    return inputs.from_coo(n, n, np.repeat(np.arange(n), 64), col.ravel(), rng.normal(size=64 * n), "full tiles")


@pytest.mark.parametrize("what", ["lanes of small rows", "sums of heavy rows", "rows, then tiles", "kernels by tiles"])
def test_the_same_bits_whatever_came_before(tsp, oracle, what):
    """Products of the same sizes on one handle, in several orders and each of them repeated, against the bits of a new
    handle: what the handle has learnt of the last one may not show in the result."""
    rng = np.random.default_rng(21)
    B = None
    if what == "lanes of small rows":               # rows of up to 16 entries are small or not, by how many there are
        n = 1600
        even, nine, most = np.full(n, 4), np.full(n, 3), np.full(n, 2)
        nine[::6] = 9
        nine[1:3] -= 1
        most[::7] = 16
        most[1:4] -= 2
        all_of = [_exact_lengths(rng, n, k, lambda m: rng.normal(size=m)) for k in (even, nine, most)]
        B = _exact_lengths(rng, n, np.full(n, 8), lambda m: rng.normal(size=m))
    elif what == "sums of heavy rows":              # 32-bit integers, 64-bit integers, fp64
        n = 900
        values = [lambda m: rng.choice([-1.0, 1.0], m), lambda m: rng.uniform(-1, 1, m), lambda m: rng.normal(size=m) * 10.0 ** rng.integers(-3, 4, m)]
        all_of = [_exact_lengths(rng, n, np.full(n, 30), v) for v in values]
    elif what == "rows, then tiles":
        n = 4096
        all_of = [_exact_lengths(rng, n, np.full(n, 64), lambda m: rng.normal(size=m)), _full_tiles(rng, n)]
    else:                                           # whole tile-rows, tiles of a few entries, full tiles
        n = 1600
        r = np.arange(n)
        band = inputs.from_coo(n, n, np.repeat(r, 3), np.sort((r[:, None] + [0, 1, 2]) % n, axis=1).ravel(), rng.normal(size=3 * n), "band")
        long = np.full(n, 3)
        long[:16], long[16:792] = 100, 1            # (as many entries in all)
        all_of = [band, _exact_lengths(rng, n, np.full(n, 3), lambda m: rng.normal(size=m)), _exact_lengths(rng, n, long, lambda m: rng.normal(size=m))]
        assert len({A.nnz for A in all_of}) == 1
    dev = [tsp.to_device(A) for A in all_of]
    dB = None if B is None else tsp.to_device(B)

    def handle():
        h = tsp.Handle()
        if what == "kernels by tiles":
            h.set_option(tsp.OPT_WORK_ORDER, 2)
        return h

    want = []
    for A, dA in zip(all_of, dev):
        h = handle()
        want.append(_bits(h, tsp, dA, dB))
        ref = oracle.spgemm(A, A if B is None else B, threads=4)
        assert np.array_equal(want[-1][1][0], ref.row_ptr) and np.array_equal(want[-1][1][1], ref.col)
        assert np.all(np.abs(want[-1][1][2].view(np.float32).astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
        h.close()
    h = handle()
    try:
        k = len(dev)
        for i in (0, 0, 0, 1, 1, k - 1, k - 1, 1, 0, k - 1, 0, 0):
            print(f"{what}: product {i}", flush=True)
            by_rows, got = _bits(h, tsp, dev[i], dB)
            assert by_rows == want[i][0]
            for x, y in zip(got, want[i][1]):
                assert np.array_equal(x, y)
    finally:
        h.close()


@pytest.mark.parametrize("count", [2, 8, 9, 11])
@pytest.mark.parametrize("options", [{}, {"OPT_WORK_ORDER": 1}])
def test_products_in_turn(tsp, oracle, count, options):
    """Two and more products in turn on one handle, which remembers eight: by rows, by tiles, graphs by tiles (with an order
    of their tile-rows that the handle keeps), rectangles; every result against the oracle's, the repeated ones bit by bit."""
    rng = np.random.default_rng(count)
    all_of = []
    for i in range(count):
        if i % 4 == 0:
            all_of.append((_matrix(rng, 500 + 16 * i, 700, 5, "A"), _matrix(rng, 700, 300 + i, 4, "P")))
        elif i % 4 == 1:
            all_of.append((inputs.block_clustered(2048 + 16 * i, seed=i), None))
        elif i % 4 == 2:
            all_of.append((inputs.random_fixed_per_row(1100 + i, 12, seed=i), None))
        else:
            all_of.append((_matrix(rng, 300 + i, 500, 3, "R", dense=(1, 7)), _matrix(rng, 500, 900, rng.integers(0, 9, 500), "AP", dense=(0, 9))))
    want = [oracle.spgemm(A, B or A, threads=4) for A, B in all_of]
    h = tsp.Handle()
    try:
        for key, value in options.items():
            h.set_option(getattr(tsp, key), value)
        dev = [(tsp.to_device(A), None if B is None else tsp.to_device(B)) for A, B in all_of]
        first = {}
        for i in list(range(count)) * 3 + [int(x) for x in rng.integers(0, count, 12)]:
            print(f"product {i} of {count}", flush=True)
            _, got = _bits(h, tsp, *dev[i])
            assert np.array_equal(got[0], want[i].row_ptr) and np.array_equal(got[1], want[i].col)
            assert np.all(np.abs(got[2].view(np.float32).astype(np.float64) - want[i].val) <= 1e-5 * want[i].mag + 1e-7)
            for x, y in zip(got, first.setdefault(i, got)):
                assert np.array_equal(x, y)
    finally:
        h.close()


_VALUES = {
    "ones": lambda rng, m: rng.choice([-1.0, 1.0], m),                                # 32-bit sums
    "below one": lambda rng, m: rng.uniform(-1, 1, m),                                # 64-bit sums
    "normal": lambda rng, m: rng.normal(size=m),                                      # beyond them: fp64
    "up to 100": lambda rng, m: rng.uniform(-100, 100, m),
    "largest and smallest": lambda rng, m: rng.choice([65504.0, -65504.0, 2.0 ** -24, -2.0 ** -24, 1.0], m),
    "zeros": lambda rng, m: np.where(rng.random(m) < 0.5, 0.0, -0.0),
    "some zeros": lambda rng, m: np.where(rng.random(m) < 0.5, 0.0, rng.normal(size=m)),
    "infinities": lambda rng, m: np.where(rng.random(m) < 0.01, np.inf, rng.normal(size=m)),
    "both infinities": lambda rng, m: np.where(rng.random(m) < 0.02, rng.choice([-np.inf, np.inf], m), rng.normal(size=m)),
    "NaN": lambda rng, m: np.where(rng.random(m) < 0.01, np.nan, rng.uniform(-1, 1, m)),
}


@pytest.mark.parametrize("values", sorted(_VALUES))
@pytest.mark.parametrize("left,right,cols", [(60, 40, 900), (300, 25, 20001)])
def test_values_of_heavy_rows(tsp, oracle, values, left, right, cols):
    """Every accumulator of the heavy rows, in a first call and launched ahead: sums against the oracle's within 1e-5 of the
    sum of the products' magnitudes, infinities and NaN where the oracle has them."""
    rng = np.random.default_rng(17)
    make = lambda m: _VALUES[values](rng, m)
    A = _exact_lengths(rng, 700, np.full(400, left), make)
    B = _exact_lengths(rng, cols, np.full(700, right), make)
    want = oracle.spgemm(A, B, threads=4)
    h = tsp.Handle()
    try:
        dA, dB = tsp.to_device(A), tsp.to_device(B)
        print(f"heavy rows: {values}, {left} x {right}", flush=True)
        first = None
        for _ in range(3):
            by_rows, got = _bits(h, tsp, dA, dB)
            assert by_rows
            assert np.array_equal(got[0], want.row_ptr) and np.array_equal(got[1], want.col)
            val, finite = got[2].view(np.float32).astype(np.float64), np.isfinite(want.val)
            assert np.array_equal(val[~finite], want.val[~finite], equal_nan=True)
            assert np.all(np.abs(val[finite] - want.val[finite]) <= 1e-5 * want.mag[finite] + 1e-7)
            for x, y in zip(got, first or got):
                assert np.array_equal(x, y)
            first = got
    finally:
        h.close()


@pytest.mark.parametrize("values", ["below one", "normal"])
@pytest.mark.parametrize("per_row", [2, 17])
@pytest.mark.parametrize("entries", [1820, 1821, 3641, 9000, 21000])
def test_tasks_of_very_long_rows(tsp, oracle, values, per_row, entries):
    """Rows of A so long that their windows of columns (18) are dealt to one task, to two, to groups and one by one, among
    rows of three entries; short and longer rows of B, which the fp64 sums take four at a time and one at a time."""
    rng = np.random.default_rng(entries + per_row)
    make = lambda m: _VALUES[values](rng, m)
    lengths = np.full(300, 3)
    lengths[[0, 131, 299]] = entries
    A = _exact_lengths(rng, 25000, lengths, make)
    B = _exact_lengths(rng, 70001, np.full(25000, per_row), make)
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B)
    finally:
        h.close()


@pytest.mark.parametrize("values", ["ones", "below one"])
@pytest.mark.parametrize("cols", [6000, 70001])
@pytest.mark.parametrize("entries", [17, 33, 511, 512, 513, 1025])
def test_pieces_of_heavy_rows_dealt_to_waves(tsp, oracle, values, cols, entries):
    """Rows of A of as many entries as a block has threads and either side, whose segments of B are cut into pieces of 16
    elements: rows of B of no, one, 15 to 17, 33 and very many elements; tables of few and of many columns, several steps."""
    rng = np.random.default_rng(entries + cols)
    make = lambda m: _VALUES[values](rng, m)
    lengths = np.full(300, 20)
    lengths[::37] = entries
    A = _exact_lengths(rng, 1100, lengths, make)
    B = _exact_lengths(rng, cols, rng.choice([0, 1, 15, 16, 17, 33, 5000], 1100, p=[0.2, 0.2, 0.15, 0.15, 0.1, 0.18, 0.02]), make)
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B)
    finally:
        h.close()


@pytest.mark.parametrize("left,lengths", [(8, (1, 9)), (8, (0, 17, 5)), (16, (1, 100)), (16, (17, 0, 33, 2)), (12, (6, 6, 40)), (9, (1, 1, 1, 150))])
def test_lists_longer_than_their_lanes(tsp, oracle, left, lengths):
    """Small rows some of whose lists go on beyond the lanes of a group, none, one and several times, others empty, in every place."""
    rng = np.random.default_rng(left + sum(lengths))
    B = _exact_lengths(rng, 3000, rng.choice(lengths, 1500), lambda m: rng.uniform(-1, 1, m))
    A = _exact_lengths(rng, 1500, rng.integers(0, left + 1, 1000), lambda m: rng.uniform(-1, 1, m))
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B, calls=3)
    finally:
        h.close()


@pytest.mark.parametrize("rows", [2049, 4096, 4097, 6200])
@pytest.mark.parametrize("left,right", [(2, 3), (5, 3), (8, 4), (5, 12), (16, 9)])
def test_small_rows_finished_and_moved_together(tsp, oracle, rows, left, right):
    """Products of small rows only, launched ahead (k_small_finish), of so few to so many entries per row that a block has 256, 128,
    64 and 32 rows; then, of the same sizes, one with more entries than there is room for, one with heavy rows, one with an
    empty end, and the first one again."""
    rng = np.random.default_rng(rows + left)
    ones = lambda m: rng.choice([-1.0, 1.0], m)
    B = _exact_lengths(rng, 3000, np.full(2000, right), ones)
    near = np.minimum(np.arange(rows)[:, None] % 7 + np.arange(left), 1999)
    first = inputs.from_coo(rows, 2000, np.repeat(np.arange(rows), left), near.reshape(-1), ones(rows * left), "few rows of B")
    spread = _exact_lengths(rng, 2000, np.full(rows, left), ones)
    lengths = np.full(rows, left)
    lengths[5], lengths[9:9 + 400 // left + 1] = left + 400, 0
    lengths[9] = lengths.sum() * 0 + rows * left - (lengths.sum() - lengths[9])
    heavy = _exact_lengths(rng, 2000, lengths, ones)
    ends = np.full(rows, left)
    ends[-64:] = 0
    ends[:64] = 2 * left
    h = tsp.Handle()
    try:
        for A in (first, spread, heavy, first, _exact_lengths(rng, 2000, ends, ones), first):
            _check(h, tsp, oracle, A, B, calls=2)
    finally:
        h.close()


@pytest.mark.parametrize("rows,left", [(300, 20), (65600, 9)])
def test_long_tile_rows_by_more_threads(tsp, oracle, rows, left):
    """Rows of 512 entries and more among short ones, in few tile-rows and in many: from the second call on k_row_prepare has more
    threads to a tile-row, whatever the operand at hand holds."""
    rng = np.random.default_rng(rows)
    ones = lambda m: rng.choice([-1.0, 1.0], m)
    B = _exact_lengths(rng, 900, np.full(800, 3), ones)
    lengths = np.full(rows, left)
    lengths[[0, 33, 34, rows - 1]] = [512, 799, 800, 513]
    even = np.full(rows, left)
    even[: lengths.sum() - even.sum()] += 1                 # the same number of entries, no long row
    h = tsp.Handle()
    try:
        for l in (lengths, even, lengths):
            _check(h, tsp, oracle, _exact_lengths(rng, 800, l, ones), B, calls=3 if l is lengths else 1)
    finally:
        h.close()


@pytest.mark.parametrize("a_row,b_row", [(1, 1), (2, 9), (6, 6), (7, 7), (8, 2), (8, 12), (3, 17)])
@pytest.mark.parametrize("rows", [12288, 12289])
def test_lanes_of_few_rows(tsp, oracle, rows, a_row, b_row):
    """Either side of the number of rows, and of the products per row (38), from which small rows have 16 lanes, lists of B
    narrower than 8 lanes, than 16 and not; then an operand of the same sizes with many rows of 9 to 16 entries, and back."""
    rng = np.random.default_rng(rows + 10 * a_row + b_row)
    values = lambda m: rng.normal(size=m)
    B = _exact_lengths(rng, 5003, np.full(2000, b_row), values)
    even = np.full(rows, a_row)
    # every 15th or 5th row of 10 to 16 entries, the others as even as what is left for them goes
    every, entries = (15, 15) if a_row == 1 else (5, min(5 * a_row, 16))
    longer = np.arange(rows) % every == 3
    longer[rows // every * every:] = False
    left, others = rows * a_row - entries * longer.sum(), rows - longer.sum()
    wide = np.where(longer, entries, left // others + (np.cumsum(~longer) <= left % others))
    assert wide.sum() == even.sum() and wide.min() >= 0 and 9 <= wide.max() <= 16
    h = tsp.Handle()
    try:
        for l in (even, wide, even):
            _check(h, tsp, oracle, _exact_lengths(rng, 2000, l, values), B, by_rows=None)
    finally:
        h.close()


@pytest.mark.parametrize("rows,a_row,b_row", [(2000, 3, 12), (12288, 2, 9), (12288, 8, 9), (12289, 5, 9), (12289, 3, 13), (20000, 5, 12), (12289, 2, 9), (3000, 7, 3), (3000, 9, 12)])
def test_sums_of_9_to_16_entries_round_once(tsp, oracle, rows, a_row, b_row):
    """Rows of 9 to 16 entries with short rows of B behind them, too few of them to be what the lanes are chosen for: where the
    mean row of A has at most 8 entries they are heavy with 8 lanes to a row (exact sums), and with 16 they are small and have to
    be summed as well, by narrow lists of B and by wide ones, either side of 12,288 rows and of 48 products.  All products are
    multiples of 2^-30 below 1: 16 of them add up exactly in fp64 and in integers, and fp32 does not hold them."""
    rng = np.random.default_rng(rows + 10 * a_row + b_row)
    values = lambda m: (rng.uniform(2.0 ** -4, 1, m).astype(np.float16) * rng.choice([-1, 1], m)).astype(np.float64)
    lengths = np.full(rows, a_row)
    some = np.sort(rng.choice(rows, rows // 70, replace=False))
    if a_row <= 8:
        lengths[some] = rng.integers(9, 17, some.size)
        lengths[np.setdiff1d(np.arange(rows), some)[: int(lengths.sum()) - a_row * rows]] -= 1
    first = np.where(np.isin(np.arange(rows), some), 0, 100)                    # of 100 rows of B of one entry, or of 400 others
    col = np.concatenate([np.sort(rng.choice(100 if f == 0 else 400, k, replace=False)) + f for f, k in zip(first, lengths)])
    A = inputs.from_coo(rows, 500, np.repeat(np.arange(rows), lengths), col, values(col.size), "some of 9 to 16")
    b_col = np.concatenate([rng.integers(0, 3, 100)] + [np.sort(rng.choice(150, b_row * 5 // 4, replace=False)) for _ in range(400)])
    B = inputs.from_coo(500, 150, np.repeat(np.arange(500), [1] * 100 + [b_row * 5 // 4] * 400), b_col, values(b_col.size), "short and longer")
    ref = oracle.spgemm(A, B, threads=4)
    rounded = np.repeat((lengths > 8) & (a_row <= 8), np.diff(ref.row_ptr))
    dA, dB = tsp.to_device(A), tsp.to_device(B)
    h = tsp.Handle()
    try:
        for _ in range(3):
            C = h.spgemm(dA, dB)
            assert h.stats()["pairs"] == 0
            row_ptr, col, val = C.to_host()
            C.free()
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val - ref.val) <= 16 * 2.0 ** -24 * ref.mag)
            assert np.array_equal(val[rounded], ref.val[rounded].astype(np.float32))
    finally:
        h.close()


# rows of A of `a_row` entries, all but one with b_row entries of B behind them and one with `other`: products either side of what
# fills one, two, four, ... registers of 8 lanes (more than 12,288 rows) and of 16, single rounds and several, longer lists than lanes
@pytest.mark.parametrize("rows,a_row,b_row,other", [
    (12291, 1, 1, 1), (12291, 7, 1, 2), (12291, 8, 1, 2), (12291, 3, 5, 6), (12291, 3, 5, 7), (12291, 8, 4, 4), (12291, 8, 4, 5), (12291, 5, 9, 2), (12291, 2, 30, 2),
    (12291, 6, 7, 13), (259, 1, 1, 1), (259, 16, 1, 1), (259, 16, 1, 2), (259, 4, 8, 8), (259, 4, 8, 9), (259, 8, 8, 8), (259, 8, 8, 9), (259, 11, 12, 8),
    (259, 11, 12, 9), (259, 16, 12, 12), (259, 6, 30, 42), (259, 3, 16, 17), (259, 2, 33, 90), (259, 13, 2, 40)])
@pytest.mark.parametrize("columns", ["the same", "others", "some of both"])
def test_products_of_small_rows_sorted(tsp, oracle, rows, a_row, b_row, other, columns):
    """Sums over one lane and over many, with all products of a row in one column of C each and with each in its own.  Products are
    multiples of 2^-30 below 1, so that fp64 sums are exact and an entry is the exact sum, rounded once."""
    rng = np.random.default_rng(rows + 1000 * a_row + 100 * b_row + other)
    values = lambda m: (rng.uniform(2.0 ** -4, 1, m).astype(np.float16) * rng.choice([-1, 1], m)).astype(np.float64)
    many, width = 60, {"the same": max(b_row, other), "others": 7001, "some of both": 2 * max(b_row, other)}[columns]
    lengths = np.r_[np.full(many, b_row), np.full(many, other)]
    B = inputs.from_coo(2 * many, 7001, np.repeat(np.arange(2 * many), lengths),
                        np.concatenate([np.sort(rng.choice(width, k, replace=False)) for k in lengths]), values(lengths.sum()), "lists")
    a_col = np.sort(np.concatenate([np.argsort(rng.random((rows, many)), axis=1)[:, : a_row - 1], many + rng.integers(0, many, (rows, 1))], axis=1), axis=1)
    A = inputs.from_coo(rows, 2 * many, np.repeat(np.arange(rows), a_row), a_col.ravel(), values(rows * a_row), "rows")
    ref = oracle.spgemm(A, B, threads=4)
    dA, dB = tsp.to_device(A), tsp.to_device(B)
    h = tsp.Handle()
    try:
        for _ in range(2):
            C = h.spgemm(dA, dB)
            row_ptr, col, val = C.to_host()
            C.free()
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            if h.stats()["pairs"] == 0:                         # (tiles where they are preferred)
                assert np.array_equal(val, ref.val.astype(np.float32))
    finally:
        h.close()


def _short(rng, rows, cols, most, dense=0):
    """Rows of 0 to `most` entries; with `dense`, a few rows of so many that no entry of the left operand meets (columns from 64 on)."""
    lengths = rng.integers(0, most + 1, rows)
    if dense:
        lengths[:3] = dense
    col = np.concatenate([np.sort(rng.choice(cols - 64, k, replace=False)) + 64 if k < 64 else np.sort(rng.choice(cols, k, replace=False)) for k in lengths])
    return inputs.from_coo(rows, cols, np.repeat(np.arange(rows), lengths), col, rng.uniform(-1, 1, col.size), "short rows")


# one chunk of rows (2048) and more, ends of tile-rows, of a wave's four, of a block's, of a group of 64 blocks (2048 rows of 8 lanes, 1024
# of 16), as many blocks of rows as it takes (262,144 rows by 16 lanes) and more, bitmaps of 16 KB (524,288 columns) and beyond, 128 entries
# per tile-row and more, rows of up to 9 entries that 8 lanes are not for, and rows of more products than its LDS has room for
@pytest.mark.parametrize("rows,inner,cols,a_row,b_row,dense,straight", [
    (257, 300, 200, 4, 4, 0, True), (2047, 1999, 3001, 3, 5, 0, True), (2048, 2048, 2048, 6, 4, 0, True), (2048, 2048, 2048, 6, 9, 0, False),
    (2049, 70, 5000, 3, 3, 0, True), (2065, 5000, 70, 5, 2, 0, True), (4099, 4099, 4099, 8, 3, 0, True), (4099, 4099, 4099, 8, 12, 0, False),
    (16384, 700, 900, 2, 2, 600, True), (20001, 20001, 20001, 5, 4, 0, True), (20001, 20001, 20001, 5, 7, 0, False), (65537, 3000, 4000, 3, 3, 2000, True),
    (3000, 90001, 90001, 3, 4, 0, True), (30000, 524288, 2000, 2, 3, 0, True), (30000, 524289, 2000, 2, 3, 0, False), (2100, 1500, 524288, 4, 3, 0, True),
    (2100, 1500, 524289, 4, 3, 0, False), (262200, 400, 500, 1, 2, 0, True), (262200, 400, 500, 9, 9, 0, False), (262144, 400, 500, "7", "5", 0, True),
    (262145, 400, 500, "7", "5", 0, False), (3008, 900, 800, "8", "3", 0, True), (3008, 900, 800, "9", "3", 0, False)])
@pytest.mark.parametrize("types", [{}, {"value_dtype": "f32", "row_ptr_dtype": "i64"}])
def test_small_rows_straight_from_the_operands(tsp, oracle, rows, inner, cols, a_row, b_row, dense, straight, types):
    """The second and later products of sizes whose first one had small rows only: the same bits as the first and the same numbers of
    tiles and of their pairs, without the pass over the operands (the convert kernel) inside the limits and with it beyond them.  Rows of
    up to so many entries, or of exactly so many where the number is a text."""
    rng = np.random.default_rng(rows + cols)
    exactly = lambda n, m, k: _exact_lengths(rng, m, np.full(n, int(k)), lambda size: rng.uniform(-1, 1, size))
    A = exactly(rows, inner, a_row) if isinstance(a_row, str) else _short(rng, rows, inner, a_row)
    B = exactly(inner, cols, b_row) if isinstance(b_row, str) else _short(rng, inner, cols, b_row, dense)
    if dense:                                                  # (the dense rows of B are met by nobody)
        assert A.col_idx.min() >= 64
    dA, dB = tsp.to_device(A, **types), tsp.to_device(B, **types)
    ref = oracle.spgemm(A, B, threads=4)
    h = tsp.Handle(phase_timers=True)
    try:
        first = None
        for call in range(3):
            C = h.spgemm(dA, dB)
            row_ptr, col, val = C.to_host()
            C.free()
            stats = h.stats()
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
            assert stats["pairs"] == 0 and (stats["kernel_us"]["convert"] == 0) == (straight and call > 0)
            now = [val.view(np.uint32), [stats[k] for k in ("a_tiles", "b_tiles", "candidate_pairs", "c_nnz")]]
            first = first or now
            assert np.array_equal(now[0], first[0]) and now[1] == first[1]
    finally:
        h.close()


@pytest.mark.parametrize("rows", [700, 2049, 12288, 12289])
def test_rows_of_nine_entries_where_there_were_none(tsp, oracle, rows):
    """Products of the same sizes without rows of more than 8 entries, with one, with many and with one that no lanes are enough for: the
    same bits as on a handle of their own."""
    rng = np.random.default_rng(rows)
    inner, total = 900, 3 * rows

    def left(longest, many=1):
        lengths = np.full(rows, 3)
        lengths[np.arange(many) * 7 % rows] = longest
        spare = lengths.sum() - total
        give = np.flatnonzero(lengths == 3)[:spare // 2 + 1]
        lengths[give[:spare // 2]] -= 2
        lengths[give[spare // 2]] -= spare % 2
        assert lengths.sum() == total
        col = np.concatenate([np.sort(rng.choice(inner, k, replace=False)) for k in lengths])
        return inputs.from_coo(rows, inner, np.repeat(np.arange(rows), lengths), col, rng.uniform(-1, 1, total), "left")

    B = _short(rng, inner, 800, 6)
    As = [left(8), left(9), left(16, rows // 20), left(17), left(3)]
    dB, dev = tsp.to_device(B), [tsp.to_device(A) for A in As]

    def product(h, k):
        C = h.spgemm(dev[k], dB)
        out = C.to_host()
        C.free()
        return out

    alone = []
    for k in range(len(As)):
        h = tsp.Handle()
        try:
            alone.append(product(h, k))
        finally:
            h.close()
        ref = oracle.spgemm(As[k], B, threads=4)
        assert np.array_equal(alone[k][0], ref.row_ptr) and np.array_equal(alone[k][1], ref.col)
        assert np.all(np.abs(alone[k][2].astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
    h = tsp.Handle()
    try:
        for k in (0, 4, 0, 1, 1, 0, 2, 2, 0, 0, 3, 0, 0, 1):
            for x, y in zip(product(h, k), alone[k]):
                assert np.array_equal(x, y), k
    finally:
        h.close()


# one chunk of rows, with the pairs of tiles by the last block and by others; more rows, from counts and from lists
@pytest.mark.parametrize("rows,inner,a_most,b_most", [(700, 900, 3, 6), (2048, 70000, 13, 1), (2500, 2500, 2, 3), (9000, 9001, 9, 3)])
def test_blocks_that_wait_give_up(tsp, oracle, rows, inner, a_most, b_most):
    """Blocks that do not wait for what the others of the launch count, on canonical operands and on others: the product is made the
    other way, or refused, and the next one that waits has nothing of it in its numbers."""
    rng = np.random.default_rng(rows)
    A, B = _short(rng, rows, inner, a_most), _short(rng, inner, 700, b_most)
    broken = inputs.from_coo(A.rows, A.cols, np.repeat(np.arange(A.rows), np.diff(A.row_ptr)), A.col_idx, A.val, "broken")
    broken.col_idx[-1] = inner
    dA, dB, bad = tsp.to_device(A), tsp.to_device(B), tsp.to_device(broken)
    ref = oracle.spgemm(A, B, threads=4)
    h = tsp.Handle(phase_timers=True)
    try:
        first = None
        def product(straight):
            nonlocal first
            C = h.spgemm(dA, dB)
            row_ptr, col, val = C.to_host()
            C.free()
            stats = h.stats()
            assert straight is None or (stats["kernel_us"]["convert"] == 0) == straight
            now = [row_ptr, col, val, [stats[k] for k in ("a_tiles", "b_tiles", "candidate_pairs", "c_nnz", "pairs")]]
            first = first or now
            assert all(np.array_equal(x, y) for x, y in zip(now, first))
        product(False)
        product(True)
        assert np.array_equal(first[0], ref.row_ptr) and np.array_equal(first[1], ref.col)
        h.set_option(tsp.OPT_GIVE_UP_WAITS, 1)
        product(False)
        h.set_option(tsp.OPT_GIVE_UP_WAITS, 0)
        for straight in (False, False, False, True, True, True):       # (three more before the next try)
            product(straight)
        h.set_option(tsp.OPT_GIVE_UP_WAITS, 1)
        with pytest.raises(tsp.TspError):                      # (by whichever kernels have seen it first)
            h.spgemm(bad, dB)
        h.set_option(tsp.OPT_GIVE_UP_WAITS, 0)
        for straight in [None] * 8 + [True, True]:
            product(straight)
    finally:
        h.close()


@pytest.mark.parametrize("rows", [700, 2500])
def test_straight_from_the_operands_again(tsp, rows):
    """After a product with a row that is not small, products of the same sizes without any go straight from the operands again, and
    not at once; with such products in turn they no longer try.  (The pass over the operands is the convert kernel.)"""
    rng = np.random.default_rng(rows)
    B = _short(rng, 900, 800, 6)
    lengths = np.full(rows, 3)
    lengths[5], lengths[20:34] = 31, 1
    As = [inputs.from_coo(rows, 900, np.repeat(np.arange(rows), l), np.concatenate([np.sort(rng.choice(900, k, replace=False)) for k in l]),
                          rng.uniform(-1, 1, 3 * rows), "left") for l in (np.full(rows, 3), lengths)]
    dB, dev = tsp.to_device(B), [tsp.to_device(A) for A in As]
    h = tsp.Handle(phase_timers=True)

    def straight(k):
        h.spgemm(dev[k], dB).free()
        return h.stats()["kernel_us"]["convert"] == 0

    try:
        straight(0)
        assert [straight(0) for _ in range(3)] == [True] * 3
        assert not straight(1)
        assert [straight(0) for _ in range(6)] == [False] * 4 + [True] * 2
        assert not straight(1)
        assert [straight(0) for _ in range(9)] == [False] * 8 + [True]
        for _ in range(4):
            assert not straight(1)
            assert not any(straight(0) for _ in range(8))
        assert any(straight(0) for _ in range(16))
    finally:
        h.close()


@pytest.mark.parametrize("rows", [9000, 40000])
def test_rows_or_tiles_whatever_came_before(tsp, oracle, rows):
    """Products of the same sizes with more than 32 products per row, one with many rows of 9 to 16 entries and one without any: the same
    way, by rows or by tiles, and the same bits as on a handle of their own.  (16 lanes to a row whichever it is, but what the rows cost
    is reckoned by their number, and with entries near the diagonal that decides.)"""
    rng = np.random.default_rng(rows)
    lengths = np.full(rows, 7)
    lengths[::20], lengths[5::20] = 13, 1

    def left(lengths, spread):
        first = np.minimum(np.arange(rows) // 4 * 4, rows - spread)
        col = np.concatenate([np.sort(rng.choice(spread, k, replace=False)) + f for f, k in zip(first, lengths)])
        return inputs.from_coo(rows, rows, np.repeat(np.arange(rows), lengths), col, rng.uniform(-1, 1, col.size), "left")

    near = np.minimum(np.arange(rows) // 16 * 16, rows - 16)
    B = inputs.from_coo(rows, rows, np.repeat(np.arange(rows), 6), np.concatenate([np.sort(rng.choice(16, 6, replace=False)) + f for f in near]),
                        rng.uniform(-1, 1, 6 * rows), "right")
    As = [left(lengths, rows // 2), left(np.full(rows, 7), 20), left(lengths, 20)]
    dB, dev = tsp.to_device(B), [tsp.to_device(A) for A in As]

    def product(h, k):
        C = h.spgemm(dev[k], dB)
        out = C.to_host()
        C.free()
        return [h.stats()["pairs"] == 0] + list(out)

    alone = []
    for k, A in enumerate(As):
        h = tsp.Handle()
        try:
            alone.append(product(h, k))
        finally:
            h.close()
        ref = oracle.spgemm(A, B, threads=4)
        assert np.array_equal(alone[k][1], ref.row_ptr) and np.array_equal(alone[k][2], ref.col)
        assert np.all(np.abs(alone[k][3].astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
    if rows == 40000:
        assert [x[0] for x in alone] == [True, True, False]
    # (the last one's tiles stay for products with about as many pairs of them, so it comes last)
    h = tsp.Handle()
    try:
        for k in (0, 0, 1, 1, 0, 1, 2):
            for x, y in zip(product(h, k), alone[k]):
                assert np.array_equal(x, y), k
    finally:
        h.close()


# pairs of tiles by the last block (one chunk of rows, B of up to 4096 tile-rows), by others from counts, and from lists (more tiles in A
# than rows and than 24,576)
@pytest.mark.parametrize("shapes", [
    ((300, 65536, 140, 2, 2), (300, 65537, 140, 2, 2)), ((2048, 65535, 300, 12, 1), (2048, 70000, 300, 13, 1)), ((2049, 2049, 2049, 3, 3), (2049, 300, 500, 9, 6)),
    ((2000, 524288, 100, 3, 1), (700, 524288, 100, 2, 1)), ((9000, 9000, 700, 2, 3), (9000, 9001, 700, 9, 3))])
def test_pairs_of_tiles_straight_from_the_operands(tsp, shapes):
    """Two products in turn on one handle: the numbers of tiles and of their pairs as counted here, every time, and from the second on
    without the pass over the operands (the convert kernel), unless rows of up to 9 entries have too many products."""
    def tiles(M):
        row = np.repeat(np.arange(M.rows), np.diff(M.row_ptr)) // 16
        return np.unique(row * ((M.cols + 15) // 16) + M.col_idx // 16)

    cases = []
    for rows, inner, cols, a_most, b_most in shapes:
        rng = np.random.default_rng(inner)
        A, B = _short(rng, rows, inner, a_most), _short(rng, inner, cols, b_most)
        of_a, of_b = tiles(A), tiles(B)
        per_row = np.bincount(of_b // ((cols + 15) // 16), minlength=(inner + 15) // 16)
        cases.append((tsp.to_device(A), tsp.to_device(B), [of_a.size, of_b.size, int(per_row[of_a % ((inner + 15) // 16)].sum())]))
    h = tsp.Handle(phase_timers=True)
    try:
        for call in range(4):
            for (*_, a_most, b_most), (dA, dB, want) in zip(shapes, cases):
                h.spgemm(dA, dB).free()
                stats = h.stats()
                assert [stats[k] for k in ("a_tiles", "b_tiles", "candidate_pairs")] == want
                assert (stats["kernel_us"]["convert"] == 0) == (call > 0 and (a_most, b_most) != (9, 6))
    finally:
        h.close()


@pytest.mark.parametrize("rows", [1800, 30000])
def test_what_is_not_for_it_straight_from_the_operands(tsp, oracle, rows):
    """Operands of the sizes of a product of small rows that are not canonical, that have more entries in C than the last one and some,
    or rows that are not small: refused, or multiplied all the same; then one of small rows again.  `straight`: without the pass over the
    operands (the convert kernel)."""
    rng = np.random.default_rng(rows)
    lengths, cols = np.full(rows, 3), 5003
    def make(lengths, width=cols):
        col = np.concatenate([np.sort(rng.choice(width, k, replace=False)) for k in lengths])
        return inputs.from_coo(rows, cols, np.repeat(np.arange(rows), lengths), col, rng.uniform(-1, 1, col.size), "left")
    B = inputs.from_coo(cols, 4001, np.repeat(np.arange(cols), 4), np.sort(rng.integers(0, 1000, (cols, 4)) * 4 + np.arange(4), axis=1).ravel(),
                        rng.uniform(-1, 1, 4 * cols), "right")
    ordinary, narrow = make(lengths), make(lengths, 5)
    long_row = lengths.copy()
    long_row[7], long_row[20:40] = 23, 2
    many_products = lengths.copy()
    many_products[100], many_products[200:205] = 8, 2
    dB = tsp.to_device(B)
    h = tsp.Handle(validate=True, phase_timers=True)
    try:
        def good(A, straight):
            ref = oracle.spgemm(A, B, threads=4)
            C = h.spgemm(tsp.to_device(A), dB)
            row_ptr, col, val = C.to_host()
            C.free()
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
            assert (h.stats()["kernel_us"]["convert"] == 0) == straight
        for straight in (False, True):
            good(narrow, straight)
        good(ordinary, True)                                   # (more entries in C than there is room for)
        for where, broken_col in ((0, -1), (500, cols), (3 * rows - 1, 1 << 30), (301, None), (302, "same")):
            broken = make(lengths)
            broken.col_idx[where] = broken.col_idx[where - 1] if broken_col == "same" else broken.col_idx[where + 1] if broken_col is None else broken_col
            with pytest.raises(tsp.TspError):
                h.spgemm(tsp.to_device(broken), dB)
        for at, value in ((0, 1), (5, 1 << 30), (6, -3), (rows, 3 * rows - 1), (16, 0), (64, 190), (rows - 1, 0)):
            broken = make(lengths)
            broken.row_ptr[at] = value
            with pytest.raises(tsp.TspError):
                h.spgemm(tsp.to_device(broken), dB)
        good(ordinary, True)
        assert make(long_row).nnz == make(many_products).nnz == ordinary.nnz
        good(make(many_products), False)
        good(ordinary, False)
        good(make(long_row), False)
        for straight in [False] * 4 + [True]:                  # (four products without such rows before the next try)
            good(ordinary, straight)
    finally:
        h.close()


@pytest.mark.parametrize("a_row,b_row", [(4, 3), (40, 30), (4, 30), (40, 3)])
@pytest.mark.parametrize("b_types", [{}, {"value_dtype": "f32"}, {"row_ptr_dtype": "i64"}])
def test_both_operands_prepared_at_once(tsp, oracle, a_row, b_row, b_types):
    """Operands of the same and of other types, by a wave per tile-row, by a block, and one by each, with numbers of tile-rows
    that are no multiple of a block's; repeated, and B not canonical in its last row."""
    rng = np.random.default_rng(a_row + 10 * b_row)
    values = lambda m: rng.choice([-1.0, 0.5, 2.0], m)
    A, B = _exact_lengths(rng, 3005, np.full(333, a_row), values), _exact_lengths(rng, 1777, np.full(3005, b_row), values)
    dA, dB = tsp.to_device(A), tsp.to_device(B, **b_types)
    ref = oracle.spgemm(A, B, threads=4)
    broken = inputs.from_coo(B.rows, B.cols, np.repeat(np.arange(B.rows), b_row), B.col_idx, B.val, "broken")
    broken.col_idx[-2:] = broken.col_idx[-2:][::-1]
    h = tsp.Handle(validate=True)
    try:
        for _ in range(3):
            C = h.spgemm(dA, dB)
            row_ptr, col, val = C.to_host()
            C.free()
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
        with pytest.raises(tsp.TspError):
            h.spgemm(dA, tsp.to_device(broken, **b_types))
    finally:
        h.close()


@pytest.mark.parametrize("inner,cols", [(3005, 839680), (3005, 839681), (3005, 1966080), (3005, 1966081), (839680, 500), (839681, 500), (1900000, 500), (700000, 839681)])
@pytest.mark.parametrize("a_row,b_row", [(4, 3), (40, 30)])
def test_operands_of_unequal_widths(tsp, oracle, inner, cols, a_row, b_row):
    """One operand of few columns and one of many, either side of the widths up to which both go in one launch of k_row_prepare and
    up to which a wave takes a tile-row; columns at both ends of the width."""
    rng = np.random.default_rng(inner + cols + a_row)
    def even(rows, width, k, of_row):
        x = np.sort(rng.integers(0, width - k + 1, (rows, k)), axis=1) + np.arange(k)
        x[::7] += width - 1 - x[::7, -1:]                      # (the last column)
        return inputs.from_coo(of_row[-1] + 1, width, np.repeat(of_row, k), x.ravel(), rng.choice([-1.0, 0.5, 2.0], rows * k), "even")
    A = even(333, inner, a_row, np.arange(333))
    used = np.unique(A.col_idx)
    B = even(used.size + (used[-1] != inner - 1), cols, b_row, used if used[-1] == inner - 1 else np.append(used, inner - 1))
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B, calls=3)
    finally:
        h.close()


@pytest.mark.parametrize("rows,left", [(3000, 9), (3000, 70), (255, 3), (32768, 1), (32769, 2)])      # (either side of a launch for B alone)
def test_long_rows_of_b_packed_by_blocks(tsp, oracle, rows, left):
    """Rows of B around the lengths from which a wave, or all waves of a block, take them (128, 1024), at the ends of a block's
    rounds (2048 entries), next to each other and 256 rows apart, among short ones (left: 16 lanes to a row, or 64)."""
    rng = np.random.default_rng(rows + left)
    ones = lambda m: rng.choice([-1.0, 1.0], m)
    lengths = np.full(rows, left)
    edges = [128, 129, 255, 257, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 9000, 0, 130, 1030]
    lengths[: len(edges)] = edges
    if rows > 600:
        lengths[256 : 256 + len(edges)] = edges[::-1]
        lengths[512 : 512 + len(edges)] = edges
    lengths[-1] = 1025
    B = _exact_lengths(rng, 140000, lengths, ones)
    A = _exact_lengths(rng, rows, rng.choice([1, 17, 40, 250], 300), ones)
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B, calls=2)
    finally:
        h.close()


@pytest.mark.parametrize("cols", [70016, 262144, 262145, 600000])
def test_words_of_16_columns(tsp, oracle, cols):
    """Rows of B of runs of columns that begin and end at the edges of words (16 columns), of places (32), of trips of the lanes
    that make the words (64 and 16 entries) and of spans (262,144 columns), and one of more words than a segment takes."""
    rng = np.random.default_rng(cols)
    edges = np.array([0, 15, 16, 31, 32, 4095, 4096, 65535, 65536, cols // 2, cols - 700, 262143 % cols, 262130 % cols])
    rows = []
    for i in range(600):
        start = edges[rng.integers(0, len(edges), 3)] - rng.integers(0, 3, 3)
        rows.append(np.unique(np.clip(np.concatenate([a + np.arange(n) for a, n in zip(start, rng.choice([1, 15, 16, 17, 33, 64, 65, 250], 3))]), 0, cols - 1)))
    rows[77] = np.arange(0, cols, 3)
    if cols < 100000:                            # (16 lanes per row where the mean row is short)
        rows = [r[:rng.integers(1, 24)] if i != 77 else r[:2000] for i, r in enumerate(rows)]
    r = np.repeat(np.arange(600), [len(x) for x in rows])
    B = inputs.from_coo(600, cols, r, np.concatenate(rows), rng.choice([-1.0, 1.0], len(r)), "runs of columns")
    A = _exact_lengths(rng, 600, rng.choice([1, 17, 40, 300], 300), lambda m: rng.choice([-1.0, 1.0], m))
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B)
    finally:
        h.close()


@pytest.mark.parametrize("cols", [131072, 131073])
def test_sizing_of_wide_and_narrow_rows(tsp, oracle, cols):
    """Either side of the number of columns from which k_heavy_count has 512 threads to a row."""
    test_words_of_16_columns(tsp, oracle, cols)


@pytest.mark.parametrize("values", ["ones", "below one"])
@pytest.mark.parametrize("cols,large", [(6000, 256), (70001, 512)])
def test_large_and_light_rows(tsp, oracle, values, cols, large):
    """Rows of A around the number of products from which a row is large; products in turn on one handle whose operands have
    equal sizes and more large rows, fewer and none, so that what the last one left does not fit."""
    rng = np.random.default_rng(cols)
    make = lambda m: _VALUES[values](rng, m)
    rows = (9 << 20) // (64 * large)                       # (8 million products from which the large rows are apart)
    B = _exact_lengths(rng, cols, np.full(1100, 64), make)
    total, all_of = rows * (large - 1), []
    for many in (0, 1, 40, 7, rows - 1):
        lengths = np.full(rows, large - 1)
        lengths[rng.choice(rows, many, replace=False)] = large
        lengths[np.argmin(lengths)] -= lengths.sum() - total
        all_of.append(_exact_lengths(rng, 1100, np.maximum(lengths, 0), make))
    h = tsp.Handle()
    try:
        for i in (0, 1, 2, 3, 0, 2, 4):
            _check(h, tsp, oracle, all_of[i], B)
    finally:
        h.close()


def test_values_that_integers_do_not_hold_by_tiles(tsp, oracle):
    """A product that is faster by rows while its sums are integers and by tiles otherwise."""
    rng = np.random.default_rng(4)
    n = 1000
    lengths = np.full(n, 200)
    h = tsp.Handle()
    try:
        for values, by_rows in (("below one", True), ("normal", False), ("normal", False)):
            A = _exact_lengths(rng, n, lengths, lambda m: _VALUES[values](rng, m))
            _check(h, tsp, oracle, A, by_rows=by_rows, calls=2)
    finally:
        h.close()


@pytest.mark.parametrize("what,by_rows", [("blocks", False), ("stencil", False), ("random", True), ("rectangles", True), ("rectangles of tiles", False),
                                          ("looks like tiles", True)])
@pytest.mark.parametrize("upload", [{}, {"value_dtype": "f32", "row_ptr_dtype": "i64"}])
def test_rows_or_tiles_at_first_sight(tsp, oracle, what, by_rows, upload):
    """Operands large enough for a look at some of their tile-rows before the look at all of them; in the last case every
    tile-row that is looked at (the odd ones of 256) holds four full tiles and the others are random."""
    rng = np.random.default_rng(6)
    n, B = 4096, None
    if what == "blocks":
        A = inputs.block_clustered(16384, seed=2)
    elif what == "stencil":
        A = inputs.stencil27_3d(13, dof=3)
    elif what == "random":
        A = _matrix(rng, n, n, 70)
    elif what == "rectangles":
        A, B = _matrix(rng, 5000, 3000, 60), _matrix(rng, 3000, 7001, 20)
    elif what == "rectangles of tiles":
        A = _full_tiles(rng, n)
        B = inputs.from_coo(n, 160, np.repeat(np.arange(n), 16), (np.arange(n)[:, None] // 16 % 10 * 16 + np.arange(16)).ravel(), rng.normal(size=16 * n))
    else:
        T, R = _full_tiles(rng, n), _exact_lengths(rng, n, np.full(n, 64), lambda m: rng.normal(size=m))
        odd = np.repeat(np.arange(n) // 16 % 2 == 1, 64)
        A = inputs.from_coo(n, n, np.repeat(np.arange(n), 64), np.where(odd, T.col_idx, R.col_idx), np.where(odd, T.val, R.val))
    assert A.nnz >= 1 << 18
    h = tsp.Handle()
    try:
        _check(h, tsp, oracle, A, B, by_rows=by_rows, calls=3, **upload)
    finally:
        h.close()


def test_rejects_what_is_not_canonical(tsp):
    import torch
    h = tsp.Handle()
    try:
        A = tsp.to_device(inputs.random_fixed_per_row(600, 5, seed=3))
        h.spgemm(A, A).free()
        good_col, good_ptr = A.col_idx, A.row_ptr
        for k, value in [(0, -1), (77, 600), (78, int(good_col[77])), (2999, 0)]:
            A.col_idx = good_col.clone()
            A.col_idx[k] = value
            with pytest.raises(tsp.TspError) as e:
                h.spgemm(A, A)
            assert e.value.status == -3
        A.col_idx = good_col
        for k, value in [(0, 1), (17, -5), (300, 5000), (600, 2999)]:
            A.row_ptr = good_ptr.clone()
            A.row_ptr[k] = value
            with pytest.raises(tsp.TspError) as e:
                h.spgemm(A, A)
            assert e.value.status == -3
        A.row_ptr = good_ptr
        C = h.spgemm(A, A)
        assert C.nnz > 0 and h.stats()["pairs"] == 0
        C.free()
    finally:
        h.close()


@pytest.mark.parametrize("row_ptr_dtype", ["i32", "i64"])
def test_rejects_row_pointers_that_go_up_and_down(tsp, row_ptr_dtype):
    """On sizes seen before, where the kernels run before the host knows that an operand is not canonical: rows that begin
    behind the next one, so that a row has entries that were counted for another, with long rows of B behind them; lengths
    of rows of B that do not fit their type.  tests/test_row_bounds.py models what the kernels rest on."""
    import torch
    n = 600
    rng = np.random.default_rng(2)
    b_len = np.ones(n, np.int64)
    b_len[::50] = 40
    B = inputs.from_coo(n, n, np.repeat(np.arange(n), b_len), np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in b_len]),
                        rng.uniform(-1, 1, b_len.sum()))
    A = inputs.from_coo(n, n, np.repeat(np.arange(n), 4), np.concatenate([np.sort(rng.choice(n, 4, replace=False)) for _ in range(n)]),
                        rng.uniform(-1, 1, 4 * n))
    far = 2 ** 31 - 1 if row_ptr_dtype == "i32" else 2 ** 62
    h = tsp.Handle()
    try:
        dA, dB = tsp.to_device(A, row_ptr_dtype=row_ptr_dtype), tsp.to_device(B, row_ptr_dtype=row_ptr_dtype)
        # rows 50 * i of B are long: the entries that change hands below meet three of them
        dA.col_idx[12:15] = torch.tensor([0, 50, 100], dtype=torch.int32)
        dA.col_idx[15] = 150
        good_a, good_b = dA.row_ptr, dB.row_ptr
        for _ in range(2):
            h.spgemm(dA, dB).free()
            assert h.stats()["pairs"] == 0
        bumps = [("A", {3: 15, 4: 12}), ("A", {3: 15}), ("A", {16: 80, 17: 70}), ("A", {15: 66, 16: 63}), ("A", {20: 2400, 21: 0}), ("A", {599: 2399, 598: 2400}),
                 ("B", {3: 40, 4: 2}), ("B", {16: 120, 17: 10}), ("B", {1: -far, 2: far}), ("B", {5: far, 6: -far}), ("A", {7: -far, 8: far}),
                 ("B", {i: (i * 977) % B.nnz for i in range(1, 500)})]
        for which, values in bumps:
            print("row pointers:", which, str(values)[:60], flush=True)
            M, good = (dA, good_a) if which == "A" else (dB, good_b)
            M.row_ptr = good.clone()
            for at, value in values.items():
                M.row_ptr[at] = value
            with pytest.raises(tsp.TspError) as e:
                h.spgemm(dA, dB)
            assert e.value.status == -3
            M.row_ptr = good
        C = h.spgemm(dA, dB)
        assert C.nnz > 0 and h.stats()["pairs"] == 0
        C.free()
    finally:
        h.close()
