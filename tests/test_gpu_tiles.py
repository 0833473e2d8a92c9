"""The tile kernels at the sizes where they can go wrong, against the CPU oracle: the conversion of tile-rows of hundreds to
thousands of entries (k_convert_block and k_convert_large of csrc/convert.hip), with entries either side of what the
registers of a block hold, tiles either side of a window, spans either side of the bitmap and empty tile-rows; and task
lists in arrays sized after another product.  Needs an MI355X."""
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


def _tile_rows(rng, cols, tiles, entries):
    """Tile-row i: entries[i] entries spread over tiles[i] tiles (every tile holds one at least)."""
    keys = []
    for i, (t, n) in enumerate(zip(tiles, entries)):
        if n == 0:
            continue
        col = np.sort(rng.choice(cols // 16, t, replace=False))
        slots = rng.permutation(t * 256)
        first = np.arange(t) * 256 + rng.integers(0, 256, t)
        pick = np.unique(np.concatenate([first, slots[:n]]))[:max(n, t)]
        tile, r, c = pick // 256, pick % 256 // 16, pick % 16
        keys.append((i * 16 + r) * cols + col[tile] * 16 + c)
    key = np.unique(np.concatenate(keys))
    return inputs.from_coo(16 * len(tiles), cols, key // cols, key % cols, rng.uniform(-1, 1, key.size), "tile-rows")


def _dense(view, form, t):
    mask = int(view[f"{form}_group_mask"][t]) & 0xFFFFFFFF
    off = int(view[f"{form}_group_off"][t]) & 0xFFFFFFFF
    groups = [g for g in range(32) if (mask >> g) & 1]
    rows = view[f"{form}_elements"][off * 8:(off + len(groups)) * 8].reshape(-1, 8)
    out = np.zeros((16, 16), dtype=np.float16)
    for g, x in zip(groups, rows):
        if form == "left":
            out[g % 16, 8 * (g // 16):8 * (g // 16) + 8] = x
        else:
            out[8 * (g // 16):8 * (g // 16) + 8, g % 16] = x
    return out


@pytest.mark.parametrize("cols,tiles,entries", [
    (4096, (4, 5, 4), (1023, 1024, 1025)),
    (4096, (31, 32, 33, 34), (1024, 1024, 1024, 1025)),
    (4096, (8, 0, 8, 7), (1536, 0, 1537, 1500)),
    (4096, (64, 65, 9), (2047, 2048, 2049)),
    (4096, (256, 1, 200), (9000, 256, 700)),
    (524288, (40, 40), (900, 1000)),
    (600000, (40, 2, 40), (900, 300, 1000)),
])
@pytest.mark.parametrize("upload", [{}, {"value_dtype": "f32", "row_ptr_dtype": "i64"}])
def test_tile_rows_of_many_entries(tsp, oracle, cols, tiles, entries, upload):
    rng = np.random.default_rng(cols + sum(entries))
    A = _tile_rows(rng, cols, tiles, entries)
    print(f"convert: {A.rows}x{A.cols}, nnz {A.nnz}", flush=True)
    bm = oracle.bitmap_format(A, 16)
    h = tsp.Handle(validate=True)
    try:
        dA = tsp.to_device(A, **upload)
        for forms in (tsp.FORM_LEFT, tsp.FORM_RIGHT, tsp.FORM_LEFT | tsp.FORM_RIGHT):
            t = h.convert(dA, forms)
            view = t.view()
            slot = tsp.tile_indices(view).cpu().numpy()
            v = {k: (x.cpu().numpy() if hasattr(x, "cpu") else x) for k, x in view.items()}
            assert np.array_equal(v["tile_col"][slot], bm.tile_col)
            assert np.array_equal(v["row_mask"].view(np.uint16).reshape(-1, 16)[slot], bm.row_mask.astype(np.uint16))
            for i in range(slot.size):
                occ = (bm.row_mask[i].astype(np.uint32)[:, None] >> np.arange(16)) & 1 == 1
                want = np.zeros((16, 16), dtype=np.float16)
                want[occ] = bm.elements[bm.index[i]:bm.index[i + 1]]
                for form, bit in (("left", tsp.FORM_LEFT), ("right", tsp.FORM_RIGHT)):
                    if forms & bit:
                        assert np.array_equal(_dense(v, form, int(slot[i])).view(np.uint16), want.view(np.uint16)), (i, form)
            t.free()
    finally:
        h.close()


@pytest.mark.parametrize("cols,tiles,entries", [
    (4096, (8, 9, 7, 1), (600, 560, 500, 256)),                # few tiles
    (4096, (15, 16, 17, 18, 8), (767, 768, 769, 30, 400)),     # the bitmap's half of the image; three entries per thread
    (4096, (32, 33, 65, 3, 250), (560, 570, 600, 500, 520)),   # windows of 32
    (4096, (4, 5, 6), (590, 590, 590)),                        # the mean up to which three registers are taken
    (4096, (4, 5, 6), (591, 591, 591)),
    (4096, (8, 8, 9, 4, 1, 5, 1), (1024, 1023, 1025, 769, 100, 100, 16)),      # a fourth entry of all threads, of one, one entry too many
    (4096, (16, 17, 33, 2, 3), (1024, 900, 770, 30, 20)),
    (524288, (8, 40, 0, 5), (700, 760, 0, 480)),               # spans about the bitmap's
    (524288, (40, 8, 2, 1), (1000, 800, 100, 30)),
    (600000, (30, 2, 8), (500, 300, 600)),
])
@pytest.mark.parametrize("upload", [{}, {"value_dtype": "f32", "row_ptr_dtype": "i64"}])
def test_tile_rows_of_500_entries(tsp, oracle, cols, tiles, entries, upload):
    test_tile_rows_of_many_entries(tsp, oracle, cols, tiles, entries, upload)


@pytest.mark.parametrize("tile_rows,large,small", [
    (40, 2100, 0), (40, 2049, 2049), (40, 2060, 2037),      # a mean either side of what k_convert_block is for, all or half of them large
    (1300, 2100, 1500), (2100, 2050, 60),                   # the same with more tile-rows than k_convert_large has blocks
])
@pytest.mark.parametrize("phases", [False, True])
def test_large_tile_rows_beside_others(tsp, tile_rows, large, small, phases):
    """Times the identity: C is A.  Every third tile-row has `small` entries, the others `large` ones, in 400 columns."""
    rng = np.random.default_rng(tile_rows + large)
    cols = 400
    r, c = [], []
    for i in range(tile_rows):
        pick = np.sort(rng.choice(16 * cols, small if i % 3 == 1 else large, replace=False))
        r.append(16 * i + pick // cols), c.append(pick % cols)
    r, c = np.concatenate(r), np.concatenate(c)
    A = inputs.from_coo(16 * tile_rows, cols, r, c, rng.uniform(-1, 1, r.size), "large tile-rows")
    eye = inputs.from_coo(cols, cols, np.arange(cols), np.arange(cols), np.ones(cols), "identity")
    print(f"large tile-rows: {A.rows}x{cols}, nnz {A.nnz}", flush=True)
    h = tsp.Handle(validate=True)
    try:
        h.set_option(tsp.OPT_WORK_ORDER, 2)                 # (the tile kernels, whatever the operands)
        dA, dI = tsp.to_device(A), tsp.to_device(eye)
        for _ in range(2):
            if phases:
                left, right = h.convert(dA, tsp.FORM_LEFT), h.convert(dI, tsp.FORM_RIGHT)
                plan = h.symbolic(left, right)
                C = h.numeric(left, right, plan)
                plan.free(), left.free(), right.free()
            else:
                C = h.spgemm(dA, dI)
            row_ptr, col, val = C.to_host()
            C.free()
            assert np.array_equal(row_ptr, A.row_ptr) and np.array_equal(col, A.col_idx)
            assert np.array_equal(val, np.asarray(A.val, dtype=np.float16).astype(np.float32))
    finally:
        h.close()


def _full_tiles(rng, tile_rows, tile_cols_of):
    """Four full tiles per tile-row, in the tile columns tile_cols_of(tile-row)."""
    r, c = [], []
    rr, cc = np.repeat(np.arange(16), 16), np.tile(np.arange(16), 16)
    for i in range(tile_rows):
        for j in tile_cols_of(i):
            r.append(i * 16 + rr)
            c.append(int(j) * 16 + cc)
    r, c = np.concatenate(r), np.concatenate(c)
    return inputs.from_coo(16 * tile_rows, 16 * tile_rows, r, c, rng.uniform(-1, 1, r.size), "full tiles")


@pytest.mark.parametrize("phases", [False, True])
def test_another_structure_of_the_same_sizes(tsp, oracle, phases):
    """Products of the same rows and entries, with few and with many tiles in C: the second one does not fit the arrays
    sized after the first, the third one does."""
    n = 1025
    rng = np.random.default_rng(5)
    narrow = _full_tiles(rng, n, lambda i: (np.arange(4) + i // 4 * 4) % n)
    wide = _full_tiles(rng, n, lambda i: rng.choice(n, 4, replace=False))
    ref = [oracle.spgemm(A, A, threads=4) for A in (narrow, wide)]
    h = tsp.Handle(validate=True)
    try:
        dev = [tsp.to_device(A) for A in (narrow, wide)]
        for which in (0, 0, 1, 0, 1, 1):
            if phases:
                t = h.convert(dev[which])
                plan = h.symbolic(t, t)
                C = h.numeric(t, t, plan)
                plan.free(), t.free()
            else:
                C = h.spgemm(dev[which], dev[which])
                assert h.stats()["pairs"] == n * 16
            row_ptr, col, val = C.to_host()
            C.free()
            want = ref[which]
            assert np.array_equal(row_ptr, want.row_ptr) and np.array_equal(col, want.col)
            assert np.all(np.abs(val.astype(np.float64) - want.val) <= 1e-5 * want.mag + 1e-7)
    finally:
        h.close()


@pytest.mark.parametrize("tile_rows", [1, 40, 1025])
def test_another_result_of_the_same_tiles(tsp, oracle, tile_rows):
    """Products of one tile structure with more and with fewer entries in C, and with longer and with shorter rows of
    tiles: the multiplication that has been launched for as many entries as the last product had may not run."""
    k = np.arange(16)
    near = (np.concatenate([k, k[1:]]), np.concatenate([k, k[:-1]]))                # two diagonals
    arrow = (np.concatenate([k, 0 * k[1:]]), np.concatenate([0 * k, k[1:]]))        # a row and a column: a full product
    rng = np.random.default_rng(tile_rows)

    def blocks(local, shift):
        cols = (np.arange(tile_rows) + shift * (np.arange(tile_rows) % 3 == 0)) % tile_rows
        r = (np.arange(tile_rows)[:, None] * 16 + local[0]).ravel()
        c = (cols[:, None] * 16 + local[1]).ravel()
        return inputs.from_coo(16 * tile_rows, 16 * tile_rows, r, c, rng.uniform(-1, 1, r.size), "tiles")

    all_of = [blocks(near, 0), blocks(arrow, 0), blocks(arrow, 1)]
    ref = [oracle.spgemm(A, A, threads=4) for A in all_of]
    h = tsp.Handle(validate=True)
    try:
        h.set_option(tsp.OPT_WORK_ORDER, 2)        # (the tile kernels, whatever the operands)
        dev = [tsp.to_device(A) for A in all_of]
        for which in (0, 0, 1, 1, 0, 2, 2, 1):
            C = h.spgemm(dev[which], dev[which])
            row_ptr, col, val = C.to_host()
            C.free()
            want = ref[which]
            assert h.stats()["pairs"] == tile_rows
            assert np.array_equal(row_ptr, want.row_ptr) and np.array_equal(col, want.col)
            assert np.all(np.abs(val.astype(np.float64) - want.val) <= 1e-5 * want.mag + 1e-7)
    finally:
        h.close()


@pytest.mark.parametrize("tile_rows", [1, 1024, 1025, 65537])
def test_prefix_sums_over_tile_rows(tsp, oracle, tile_rows):
    """Tile-rows either side of a block of the prefix sums, and more than 64 blocks."""
    rng = np.random.default_rng(tile_rows)
    n = 16 * tile_rows - 3
    r = np.concatenate([np.arange(n), rng.integers(0, n, n // 4)])
    c = np.concatenate([(np.arange(n) * 7) % n, rng.integers(0, n, n // 4)])
    key = np.unique(r * n + c)
    A = inputs.from_coo(n, n, key // n, key % n, rng.uniform(-1, 1, key.size), "two per row")
    want = oracle.spgemm(A, A, threads=4)
    h = tsp.Handle(validate=True)
    try:
        dA = tsp.to_device(A)
        t = h.convert(dA)
        plan = h.symbolic(t, t)
        C = h.numeric(t, t, plan)
        row_ptr, col, val = C.to_host()
        assert np.array_equal(row_ptr, want.row_ptr) and np.array_equal(col, want.col)
        assert np.all(np.abs(val.astype(np.float64) - want.val) <= 1e-5 * want.mag + 1e-7)
        C.free(), plan.free(), t.free()
    finally:
        h.close()


@pytest.mark.parametrize("tile_rows,tile_cols,right_tiles", [
    (1, 1, 3), (3, 64, 60), (63, 40, 3), (64, 2000, 3), (64, 2000, 60), (65, 24576, 3), (129, 24576, 60), (129, 24577, 3), (4096, 31, 3),
    (4160, 33, 3), (4160, 130, 60), (32768, 20, 3), (32769, 20, 3)])
def test_sizes_of_tile_rows_found_with_the_task_list(tsp, oracle, tile_rows, tile_cols, right_tiles):
    """Products of sizes that the handle knows, whose task list is made without a count of the tile-rows first: as many of them as a
    group and one more or less, as many as there are slots for, few pairs and many, B as wide as the bitmap holds and one tile more; empty
    tile-rows, and the last one with and without an entry.  The plan is that of the first product, array by array, also after one with
    more in it, whose arrays do not do."""
    rng = np.random.default_rng(tile_rows)
    inner = 70

    def operand(rows, cols, tiles):
        r, c = [], []
        for i in range(rows):
            for j in rng.choice(cols, min(cols, tiles(i)), replace=False):
                r.append(i * 16 + rng.integers(0, 16, 3))
                c.append(j * 16 + rng.integers(0, 16, 3))
        key = np.unique(np.concatenate(r) * (16 * cols) + np.concatenate(c))
        return key // (16 * cols), key % (16 * cols)

    def same_number(entries, rows, cols):
        n = min(x[0].size for x in entries)
        out = []
        for r, c in entries:
            keep = np.sort(rng.permutation(r.size)[:n])
            out.append(inputs.from_coo(16 * rows, 16 * cols, r[keep], c[keep], rng.uniform(-1, 1, n), "tiles"))
        return out

    few = operand(tile_rows, inner, lambda i: 0 if i % 7 == 5 and i else 1 + i % 3)
    more = operand(tile_rows, inner, lambda i: 66 if i in (0, tile_rows - 1) else 2 + i % 2)
    As = same_number([few, more], tile_rows, inner)
    r, c = operand(inner, tile_cols, lambda i: right_tiles + i % 5)
    B = inputs.from_coo(16 * inner, 16 * tile_cols, r, c, rng.uniform(-1, 1, r.size), "right")
    want = [oracle.spgemm(A, B, threads=4) for A in As]
    h = tsp.Handle(validate=True)
    try:
        dA, dB = [tsp.to_device(A) for A in As], tsp.to_device(B)
        first = {}
        for which in (0, 0, 0, 1, 0, 1, 1):
            ta, tb = h.convert(dA[which], tsp.FORM_LEFT), h.convert(dB, tsp.FORM_RIGHT)
            plan = h.symbolic(ta, tb)
            view = {k: x.cpu().numpy() if hasattr(x, "cpu") else x for k, x in plan.view().items()}
            C = h.numeric(ta, tb, plan)
            row_ptr, col, val = C.to_host()
            for x in (C, plan, ta, tb):
                x.free()
            ref = want[which]
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
            for k, v in first.setdefault(which, view).items():
                assert np.array_equal(view[k], v), k
    finally:
        h.close()


# a wave per tile-row before and after, a block before and after, first a wave and then a block, and then neither: for more than 1024 pairs,
# for more than 64 tiles of A, and for a few long tile-rows among more than 4096
@pytest.mark.parametrize("tile_rows,tiles,more,right_tiles,counted", [
    (30, 4, 6, 3, False), (30, 4, 50, 3, False), (30, 40, 60, 3, False), (30, 20, 30, 40, True), (90, 4, 70, 3, True), (4200, 2, 7, 3, False), (4200, 2, 60, 12, True)])
def test_a_tile_row_with_more_than_any_before(tsp, oracle, tile_rows, tiles, more, right_tiles, counted):
    """A product of sizes that the handle knows, one of whose tile-rows has more pairs than any had: the tile-rows, whose sizes the task
    list has found by then, are not counted (its first kernel) unless their sizes are beyond it, and the product is what it is on a
    handle of its own."""
    rng = np.random.default_rng(tile_rows + more)
    inner = 70

    def operand(rows, cols, number, total):
        r = np.repeat(np.arange(rows), number)
        c = np.concatenate([np.sort(rng.choice(cols, k, replace=False)) for k in number])
        r, c = np.repeat(r, 4) * 16 + np.tile(np.arange(4), r.size), np.repeat(c, 4) * 16 + np.tile(np.arange(4) * 5, c.size)
        keep = np.sort(rng.permutation(r.size)[:total])
        return inputs.from_coo(16 * rows, 16 * cols, r[keep], c[keep], rng.uniform(-1, 1, total), "tiles")

    number = np.full(tile_rows, tiles)
    other = number.copy()
    other[tile_rows // 2] = more
    total = int(number.sum()) * 4
    As = [operand(tile_rows, inner, n, total) for n in (number, other)]
    B = operand(inner, 50, np.full(inner, right_tiles), inner * right_tiles * 4)
    dB, dev = tsp.to_device(B), [tsp.to_device(A) for A in As]
    ref = oracle.spgemm(As[1], B, threads=4)

    def product(h, k):
        C = h.spgemm(dev[k], dB)
        out = C.to_host()
        C.free()
        stats = h.stats()
        return list(out) + [[stats[k] for k in ("a_tiles", "b_tiles", "candidate_pairs", "pairs", "c_tiles", "c_nnz")], stats["kernel_us"]["sym_count"]]

    h, alone = tsp.Handle(phase_timers=True), tsp.Handle()
    try:
        for x in (h, alone):
            x.set_option(tsp.OPT_WORK_ORDER, 2)        # (the tile kernels, whatever the operands)
        want = product(alone, 1)
        assert np.array_equal(want[0], ref.row_ptr) and np.array_equal(want[1], ref.col)
        assert np.all(np.abs(want[2].astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
        assert product(h, 0)[4] > 0 and product(h, 0)[4] == 0
        for _ in range(2):
            got = product(h, 1)
            assert (got[4] > 0) == counted
            assert all(np.array_equal(x, y) for x, y in zip(got[:4], want[:4]))
            assert (product(h, 0)[4] > 0) == counted
    finally:
        h.close()
        alone.close()


@pytest.mark.parametrize("left,right", [((1, 0), (0, 0)), ((0, 0), (1, 0)), ((1, 1), (0, 1)), (None, None)])
def test_tile_rows_of_many_entries_where_there_were_none(tsp, oracle, left, right):
    """Products of the same sizes with and without tile-rows for the kernel that is not launched where the last one had none."""
    n, tiles = 40, 40
    rng = np.random.default_rng(7)

    def operand(large):
        entries = np.full(n, 700)
        if large:
            entries = np.where(np.isin(np.arange(n), (0, 17, n - 1)), 3000, 514)       # (about as many entries altogether)
        A = _tile_rows(rng, 16 * n, np.full(n, tiles), entries)
        keep = np.sort(rng.permutation(A.nnz)[:27000])
        row = np.repeat(np.arange(A.rows), np.diff(A.row_ptr))[keep]
        return inputs.from_coo(A.rows, A.cols, row, A.col_idx[keep], rng.uniform(-1, 1, keep.size), "large" if large else "even")

    kinds = [operand(False), operand(True)]
    dev = [tsp.to_device(A) for A in kinds]
    h = tsp.Handle(validate=True)
    try:
        h.set_option(tsp.OPT_WORK_ORDER, 2)        # (the tile kernels, whatever the operands)
        pairs = [(0, 0), (0, 0), (1, 1), (0, 0), (1, 1), (1, 1)] if left is None else [(0, 0), (0, 0), left, (0, 0), right, right, (0, 0)]
        others = dev if left is None else [tsp.to_device(A) for A in kinds]
        want = {}
        for i, j in pairs:
            if (i, j) not in want:
                want[i, j] = oracle.spgemm(kinds[i], kinds[j], threads=4)
            C = h.spgemm(dev[i], others[j])
            row_ptr, col, val = C.to_host()
            C.free()
            ref = want[i, j]
            assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(col, ref.col)
            assert np.all(np.abs(val.astype(np.float64) - ref.val) <= 1e-5 * ref.mag + 1e-7)
    finally:
        h.close()


def test_tile_rows_of_many_entries_again_and_again(tsp):
    """Products of the same sizes with tile-rows for that kernel and without: after one that has some where it was not launched, it is
    launched for all until four without any have come one behind the other, and then for eight.  (Where it is not launched the list of
    those tile-rows is kept, a block more than the product takes otherwise.)"""
    n, rng = 40, np.random.default_rng(8)

    def operand(entries):
        A = _tile_rows(rng, 16 * n, np.full(n, 40), entries)
        keep = np.sort(rng.permutation(A.nnz)[:27000])
        row = np.repeat(np.arange(A.rows), np.diff(A.row_ptr))[keep]
        return tsp.to_device(inputs.from_coo(A.rows, A.cols, row, A.col_idx[keep], rng.uniform(-1, 1, keep.size), "tile-rows"))

    even, large = operand(np.full(n, 700)), operand(np.where(np.isin(np.arange(n), (0, 17, n - 1)), 3000, 514))
    h = tsp.Handle()
    try:
        h.set_option(tsp.OPT_WORK_ORDER, 2)        # (the tile kernels, whatever the operands)

        def blocks(A):
            h.trim()
            before = set(h._blocks)
            C = h.spgemm(A, A)
            new = len(set(h._blocks) - before)
            C.free()
            return new

        blocks(even)
        left = blocks(even)                                    # (not launched)
        blocks(large)                                          # (missed)
        always = blocks(large)
        assert left == always + 1
        assert [blocks(even) for _ in range(6)] == [always] * 4 + [left] * 2
        blocks(large)
        for _ in range(2):
            assert [blocks(even) for _ in range(7)] == [always] * 7
            assert blocks(large) == always
        assert [blocks(even) for _ in range(10)] == [always] * 8 + [left] * 2
    finally:
        h.close()


@pytest.mark.parametrize("left_tiles", [1, 31, 32, 33, 63, 64, 65])
def test_tile_rows_of_many_left_tiles(tsp, oracle, left_tiles):
    """A tile-row of A with as many tiles as the words of contributors hold, one more and one less, among short ones."""
    n = 1030
    rng = np.random.default_rng(left_tiles)
    A = _full_tiles(rng, n, lambda i: rng.choice(n, left_tiles, replace=False) if i in (7, n - 1) else (np.array([i, i * 5 + 1]) % n))
    keep = rng.random(A.col_idx.size) < 0.3
    rows = np.repeat(np.arange(A.rows), np.diff(A.row_ptr))[keep]
    A = inputs.from_coo(A.rows, A.cols, rows, A.col_idx[keep], rng.uniform(-1, 1, rows.size), "many left tiles")
    want = oracle.spgemm(A, A, threads=4)
    h = tsp.Handle(validate=True)
    try:
        dA = tsp.to_device(A)
        for _ in range(2):
            t = h.convert(dA)
            plan = h.symbolic(t, t)
            C = h.numeric(t, t, plan)
            row_ptr, col, val = C.to_host()
            assert np.array_equal(row_ptr, want.row_ptr) and np.array_equal(col, want.col)
            assert np.all(np.abs(val.astype(np.float64) - want.val) <= 1e-5 * want.mag + 1e-7)
            C.free(), plan.free(), t.free()
    finally:
        h.close()
