"""The bound that the table of a small row in csrc/rowwise.hip rests on, modelled on the CPU: whatever the row pointers of
the operands hold, a row of A that goes through the table has no more intermediate products than were counted for it, so
that a free slot is left and the search for one ends.  The model restates what k_row_prepare counts and what k_row_small
takes; `mended=False` is the form without the non-decreasing starts, for which the bound does not hold."""
import numpy as np
import pytest

T = 16


def _starts(raw, nnz, mended=True):
    """RowMatrix::start, and the 17 pointers each tile-row counts with."""
    rows = len(raw) - 1
    start, views = np.zeros(rows + 1, np.int64), []
    for i0 in range(0, rows, T):
        p = np.clip([raw[min(i0 + i, rows)] for i in range(T + 1)], 0, nnz)
        if mended:
            p = np.maximum.accumulate(p)
        views.append(p)
        for i in range(T + 1):
            if (i < T) if i0 + i < rows else True:
                start[min(i0 + i, rows)] = p[i]
    return start, views


def _counted(raw, nnz, col, b_raw, b_nnz, mended=True):
    """Products counted per row of A: every entry of a tile-row for the row that a search among its pointers names."""
    rows = len(raw) - 1
    ub = np.zeros(((rows + T - 1) // T) * T, np.int64)
    for I, p in enumerate(_starts(raw, nnz, mended)[1]):
        for k in range(p[0], p[T]):
            r = 0
            for step in (8, 4, 2, 1):
                if p[r + step] <= k:
                    r += step
            s, e = int(b_raw[col[k]]), int(b_raw[col[k] + 1])
            if mended:
                s, e = min(max(s, 0), b_nnz), min(max(e, 0), b_nnz)
                n = e - s
            else:
                n = (e - s + 2 ** 63) % 2 ** 64 - 2 ** 63           # 64-bit arithmetic wraps round
            ub[I * T + r] += min(max(n, 0), (1 << 25) - 1)
    return ub


def _taken(raw, nnz, col, b_raw, b_nnz, mended=True):
    """Products k_row_small forms per row, by the arrays of starts alone."""
    start, b_start = _starts(raw, nnz, mended)[0], _starts(b_raw, b_nnz, mended)[0]
    return [sum(max(b_start[col[k] + 1] - b_start[col[k]], 0) for k in range(start[r], start[r + 1])) for r in range(len(raw) - 1)]


def _garbled(rng, row_ptr, nnz):
    raw = [int(x) for x in row_ptr]
    for _ in range(int(rng.integers(1, 6))):
        i = int(rng.integers(0, len(raw)))
        raw[i] = int(rng.choice([raw[i] + int(rng.integers(-9, 10)), int(rng.integers(-5, nnz + 5)), -2 ** 62 - 7, 2 ** 62 + 9, 2 ** 63 - 1, -2 ** 63]))
    return raw


@pytest.mark.parametrize("seed", range(40))
def test_no_small_row_has_more_products_than_were_counted(seed):
    rng = np.random.default_rng(seed)
    rows, inner = int(rng.integers(17, 70)), int(rng.integers(17, 50))
    a_len, b_len = rng.integers(0, 9, rows), np.where(rng.random(inner) < 0.2, 40, 1)
    a_ptr, b_ptr = np.concatenate([[0], np.cumsum(a_len)]), np.concatenate([[0], np.cumsum(b_len)])
    nnz, b_nnz = int(a_ptr[-1]), int(b_ptr[-1])
    col = rng.integers(0, inner, nnz)
    a_raw = _garbled(rng, a_ptr, nnz) if seed % 3 != 1 else [int(x) for x in a_ptr]
    b_raw = _garbled(rng, b_ptr, b_nnz) if seed % 3 != 0 else [int(x) for x in b_ptr]
    taken, ub = _taken(a_raw, nnz, col, b_raw, b_nnz), _counted(a_raw, nnz, col, b_raw, b_nnz)
    assert all(t <= u for t, u in zip(taken, ub))


def test_the_bound_fails_without_non_decreasing_starts():
    """Row 3 begins behind row 4: row 2 takes three entries that are counted for row 4, and they meet long rows of B."""
    b_ptr = [0, 1, 2, 3, 4, 44, 84, 124]
    a_ptr = [0, 4, 8, 12, 16] + [20 + 4 * i for i in range(16)]
    col = np.arange(int(a_ptr[-1])) % 4
    col[12:15] = [4, 5, 6]
    bad = list(a_ptr)
    bad[3], bad[4] = 15, 12
    assert _counted(bad, len(col), col, b_ptr, 124, mended=False)[2] <= 24 < 32 < _taken(bad, len(col), col, b_ptr, 124, mended=False)[2]
    assert _taken(bad, len(col), col, b_ptr, 124)[2] <= _counted(bad, len(col), col, b_ptr, 124)[2]
    # and where the length of a row of B overflows 64 bits
    far = [0, -2 ** 62 - 7, 2 ** 62 + 9] + b_ptr[3:]
    assert _counted(a_ptr, len(col), col, far, 124, mended=False)[0] < _taken(a_ptr, len(col), col, far, 124, mended=False)[0]
