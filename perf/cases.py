"""The products this library is timed on, from the smallest call to the largest.

Every case is a plain dict: the kind of matrix, its size, the types of its arrays and the call made on it.  The
inputs are made on the GPU and have the structure of the generators in ``paper_2009_14600_amd/inputs.py`` (mesh
operators, stencils with several unknowns per node, power-law graphs, block-clustered and uniformly random matrices,
ragged rectangles).  Values differ from seed to seed, and so do the patterns of the matrices that are not meshes: their
rows and columns are renumbered by the seed, which keeps the size of the result.

One program works on one kind of product with one handle: the states of one case share it, each state has operands of
its own and holds its latest result, which it gives back before it asks for the next one.
"""
from __future__ import annotations

import json
import weakref

import torch

from paper_2009_14600_amd import tsp


def listed() -> list:
    return [
        # A mesh operator of a small grid: the coarse levels of a solver, the smallest calls; launches and latency count.
        {"name": "mesh2d_37", "kind": "mesh2d", "g": 37, "values": "f32", "row_ptr": "i32", "call": "spgemm"},
        # The benchmark's first configuration: a small uniformly random matrix, one entry in nearly every tile.
        {"name": "random_1024", "kind": "random", "n": 1024, "per_row": 8, "values": "f16", "row_ptr": "i32", "call": "spgemm"},
        # The second: the 5-point operator on a 512 x 512 grid, the ordinary mesh problem.
        {"name": "mesh2d_512", "kind": "mesh2d", "g": 512, "values": "f16", "row_ptr": "i32", "call": "spgemm"},
        # The third: three coupled unknowns per node, 27 neighbours: structural mechanics, the regime of the tiled method.
        {"name": "stencil27_48x3", "kind": "stencil27", "g": 48, "dof": 3, "values": "f16", "row_ptr": "i32", "call": "spgemm"},
        # The fourth, the headline: two-hop neighbourhoods of a power-law graph; the largest case.
        {"name": "rmat_18", "kind": "rmat", "scale": 18, "edge_factor": 16, "values": "f16", "row_ptr": "i32", "call": "spgemm"},
        # The fifth: half-full 16 x 16 blocks at random places.
        {"name": "blocks_131072", "kind": "blocks", "nb": 8192, "blocks": 4, "edge": 16, "fill": 0.5, "values": "f16",
         "row_ptr": "i32", "call": "spgemm"},
        # A large uniformly random matrix with short rows: the least favourable structure for tiles.
        {"name": "random_65536", "kind": "random", "n": 65536, "per_row": 8, "values": "f32", "row_ptr": "i32", "call": "spgemm"},
        # Operator times prolongator of a multigrid set-up (64^3 grid, aggregates of 2^3 nodes): rectangular A*B in the
        # types such a program has.
        {"name": "coarsen3d_64", "kind": "coarsen3d", "g": 64, "values": "f32", "row_ptr": "i64", "call": "spgemm"},
        # Ragged rectangles of moderate density with empty rows: nearly every output tile filled, long inner sums.
        {"name": "ragged_4099", "kind": "ragged", "rows": 4099, "inner": 2051, "cols": 6007, "density": 0.02, "values": "f32",
         "row_ptr": "i64", "call": "spgemm"},
        # A signed graph of medium size whose cancelled entries are to leave the result (the strictly sparse option).
        {"name": "signed_rmat_14", "kind": "rmat", "scale": 14, "edge_factor": 12, "values": "f16", "row_ptr": "i32",
         "call": "spgemm_compact"},
        # The phases by hand: the right operand stays in tile form, left operands come and go.
        {"name": "phases_blocks_24576", "kind": "blocks", "nb": 1537, "blocks": 6, "edge": 16, "fill": 0.35, "values": "f32",
         "row_ptr": "i32", "call": "phases"},
        # The compaction of zeros alone on a result with a fifth of its values cancelled, into the caller's own arrays.
        {"name": "compact_200003", "kind": "zeros", "rows": 200003, "per_row": 60, "share": 0.2, "call": "compact_static"},
    ]


def draw(rng) -> dict:
    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    types = {"values": rng.choice(["f16", "f32"]), "row_ptr": rng.choice(["i32", "i32", "i64"])}
    call = rng.choice(["spgemm", "spgemm", "spgemm", "phases"])
    kind = rng.choice(["mesh2d", "random", "stencil27", "rmat", "blocks", "coarsen3d", "ragged", "zeros"])
    if kind == "mesh2d":
        return {"kind": kind, "g": log(24, 1000), **types, "call": call}
    if kind == "random":
        return {"kind": kind, "n": log(200, 80000), "per_row": rng.randint(3, 12), **types, "call": call}
    if kind == "stencil27":
        dof = rng.randint(1, 4)
        return {"kind": kind, "g": log(7, 48 if dof < 4 else 40), "dof": dof, **types, "call": call}
    if kind == "rmat":
        # (the compaction is drawn here only: these sums are exact, so that which of them are zero is certain)
        scale = rng.randint(10, 17)
        return {"kind": kind, "scale": scale, "edge_factor": rng.randint(4, 16), **types,
                "call": rng.choice(["spgemm", "spgemm_compact", "phases"]) if scale <= 15 else "spgemm"}
    if kind == "blocks":
        return {"kind": kind, "nb": log(60, 8192), "blocks": rng.randint(2, 6), "edge": rng.choice([12, 16, 16, 16, 20]),
                "fill": round(rng.uniform(0.2, 0.9), 2), **types, "call": call}
    if kind == "coarsen3d":
        return {"kind": kind, "g": log(10, 100), **types, "call": call}
    if kind == "ragged":
        return {"kind": kind, "rows": log(100, 6000), "inner": log(100, 6000), "cols": log(100, 6000),
                "density": round(0.002 * 25 ** rng.random(), 5), **types, "call": call}
    return {"kind": kind, "rows": log(1000, 500000), "per_row": log(4, 100), "share": round(rng.uniform(0.0, 0.5), 2),
            "call": rng.choice(["compact", "compact_static"])}


# ---- inputs -------------------------------------------------------------------------------------------------------
class _Pattern:
    """A canonical CSR pattern on the device: row lengths and ascending column indices."""

    def __init__(self, rows, cols, lengths, col):
        self.rows, self.cols = int(rows), int(cols)
        self.row_ptr = torch.zeros(self.rows + 1, dtype=torch.int64, device=col.device)
        torch.cumsum(lengths, 0, out=self.row_ptr[1:])
        self.col = col.to(torch.int32)


def _from_keys(rows, cols, keys) -> _Pattern:
    """From the ascending, distinct keys row * cols + column."""
    r = torch.div(keys, cols, rounding_mode="floor")
    return _Pattern(rows, cols, torch.bincount(r, minlength=rows), keys - r * cols)


def _rows_of(p):
    return torch.repeat_interleave(torch.arange(p.rows, device=p.col.device), p.row_ptr[1:] - p.row_ptr[:-1])


def _rolled(p, down, right) -> _Pattern:
    """The rows moved on by `down` and the columns by `right`, around the ends."""
    r, c = (_rows_of(p) + down) % p.rows, (p.col.long() + right) % p.cols
    return _from_keys(p.rows, p.cols, (r * p.cols + c).sort().values)


def _moves(seed):
    return torch.randint(0, 1 << 30, (3,), generator=torch.Generator().manual_seed(31 + seed)).tolist()


def _renumbering(case, seed):
    """Bits by which the vertices of a graph are renumbered (low ones: the hubs stay at the low indices)."""
    return _moves(seed)[0] & ((1 << (case["scale"] // 2)) - 1)


def _distinct(gen, dev, lists, count, limit):
    """`lists` ascending lists of `count` distinct numbers below `limit`."""
    x = torch.randint(0, limit - count + 1, (lists, count), generator=gen, device=dev)
    return x.sort(dim=1).values + torch.arange(count, device=dev)


def _grid_operator(shape, offsets, dev) -> _Pattern:
    """Neighbours at the given offsets on a grid in natural order, cut off at the boundary; x runs fastest."""
    n = 1
    for s in shape:
        n *= s
    idx = torch.arange(n, device=dev)
    at, coords = idx, []
    for s in reversed(shape):
        coords.append(at % s)
        at = torch.div(at, s, rounding_mode="floor")
    strides, st = [], 1
    for s in reversed(shape):
        strides.append(st)
        st *= s
    cols, oks = [], []
    for off in sorted(offsets, key=lambda o: sum(a * b for a, b in zip(o, strides))):
        ok = torch.ones(n, dtype=torch.bool, device=dev)
        for c, d, s in zip(coords, off, reversed(shape)):
            ok &= (c + d >= 0) & (c + d < s)
        oks.append(ok)
        cols.append(idx + sum(a * b for a, b in zip(off, strides)))
    ok = torch.stack(oks, 1)
    return _Pattern(n, n, ok.sum(1), torch.stack(cols, 1)[ok])


def _patterns(case, seed, dev):
    """(A, B) of the case; B is None for A*A."""
    gen = torch.Generator(device=dev).manual_seed(200914600)
    moves = _moves(seed)
    kind = case["kind"]
    if kind == "mesh2d":
        g = case["g"]
        return _grid_operator((g, g), [(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1)], dev), None
    if kind == "random":
        n, k = case["n"], case["per_row"]
        p = _Pattern(n, n, torch.full((n,), k, device=dev), _distinct(gen, dev, n, k, n).reshape(-1))
        return _rolled(p, moves[0], moves[0]), None
    if kind == "stencil27":
        g, dof = case["g"], case["dof"]
        idx = torch.arange(g ** 3, device=dev)
        x, y, z = idx % g, torch.div(idx, g, rounding_mode="floor") % g, torch.div(idx, g * g, rounding_mode="floor")
        near = torch.stack([(x + dx) % g + g * ((y + dy) % g + g * ((z + dz) % g))
                            for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)], 1).sort(dim=1).values
        cols = (near[:, :, None] * dof + torch.arange(dof, device=dev)).reshape(g ** 3, 1, 27 * dof)
        n = g ** 3 * dof
        return _Pattern(n, n, torch.full((n,), 27 * dof, device=dev), cols.expand(-1, dof, -1).reshape(-1)), None
    if kind == "rmat":
        n, m = 1 << case["scale"], case["edge_factor"] << case["scale"]
        r = torch.zeros(m, dtype=torch.int64, device=dev)
        c = torch.zeros_like(r)
        for _ in range(case["scale"]):                     # quadrant probabilities 0.57, 0.19, 0.19, 0.05
            u = torch.rand(m, generator=gen, device=dev)
            r = 2 * r + (u >= 0.76)
            c = 2 * c + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
        flip = _renumbering(case, seed)
        r, c = r[r != c] ^ flip, c[r != c] ^ flip
        return _from_keys(n, n, torch.unique(torch.cat([r * n + c, c * n + r]))), None
    if kind == "blocks":
        def one(down, right):
            nb, k, e = case["nb"], case["blocks"], case["edge"]
            at = _distinct(gen, dev, nb, k, nb)
            full = torch.rand((nb, e, k, e), generator=gen, device=dev) < case["fill"]
            cols = (at[:, None, :, None] * e + torch.arange(e, device=dev)).expand(nb, e, k, e)
            return _rolled(_Pattern(nb * e, nb * e, full.reshape(nb * e, -1).sum(1), cols[full]), e * down, e * right)
        if case["call"] == "phases":
            return one(moves[0], moves[1]), one(moves[1], moves[2])
        return one(moves[0], moves[0]), None
    if kind == "coarsen3d":
        g = case["g"]
        A = _grid_operator((g, g, g), [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)], dev)
        idx, h = torch.arange(g ** 3, device=dev), (g + 1) // 2
        x, y, z = [torch.div(v, 2, rounding_mode="floor") for v in
                   (idx % g, torch.div(idx, g, rounding_mode="floor") % g, torch.div(idx, g * g, rounding_mode="floor"))]
        return A, _Pattern(g ** 3, h ** 3, torch.ones(g ** 3, dtype=torch.int64, device=dev), x + h * (y + h * z))
    if kind == "ragged":
        def one(rows, cols):
            full = torch.rand((rows, cols), generator=gen, device=dev) < case["density"]
            full[torch.rand(rows, generator=gen, device=dev) < 0.1] = False        # a tenth of the rows is empty
            return _Pattern(rows, cols, full.sum(1), full.nonzero()[:, 1])
        return (_rolled(one(case["rows"], case["inner"]), moves[0], moves[1]),
                _rolled(one(case["inner"], case["cols"]), moves[1], moves[2]))
    raise ValueError(kind)


def _values(case, seed, p, which):
    gen = torch.Generator(device=p.col.device).manual_seed(77 + 1000 * seed + which)
    if case["kind"] == "rmat":
        # +1 and -1 (agreeing and disagreeing links): a sign of the link itself, and one for each of its ends from the
        # seed, which turn the signs of whole rows and columns of the result and keep the places that cancel
        flip = _renumbering(case, seed)
        r, c = _rows_of(p), p.col.long()
        link = (((r ^ flip) * 40503 + (c ^ flip) * 30011) >> 7) & 1
        end = torch.randint(0, 2, (p.rows,), generator=gen, device=p.col.device)
        v = 1.0 - 2.0 * (link ^ end[r] ^ end[c])
    else:
        v = torch.rand(p.col.numel(), generator=gen, device=p.col.device) * 2.0 - 1.0
    return v.to(torch.float16 if case["values"] == "f16" else torch.float32)


def _operand(case, seed, p: _Pattern, which):
    row_ptr = p.row_ptr if case["row_ptr"] == "i64" else p.row_ptr.to(torch.int32)
    return tsp.DeviceCSR(p.rows, p.cols, row_ptr, p.col, _values(case, seed, p, which))


class _Program:
    """What the states of one case share: the handle."""

    def __init__(self, case):
        self.handle = tsp.Handle()
        if case["call"] == "spgemm_compact":
            self.handle.set_option(tsp.OPT_COMPACT_ZEROS, 1)

    def __del__(self):
        self.handle.close()


_programs = weakref.WeakValueDictionary()


def _program(case) -> _Program:
    key = json.dumps({k: v for k, v in case.items() if k != "name"}, sort_keys=True)
    p = _programs.get(key)
    if p is None:
        p = _programs[key] = _Program(case)
    return p


class _State:
    C = None
    kept = None

    def __init__(self, case, seed):
        dev = torch.device("cuda", torch.cuda.current_device())
        self.call = case["call"]
        self.program = _program(case)
        self.handle = self.program.handle
        if case["kind"] == "zeros":
            self.A = _result_with_zeros(case, seed, dev)
            if self.call == "compact_static":
                self.out = (torch.empty(case["rows"] + 1, dtype=torch.int64, device=dev),
                            torch.zeros(self.A.nnz, dtype=torch.int32, device=dev),
                            torch.zeros(self.A.nnz, dtype=torch.float32, device=dev))
            return
        a, b = _patterns(case, seed, dev)
        self.A = _operand(case, seed, a, 0)
        self.B = self.A if b is None else _operand(case, seed, b, 1)
        if self.call == "phases":
            self.kept = self.handle.convert(self.B, tsp.FORM_RIGHT)

    def __del__(self):
        for x in (self.C, self.kept):
            if x is not None:
                x.free()


def _result_with_zeros(case, seed, dev):
    """A CSR result as tsp_spgemm gives it, with rows of varying length and a share of its values zero."""
    gen = torch.Generator(device=dev).manual_seed(5)
    rows, mean = case["rows"], case["per_row"]
    lengths = torch.randint(0, 2 * mean + 1, (rows,), generator=gen, device=dev).roll(seed)
    n = int(lengths.sum())
    first = torch.zeros(rows + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lengths, 0, out=first[1:])
    col = 3 * (torch.arange(n, device=dev) - torch.repeat_interleave(first[:-1], lengths))
    zero = (torch.rand(n, generator=gen, device=dev) < case["share"]).roll(7 * seed)
    val = torch.rand(n, generator=torch.Generator(device=dev).manual_seed(6 + seed), device=dev) + 0.25
    val[zero] = 0.0
    return tsp.DeviceCSR(rows, 6 * mean + 1, first, col.to(torch.int32), val)


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    h = state.handle
    if state.call == "compact_static":
        nnz = h.compact_zeros_static(state.A, *state.out)
        return state.out[0], state.out[1][:nnz], state.out[2][:nnz]
    if state.C is not None:
        state.C.free()
        state.C = None
    if state.call == "compact":
        C = h.compact_zeros(state.A)
    elif state.call == "phases":
        left = h.convert(state.A, tsp.FORM_LEFT)
        plan = h.symbolic(left, state.kept)
        C = h.numeric(left, state.kept, plan)
        plan.free()
        left.free()
    else:
        C = h.spgemm(state.A, state.B)
    state.C = C
    return C.row_ptr, C.col_idx, C.val


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _csr_bytes(case, p):
    return (p.rows + 1) * (8 if case["row_ptr"] == "i64" else 4) + p.col.numel() * (4 + (2 if case["values"] == "f16" else 4))


def work(case):
    """The operands read once and the result written once; two operations per intermediate product.  The products are
    counted on the operands of seed 0, the entries of the result on an even sample of its rows."""
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "zeros":
        n = case["rows"] * case["per_row"]
        left = n * (1.0 - case["share"])
        return {"bytes": 16.0 * (case["rows"] + 1) + 8.0 * n + 8.0 * left, "flops": 0}
    a, b = _patterns(case, 0, dev)
    alias, b = b is None, a if b is None else b
    lengths = b.row_ptr[1:] - b.row_ptr[:-1]
    products = int(lengths[a.col.long()].sum())
    sample = torch.unique(torch.linspace(0, a.rows - 1, min(a.rows, 512), device=dev).round().long()).tolist()
    begin = a.row_ptr.tolist()
    entries = met = 0
    for r in sample:
        ks = a.col[begin[r]:begin[r + 1]].long()
        n = lengths[ks]
        total = int(n.sum())
        if not total:
            continue
        where = torch.repeat_interleave(b.row_ptr[ks] - (torch.cumsum(n, 0) - n), n) + torch.arange(total, device=dev)
        entries += int(torch.unique(b.col[where]).numel())
        met += total
    nnz = entries * products / met if met else 0.0
    read = _csr_bytes(case, a)
    if not alias and case["call"] != "phases":             # (a kept right operand is read in tile form: its values)
        read += _csr_bytes(case, b)
    elif case["call"] == "phases":
        read += 2 * b.col.numel()
    return {"bytes": float(read + 8 * (a.rows + 1) + 8.0 * nnz), "flops": 2.0 * products}


def tolerance(case):
    if case["kind"] == "zeros":
        return "exact"                                     # values are copied
    if case["kind"] == "rmat":
        return "exact"                                     # sums of +1 and -1: exact in any order
    return {"rel": 1e-5}                                   # exact products of fp16 numbers, summed in fp32
