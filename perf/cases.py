"""The work that a user has this library do, as measurable cases.

A case is one call (or the one sequence of calls) that a program makes with operands on the GPU:

  spgemm     C = A * B in one call, the result in fresh buffers: the usual way in
  phases     symbolic and numeric phase called by themselves, the plan released afterwards
  numeric    numeric phase alone on a kept plan and kept result buffers: new values on an unchanged
             structure, as in a time step or a solver that assembles the same operator again
  pipelined  C = A * B handed out in row blocks
  outer      both operands brought from CSR into the doubly compressed formats, then the outer product
  ttm        sparse 3-tensor (coordinates in any order) times sparse matrix; with fold also the result's
             coordinates

over the operands of the library's own configurations: uniform random rows, ragged random rows (ordered or
not, with repeated columns), the 27-point stencil, R-MAT power-law graphs, the paper's deduplication sweep and
uniform random tensors.  Inputs are made on the GPU from the seed alone.
"""
import math

import torch

from paper_2404_04541_amd import binding as sg

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # configuration 1, the smallest product in use: launches and host time are what it costs
        {"name": "uniform_1000", "op": "spgemm", "kind": "uniform", "dtype": "f64", "m": 1000, "k": 1000, "n": 1000, "a_row": 10, "b_row": 10, "square": True},
        # ragged rows of any length in any order, sizes that divide nothing: general sparse matrices
        {"name": "ragged_5003", "op": "spgemm", "kind": "ragged", "dtype": "f32", "m": 5003, "k": 3001, "n": 7777, "a_mean": 40.0, "b_mean": 25.0, "ordered": False, "repeats": True},
        # a small power-law graph squared: every row class at once, and too little work to fill the card
        {"name": "rmat_14", "op": "spgemm", "kind": "rmat", "dtype": "f32", "scale": 14, "edges": 16},
        # configuration 2, a discretised operator squared (algebraic multigrid, two-step stencils)
        {"name": "stencil_128", "op": "phases", "kind": "stencil", "dtype": "f64", "grid": 128},
        # the same operator on a coarser, odd grid with new coefficients: the structure's plan is kept
        {"name": "stencil_61_values", "op": "numeric", "kind": "stencil", "dtype": "f64", "grid": 61},
        # configuration 3 at half its vertices (both results of a comparison have to fit the card): the largest
        {"name": "rmat_19", "op": "spgemm", "kind": "rmat", "dtype": "f32", "scale": 19, "edges": 16},
        # configuration 4, a tall sparse product with short rows (restriction, graph lookup)
        {"name": "rect_4194304", "op": "spgemm", "kind": "uniform", "dtype": "f64", "m": 4194304, "k": 4194304, "n": 65536, "a_row": 8, "b_row": 4, "square": False},
        # configuration 5 from coordinates in any order: unfolding and product
        {"name": "ttm_10m", "op": "ttm", "kind": "tensor", "dtype": "f64", "I": 2048, "J": 2048, "K": 2048, "nnz": 10000000, "mode": 3, "l": 2048, "m_row": 16, "fold": False},
        # a small tensor with unequal odd extents over its first mode, back to a coordinate tensor
        {"name": "ttm_mode1_200k", "op": "ttm", "kind": "tensor", "dtype": "f32", "I": 301, "J": 997, "K": 703, "nnz": 200003, "mode": 1, "l": 512, "m_row": 8, "fold": True},
        # the paper's first-order sweep in its middle: ten products for every entry of the result
        {"name": "dedup_10000", "op": "spgemm", "kind": "dedup", "dtype": "f64", "kdim": 10000},
        # the paper's leading example, the outer product through a coordinate workspace
        {"name": "outer_1m", "op": "outer", "kind": "uniform", "dtype": "f64", "m": 1000003, "k": 1000003, "n": 65536, "a_row": 8, "b_row": 4, "square": False},
        # a power-law graph squared and consumed in row blocks
        {"name": "pipelined_rmat_17", "op": "pipelined", "kind": "rmat", "dtype": "f32", "scale": 17, "edges": 16, "blocks": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    dtype = rng.choice(["f32", "f64"])
    family = rng.choice(["uniform", "uniform", "ragged", "ragged", "stencil", "stencil_values", "rmat", "rmat", "ttm", "ttm", "dedup", "outer", "pipelined"])
    if family == "uniform":
        m = _log_int(rng, 500, 3000000)
        square = rng.random() < 0.3
        k = m if square else _log_int(rng, 500, 3000000)
        n = m if square else _log_int(rng, 300, 500000)
        a = rng.randint(2, 16)
        return {"op": rng.choice(["spgemm", "spgemm", "phases"]), "kind": "uniform", "dtype": dtype, "m": m, "k": k, "n": n, "a_row": a, "b_row": a if square else rng.randint(2, 16), "square": square}
    if family == "ragged":
        return {"op": "spgemm", "kind": "ragged", "dtype": dtype, "m": _log_int(rng, 300, 60000), "k": _log_int(rng, 300, 30000), "n": _log_int(rng, 300, 1000000),
                "a_mean": round(rng.uniform(2, 60), 1), "b_mean": round(rng.uniform(2, 60), 1), "ordered": rng.random() < 0.6, "repeats": rng.random() < 0.3}
    if family == "stencil":
        return {"op": "phases", "kind": "stencil", "dtype": dtype, "grid": _log_int(rng, 6, 128)}
    if family == "stencil_values":
        return {"op": "numeric", "kind": "stencil", "dtype": dtype, "grid": _log_int(rng, 6, 128)}
    if family == "rmat":
        return {"op": rng.choice(["spgemm", "phases", "numeric"]), "kind": "rmat", "dtype": dtype, "scale": rng.randint(10, 18), "edges": rng.randint(7, 16)}
    if family == "ttm":
        I, J, K = (_log_int(rng, 40, 2048) for _ in range(3))
        nnz = min(_log_int(rng, 1000, 10000000), I * J * K // 8)
        return {"op": "ttm", "kind": "tensor", "dtype": dtype, "I": I, "J": J, "K": K, "nnz": nnz, "mode": rng.randint(1, 3), "l": _log_int(rng, 64, 4096),
                "m_row": rng.randint(2, 16), "fold": rng.random() < 0.5}
    if family == "dedup":
        return {"op": "spgemm", "kind": "dedup", "dtype": dtype, "kdim": _log_int(rng, 2500, 40000)}
    if family == "outer":
        m = _log_int(rng, 1000, 1000000)
        return {"op": "outer", "kind": "uniform", "dtype": dtype, "m": m, "k": m, "n": _log_int(rng, 300, 100000), "a_row": rng.randint(2, 8), "b_row": rng.randint(2, 6), "square": False}
    return {"op": "pipelined", "kind": "rmat", "dtype": dtype, "scale": rng.randint(12, 17), "edges": rng.randint(7, 16), "blocks": rng.randint(2, 8)}


# ---- operands ------------------------------------------------------------------------------
# The pattern of a case's operands is drawn once and for all and renumbered from the seed: rows, columns and inner
# index are permuted, which leaves the number of entries of the result (and so the sizes of the outputs) as they
# are.  Graphs are renumbered by an exclusive or of the lower half of the index bits (hubs stay together); stencils
# and graphs that are handed out in row blocks (whose sizes depend on the order of the rows) stay where they are.
# Values always come from the seed.

def _generators(seed):
    return torch.Generator(device="cuda").manual_seed(0), torch.Generator(device="cuda").manual_seed(seed + 1)


def _values(nnz, lo, hi, dtype, gen):
    return torch.rand(nnz, dtype=dtype, device="cuda", generator=gen) * (hi - lo) + lo


def _order(n, gen):
    return torch.randperm(n, device="cuda", generator=gen)


def _rowptr(rows_of_entries, rows):
    rp = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(rows_of_entries, minlength=rows), 0, out=rp[1:])
    return rp


def _csr(rows, cols, r, c, values, gen=None):
    """From coordinates: columns ascending in every row or, with a generator, in any order."""
    if gen is None:
        order = torch.argsort(r * cols + c)
    else:
        order = _order(r.numel(), gen)
        order = order[torch.sort(r[order], stable=True).indices]
    return sg.DeviceCSR(rows, cols, _rowptr(r, rows), c[order].to(torch.int32), values[order])


def _uniform_rows(rows, cols, per_row, gen):
    """Coordinates of per_row distinct uniform columns in every row."""
    per_row = min(per_row, cols)
    c = torch.randint(cols, (rows, per_row), device="cuda", generator=gen)
    while True:
        c = torch.sort(c, dim=1).values
        again = torch.zeros_like(c, dtype=torch.bool)
        again[:, 1:] = c[:, 1:] == c[:, :-1]
        left = int(again.sum())
        if left == 0:
            break
        c[again] = torch.randint(cols, (left,), device="cuda", generator=gen)
    return torch.repeat_interleave(torch.arange(rows, device="cuda"), per_row), c.reshape(-1)


def _ragged_rows(rows, cols, mean, repeats, gen):
    """Row lengths spread geometrically around the mean (empty rows among them, four times the mean at most), uniform columns."""
    u = torch.rand(rows, dtype=torch.float64, device="cuda", generator=gen)
    lens = torch.clamp((-torch.log1p(-u) * mean).floor(), max=min(4 * mean + 1, cols)).to(torch.int64)
    r = torch.repeat_interleave(torch.arange(rows, device="cuda"), lens)
    c = torch.randint(cols, (r.numel(),), device="cuda", generator=gen)
    if not repeats:
        key = torch.unique(r * cols + c)
        r, c = key // cols, key % cols
    return r, c


def _stencil(grid, dtype, gen):
    """27-point stencil on a clipped grid^3, row = x + grid * (y + grid * z), values in [-1, 1)."""
    n = grid ** 3
    i = torch.arange(n, device="cuda")
    x, y, z = i % grid, (i // grid) % grid, i // (grid * grid)
    d = torch.tensor([-1, 0, 1], device="cuda")
    ok = lambda v: (v >= 0) & (v < grid)  # noqa: E731
    zz, yy, xx = z[:, None] + d, y[:, None] + d, x[:, None] + d
    keep = ok(zz)[:, :, None, None] & ok(yy)[:, None, :, None] & ok(xx)[:, None, None, :]
    col = xx[:, None, None, :] + grid * (yy[:, None, :, None] + grid * zz[:, :, None, None])
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(keep.reshape(n, 27).sum(1), 0, out=rp[1:])
    col = col[keep].to(torch.int32)
    return sg.DeviceCSR(n, n, rp, col, _values(col.numel(), -1.0, 1.0, dtype, gen))


def _rmat(scale, edges, renumber, dtype, fixed, gen):
    """R-MAT graph (0.57, 0.19, 0.19, 0.05), so many edges per vertex drawn, repeated edges merged, values in [0, 1)."""
    n = 1 << scale
    r = torch.zeros(edges * n, dtype=torch.int64, device="cuda")
    c = torch.zeros_like(r)
    for _ in range(scale):
        u = torch.rand(edges * n, device="cuda", generator=fixed)
        r = (r << 1) | (u >= 0.76)
        c = (c << 1) | (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    key = torch.unique((r << scale) | c)
    mask = torch.randint(1 << (scale // 2), (1,), device="cuda", generator=gen) if renumber else 0
    return _csr(n, n, (key >> scale) ^ mask, (key & (n - 1)) ^ mask, _values(key.numel(), 0.0, 1.0, dtype, gen))


def _dedup_sizes(kdim):
    rows = 100000000 // kdim
    return rows, max(1, round(kdim / 10)), min(1000, rows)   # rows of B, non-empty columns, entries in each of them


def _dedup(kdim, fixed):
    """Coordinates of B (rows x kdim) with a tenth of its columns non-empty, 1000 entries each."""
    rows, nc, per = _dedup_sizes(kdim)
    r = torch.topk(torch.rand((nc, rows), device="cuda", generator=fixed), per, dim=1, sorted=False).indices.reshape(-1)
    return r, torch.repeat_interleave(_order(kdim, fixed)[:nc], per)


def _tensor(I, J, K, nnz, gen):
    """nnz distinct uniform coordinates."""
    lin = torch.empty(0, dtype=torch.int64, device="cuda")
    while lin.numel() < nnz:
        more = torch.randint(I * J * K, (nnz - lin.numel() + nnz // 64 + 16,), device="cuda", generator=gen)
        lin = torch.unique(torch.cat([lin, more]))
    lin = lin[_order(lin.numel(), gen)[:nnz]]
    return [lin // (J * K), (lin // K) % J, lin % K]


def _contracted(case):
    return (case["I"], case["J"], case["K"])[case["mode"] - 1]


def prepare(case, seed):
    fixed, gen = _generators(seed)
    dtype = DTYPES[case["dtype"]]
    kind = case["kind"]
    state = {"case": case, "handle": sg.Handle()}
    if kind == "tensor":
        x = _tensor(case["I"], case["J"], case["K"], case["nnz"], fixed)
        k = _contracted(case)
        mr, mc = _uniform_rows(k, case["l"], case["m_row"], fixed)
        label = [_order(case[e], gen) for e in "IJK"]
        shuffle = _order(case["nnz"], gen)
        state["x"] = [label[d][x[d]][shuffle].to(torch.int32) for d in range(3)] + [_values(case["nnz"], -1.0, 1.0, dtype, gen)]
        state["m"] = _csr(k, case["l"], label[case["mode"] - 1][mr], _order(case["l"], gen)[mc], _values(mr.numel(), -1.0, 1.0, dtype, gen))
        return state
    if kind == "stencil":
        a = b = _stencil(case["grid"], dtype, gen)
    elif kind == "rmat":
        a = b = _rmat(case["scale"], case["edges"], case["op"] != "pipelined", dtype, fixed, gen)
    elif case.get("square"):
        m = case["m"]
        r, c = _uniform_rows(m, m, case["a_row"], fixed)
        label = _order(m, gen)
        a = b = _csr(m, m, label[r], label[c], _values(r.numel(), -1.0, 1.0, dtype, gen))
    else:
        if kind == "dedup":   # the second operand is the first one's transpose, rotated by one column
            m, k, n = _dedup_sizes(case["kdim"])[0], case["kdim"], _dedup_sizes(case["kdim"])[0]
            ar, ac = _dedup(k, fixed)
            br, bc = ac, (ar + 1) % m
        else:
            m, k, n = case["m"], case["k"], case["n"]
            if kind == "uniform":
                ar, ac = _uniform_rows(m, k, case["a_row"], fixed)
                br, bc = _uniform_rows(k, n, case["b_row"], fixed)
            else:
                ar, ac = _ragged_rows(m, k, case["a_mean"], case["repeats"], fixed)
                br, bc = _ragged_rows(k, n, case["b_mean"], case["repeats"], fixed)
        any_order = None if case.get("ordered", True) else gen
        inner = _order(k, gen)
        a = _csr(m, k, _order(m, gen)[ar], inner[ac], _values(ar.numel(), -1.0, 1.0, dtype, gen), any_order)
        b = _csr(k, n, inner[br], _order(n, gen)[bc], _values(br.numel(), -1.0, 1.0, dtype, gen), any_order)
    state["a"], state["b"] = a, b
    if case["op"] == "numeric":
        state["rowptr"], nnz, state["plan"] = sg.spgemm_symbolic(state["handle"], a, b)
        state["col"] = torch.empty(nnz, dtype=torch.int32, device="cuda")
        state["val"] = torch.empty(nnz, dtype=dtype, device="cuda")
    return state


def run(state):
    case, h = state["case"], state["handle"]
    op = case["op"]
    if op == "ttm":
        y = sg.spttm(h, case["mode"], (case["I"], case["J"], case["K"]), *state["x"], state["m"])
        if not case["fold"]:
            return y.rowptr, y.colidx, y.values
        shape = [case["I"], case["J"], case["K"]]
        shape[case["mode"] - 1] = case["l"]
        return (y.values,) + sg.sptensor_fold(h, case["mode"], shape, y)
    a, b = state["a"], state["b"]
    if op == "spgemm":
        c = sg.spgemm(h, a, b)
        return c.rowptr, c.colidx, c.values
    if op == "phases":
        rowptr, _, plan = sg.spgemm_symbolic(h, a, b)
        col, val = sg.spgemm_numeric(h, plan, a, b, rowptr)
        plan.destroy()
        return rowptr, col, val
    if op == "numeric":
        return sg.spgemm_numeric(h, state["plan"], a, b, state["rowptr"], state["col"], state["val"])
    if op == "outer":
        c = sg.spgemm_outer(h, sg.dcsc_from_csr(h, a), sg.dcsr_from_csr(h, b))
        return c.rowptr, c.colidx, c.values
    blocks, first = sg.spgemm_pipelined(h, a, b, case["blocks"])
    return first, [(c.rowptr, c.colidx, c.values) for c in blocks]


# ---- what a pass cannot do without ----------------------------------------------------------

def _distinct(slots, draws):
    """Expected number of distinct values of so many uniform draws."""
    return slots * -math.expm1(draws * math.log1p(-1.0 / slots)) if slots > 1 else min(1.0, draws)


def _sizes(case):
    """rows of A and B, entries of A and B, products, entries of C (expected values where they are drawn)."""
    kind = case["kind"]
    if kind == "uniform":
        nb = min(case["b_row"], case["n"])
        per = case["a_row"] * nb
        return case["m"], case["k"], case["m"] * case["a_row"], case["k"] * nb, case["m"] * per, case["m"] * _distinct(case["n"], per)
    if kind == "ragged":
        a, b = max(case["a_mean"] - 0.5, 0.5), max(case["b_mean"] - 0.5, 0.5)   # (the lengths are rounded down)
        return case["m"], case["k"], case["m"] * a, case["k"] * b, case["m"] * a * b, case["m"] * _distinct(case["n"], a * b)
    if kind == "stencil":
        g = case["grid"]
        return g ** 3, g ** 3, (3 * g - 2) ** 3, (3 * g - 2) ** 3, (9 * g - 10) ** 3, (5 * g - 6) ** 3
    if kind == "rmat":   # (through what scales 12 and 20 give with 16 edges; the scales between are within a tenth of it)
        s, e = case["scale"], case["edges"] / 16
        na = 2 ** s * e * (11.6 + 0.19 * s)
        return 1 << s, 1 << s, na, na, 6.72e6 * 2.733 ** (s - 12) * e ** 2, 2.343e6 * 2.832 ** (s - 12) * e ** 1.8
    rows, nc, per = _dedup_sizes(case["kdim"])
    return rows, case["kdim"], nc * per, nc * per, nc * per * per, rows * rows * -math.expm1(nc * math.log1p(-min(0.999999, (per / rows) ** 2)))


def work(case):
    v = 4 if case["dtype"] == "f32" else 8
    if case["kind"] == "tensor":
        k = _contracted(case)
        rows = case["I"] * case["J"] * case["K"] // k
        per = min(case["m_row"], case["l"])
        filled = _distinct(rows, case["nnz"])
        out = filled * _distinct(case["l"], case["nnz"] / filled * per)
        total = case["nnz"] * (12 + v) + k * (8 + per * (4 + v)) + 8 * rows + out * (4 + v) + (12 * out if case["fold"] else 0)
        return {"bytes": total, "flops": 2.0 * case["nnz"] * per}
    ra, rb, na, nb, ip, nc = _sizes(case)
    one = case["kind"] in ("stencil", "rmat") or case.get("square", False)
    operands = 8 * ra + na * (4 + v) + (0 if one else 8 * rb + nb * (4 + v))
    return {"bytes": operands + 8 * ra + nc * (4 + v), "flops": 2.0 * ip}


def tolerance(case):
    # Sums are kept in double for both value types and rounded once: two orders of summation differ in the last
    # bits of a double; single precision results differ where a sum lies next to the middle of two floats.
    return {"rel": 1e-15, "max": 2e-14} if case["dtype"] == "f64" else {"rel": 1e-9, "max": 2.5e-7}
