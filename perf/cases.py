"""The multiplies, searches and rankings that programs ask of this package, as timed cases.

A case is a dict of plain values.  `kind` says which entry point it goes
through; the rest are sizes and options:

  mul        Matrix.spmspv: y <- A x on lists, any semiring, with or without
             a bitmap mask, plain or deterministic
  graphblas  spmspv_run_graphblas: w<mask> = w + A x
  batch      Matrix.spmspv_batch: many x against one A in one call
  bfs        Matrix.bfs with parents
  msbfs      Matrix.msbfs: many searches at once
  pagerank   Matrix.pagerank

Inputs are drawn on the GPU from the seed: R-MAT graphs (a, b, c = .57, .19,
.19, relabelled at random, no self loops, no repeated entries), 7-point grids,
x with uniform distinct indices in random order and values in (0, 1].
"""
from __future__ import annotations

import math

import torch

import paper_1610_07902_amd as spv

SEMIRINGS = {"plus_times": spv.PLUS_TIMES_F32, "min_select2nd": spv.MIN_SELECT2ND_I32, "or_and": spv.OR_AND_BOOL}


# ------------------------------------------------------------------- cases
def _mul(name, graph, m, n, ef, f, semiring="plus_times", masked=False, det=False):
    return {"name": name, "kind": "mul", "graph": graph, "m": m, "n": n, "ef": ef, "f": f, "semiring": semiring,
            "masked": masked, "det": det}


def listed():
    s20, s22 = 1 << 20, 1 << 22
    return [
        # The smallest call: a local update on a 64^3 grid (a wave front's
        # tip, one step of a local solver).  Launches and the read-back count.
        _mul("mul_grid_tiny", "grid", 64 ** 3, 64 ** 3, 64, 50),
        # A small rectangular graph with odd sizes, 1 % of the columns.
        _mul("mul_rect_small", "rect", 49999, 70001, 12, 700, "min_select2nd"),
        # The headline workload: scale 22, symmetrised, 1 % of the columns.
        _mul("mul_s22_1pct", "sym", s22, s22, 16, s22 // 100),
        # A dense frontier on the same graph.
        _mul("mul_s22_10pct", "sym", s22, s22, 16, s22 // 10),
        # One masked reachability step: 3 % of a million-vertex graph's
        # columns, half the rows already visited.
        _mul("mul_masked_or", "sym", 1000003, 1000003, 16, 30011, "or_and", masked=True),
        # Reproducible sums: the deterministic mode at 2 %.
        _mul("mul_det", "sym", s20, s20, 16, s20 // 50, det=True),
        # A masked update w<mask> += A x as a GraphBLAS program writes it.
        {"name": "graphblas_add", "kind": "graphblas", "graph": "sym", "m": s20, "n": s20, "ef": 16, "f": s20 // 100,
         "mask_share": 0.5, "w_share": 0.125, "complement": False, "replace": False},
        # 64 vectors of log-uniform sizes against one graph.
        {"name": "batch_s20_64", "kind": "batch", "graph": "sym", "m": s20, "n": s20, "ef": 16, "nbatch": 64,
         "f_max": s20 // 4},
        # Direction-optimising search of a scale-22 graph, levels and parents.
        {"name": "bfs_s22", "kind": "bfs", "graph": "sym", "m": s22, "n": s22, "ef": 16, "how": "direction"},
        # Search of a high-diameter grid (766 levels), levels and parents.
        {"name": "bfs_grid256", "kind": "bfs", "graph": "grid", "m": 256 ** 3, "n": 256 ** 3, "ef": 256,
         "how": "persistent"},
        # 64 searches at once.
        {"name": "msbfs_s20_64", "kind": "msbfs", "graph": "sym", "m": s20, "n": s20, "ef": 16, "nsrc": 64},
        # PageRank to the default tolerance on a graph of odd size.
        {"name": "pagerank", "kind": "pagerank", "graph": "sym", "m": 1500007, "n": 1500007, "ef": 16, "tol": 1e-6},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mul", "mul", "mul", "mul", "mul", "mul", "graphblas", "batch", "bfs", "bfs", "msbfs",
                       "pagerank"])
    if kind == "mul":
        graph = rng.choice(["sym", "sym", "sym", "rect", "grid"])
        if graph == "grid":
            side = rng.randint(40, 200)
            m = n = side ** 3
            ef = side
        else:
            n = _log_uniform(rng, 50000, 1 << 22)
            m = n if graph == "sym" else _log_uniform(rng, 50000, 1 << 21)
            ef = rng.randint(6, 16)
        f = max(1, min(n // 10, _log_uniform(rng, max(8, n * 2e-4), n * 0.1)))
        semiring = rng.choice(["plus_times", "plus_times", "min_select2nd", "or_and"])
        return {"kind": "mul", "graph": graph, "m": m, "n": n, "ef": ef, "f": f, "semiring": semiring,
                "masked": rng.random() < 0.25, "det": semiring == "plus_times" and rng.random() < 0.25}
    if kind == "graphblas":
        n = _log_uniform(rng, 100000, 1 << 22)
        return {"kind": kind, "graph": "sym", "m": n, "n": n, "ef": rng.randint(8, 16),
                "f": _log_uniform(rng, max(8, n * 1e-3), n * 0.1), "mask_share": round(rng.uniform(0.1, 0.9), 3),
                "w_share": round(rng.uniform(0.01, 0.3), 3), "complement": rng.random() < 0.5,
                "replace": rng.random() < 0.5}
    if kind == "batch":
        n = _log_uniform(rng, 100000, 1 << 20)
        return {"kind": kind, "graph": "sym", "m": n, "n": n, "ef": rng.randint(8, 16), "nbatch": rng.randint(5, 64),
                "f_max": n // rng.randint(4, 40)}
    if kind == "bfs":
        if rng.random() < 0.4:
            side = rng.randint(60, 256)
            return {"kind": kind, "graph": "grid", "m": side ** 3, "n": side ** 3, "ef": side, "how": "persistent"}
        n = _log_uniform(rng, 200000, 1 << 22)
        return {"kind": kind, "graph": "sym", "m": n, "n": n, "ef": rng.randint(8, 16),
                "how": rng.choice(["direction", "direction", "push"])}
    if kind == "msbfs":
        n = _log_uniform(rng, 100000, 1 << 20)
        return {"kind": kind, "graph": "sym", "m": n, "n": n, "ef": rng.randint(8, 16), "nsrc": rng.randint(8, 64)}
    n = _log_uniform(rng, 100000, 1500007)
    return {"kind": kind, "graph": "sym", "m": n, "n": n, "ef": rng.randint(8, 16),
            "tol": rng.choice([1e-6, 1e-6, 1e-5, 1e-4])}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _unit(g, k):
    """k floats in (0, 1], multiples of 2^-24."""
    return (torch.randint(0, 1 << 24, (k,), generator=g, device="cuda", dtype=torch.int32) + 1).float() * 2.0 ** -24


def _rmat(g, m, n, ef, symmetric):
    """CSC arrays (colptr, rowids) of an R-MAT graph cut to m x n."""
    k = max(1, math.ceil(math.log2(max(m, n))))
    tuples = ef * n
    row = torch.zeros(tuples, dtype=torch.int32, device="cuda")
    col = torch.zeros(tuples, dtype=torch.int32, device="cuda")
    for _ in range(k):
        u = torch.rand(tuples, generator=g, device="cuda")
        row.mul_(2).add_(u >= 0.76)
        col.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    keep = (row < m) & (col < n)
    row, col = row[keep], col[keep]
    pr = torch.randperm(m, generator=g, device="cuda")
    row = pr[row.long()]
    col = (pr if symmetric else torch.randperm(n, generator=g, device="cuda"))[col.long()]
    if symmetric:
        row, col = torch.cat([row, col]), torch.cat([col, row])
    keep = row != col
    key = (col[keep] * m + row[keep]).sort()[0]
    key = key[torch.cat([torch.ones(1, dtype=torch.bool, device="cuda"), key[1:] != key[:-1]])]
    col = torch.div(key, m, rounding_mode="floor")
    rowids = (key - col * m).int()
    colptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    colptr[1:] = torch.bincount(col, minlength=n).cumsum(0)
    return colptr.int(), rowids


def _grid(side):
    """CSC arrays of the 7-point stencil (diagonal included) on a side^3 grid."""
    n = side ** 3
    v = torch.arange(n, device="cuda", dtype=torch.int32)
    x, y, z = v % side, (v // side) % side, v // (side * side)
    ok = torch.stack([z > 0, y > 0, x > 0, v >= 0, x < side - 1, y < side - 1, z < side - 1], 1)
    step = torch.tensor([-side * side, -side, -1, 0, 1, side, side * side], device="cuda", dtype=torch.int32)
    rowids = (v[:, None] + step)[ok]
    colptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    colptr[1:] = ok.sum(1).cumsum(0)
    return colptr.int(), rowids


def _graph(case, g):
    if case["graph"] == "grid":
        return _grid(case["ef"])
    return _rmat(g, case["m"], case["n"], case["ef"], case["graph"] == "sym")


def _list(g, n, f):
    return torch.randperm(n, generator=g, device="cuda")[:f].int()


def _bitmap(member):
    """A 0/1 vector as a bitmap of 32-bit words."""
    pad = (-member.numel()) % 32
    bits = torch.cat([member.long(), torch.zeros(pad, dtype=torch.int64, device="cuda")]).view(-1, 32)
    words = (bits << torch.arange(32, device="cuda")).sum(1)
    return (words - ((words >> 31) << 32)).int()


def _inputs(case, seed):
    """Everything a case's call reads, as plain tensors."""
    g = _gen(seed)
    m, n, kind = case["m"], case["n"], case["kind"]
    colptr, rowids = _graph(case, g)
    d = {"colptr": colptr, "rowids": rowids, "values": None}
    if kind in ("mul", "graphblas", "batch"):
        d["values"] = _unit(g, rowids.numel())
    if kind == "mul":
        f = case["f"]
        d["x_idx"] = _list(g, n, f)
        if case["semiring"] == "plus_times":
            d["x_val"] = _unit(g, f)
        elif case["semiring"] == "min_select2nd":
            d["x_val"] = torch.randint(0, 1 << 30, (f,), generator=g, device="cuda", dtype=torch.int32)
        else:
            d["x_val"] = (torch.rand(f, generator=g, device="cuda") < 0.9).to(torch.uint8)
        d["member"] = (torch.rand(m, generator=g, device="cuda") < 0.5) if case["masked"] else None
    elif kind == "graphblas":
        d["x_idx"], d["x_val"] = _list(g, n, case["f"]), _unit(g, case["f"])
        d["mask_idx"] = _list(g, m, max(1, int(m * case["mask_share"])))
        d["w_idx"] = _list(g, m, max(1, int(m * case["w_share"]))).sort()[0]
        d["w_val"] = _unit(g, d["w_idx"].numel())
    elif kind == "batch":
        u = torch.rand(case["nbatch"], generator=g, device="cuda", dtype=torch.float64)
        sizes = [max(1, int(round(v))) for v in torch.exp(u * math.log(case["f_max"])).tolist()]
        d["x_idx"] = torch.cat([_list(g, n, f) for f in sizes])
        d["x_val"] = _unit(g, sum(sizes))
        d["x_off"] = torch.tensor([0] + sizes, dtype=torch.int64).cumsum(0).cuda()
    elif kind in ("bfs", "msbfs"):
        k = case.get("nsrc", 1)
        if case["graph"] == "grid":
            d["roots"] = [0]    # a corner: the longest search the grid has
            if int(seed) % 2:
                d["roots"] = [n - 1]
        else:       # ends of random edges, so not isolated
            at = torch.randint(0, rowids.numel(), (k,), generator=g, device="cuda")
            d["roots"] = rowids[at].tolist()
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    flags = 0
    if case.get("det"):
        flags |= spv.DETERMINISTIC
    if kind == "msbfs" or case.get("how") == "direction":
        flags |= spv.SYMMETRIC
    A = spv.Matrix(case["m"], case["n"], d.pop("colptr"), d.pop("rowids"), d.pop("values"), flags=flags)
    d["case"], d["A"] = case, A
    # y in buffers that the program keeps, as long as the longest result
    room = case["m"] * case.get("nbatch", 1)
    value = {"min_select2nd": torch.int32, "or_and": torch.uint8}.get(case.get("semiring"), torch.float32)
    if kind in ("mul", "graphblas", "batch"):
        d["y_idx"] = torch.zeros(room, dtype=torch.int32, device="cuda")
        d["y_val"] = torch.zeros(room, dtype=value, device="cuda")
    if kind == "mul":
        member = d.pop("member")
        d["mask"] = None if member is None else _bitmap(member)
    elif kind == "batch":
        d["y_off"] = torch.zeros(case["nbatch"] + 1, dtype=torch.int64, device="cuda")
        A.attach_batch(case["nbatch"], d["x_idx"].numel(), case["nbatch"] * A.nnz)
    elif kind == "msbfs":
        A.attach_batch(case["nsrc"], msbfs=True)
    return d


def run(state):
    case, A = state["case"], state["A"]
    kind = case["kind"]
    if kind == "mul":
        out = (state["y_idx"], state["y_val"])
        _, _, nnz = A.spmspv(state["x_idx"], state["x_val"], SEMIRINGS[case["semiring"]], sorted_output=True,
                             flags=spv.DETERMINISTIC if case["det"] else 0, out=out, mask=state["mask"])
        return [*out, nnz]
    if kind == "graphblas":
        mflags = (spv.MASK_COMPLEMENT if case["complement"] else 0) | (spv.MASK_REPLACE if case["replace"] else 0)
        y_idx, y_val = state["y_idx"], state["y_val"]
        nnz = spv.spmspv_run_graphblas(A.handle, spv.PLUS_TIMES_F32, 0, state["x_idx"].numel(), state["x_idx"],
                                       state["x_val"], state["mask_idx"], None, state["mask_idx"].numel(), mflags,
                                       spv.ACCUM_ADD, state["w_idx"], state["w_val"], state["w_idx"].numel(), y_idx,
                                       y_val, y_idx.numel())
        return [y_idx, y_val, nnz]
    if kind == "batch":
        out = (state["y_off"], state["y_idx"], state["y_val"])
        A.spmspv_batch(state["x_off"], state["x_idx"], state["x_val"], out=out)
        return list(out)
    if kind == "bfs":
        flags = {"direction": spv.DIRECTION_OPT | spv.USE_GRAPH, "push": spv.USE_GRAPH,
                 "persistent": spv.PERSISTENT}[case["how"]]
        level, parent, levels = A.bfs(state["roots"][0], flags=flags)
        return [level, parent, levels]
    if kind == "msbfs":
        level, parent, levels = A.msbfs(state["roots"], flags=spv.DIRECTION_OPT)
        return [level, parent, levels]
    rank, iters = A.pagerank(tol=case["tol"])
    return [rank, iters]


# -------------------------------------------------------- 64-bit references
def _products(d, x_idx):
    """Entry numbers of the columns x selects and the x position of each."""
    start = d["colptr"][x_idx.long()].long()
    length = d["colptr"][x_idx.long() + 1].long() - start
    pos = torch.repeat_interleave(torch.arange(x_idx.numel(), device="cuda"), length)
    first = length.cumsum(0) - length
    entry = torch.arange(pos.numel(), device="cuda") - first[pos] + start[pos]
    return entry, pos


def _times(d, m, x_idx, x_val):
    """(A x in 64 bits, touched rows)."""
    entry, pos = _products(d, x_idx)
    rows = d["rowids"][entry].long()
    t = torch.zeros(m, dtype=torch.float64, device="cuda")
    t.index_add_(0, rows, d["values"][entry].double() * x_val.double()[pos])
    seen = torch.zeros(m, dtype=torch.bool, device="cuda")
    seen[rows] = True
    return t, seen


def _whole(room, rows, values):
    """The list (rows, values) at the front of zeroed buffers."""
    y_idx = torch.zeros(room, dtype=torch.int64, device="cuda")
    y_val = torch.zeros(room, dtype=torch.float64, device="cuda")
    y_idx[:rows.numel()], y_val[:rows.numel()] = rows, values
    return [y_idx, y_val]


def exact(case, seed):
    kind, m, n = case["kind"], case["m"], case["n"]
    if kind in ("bfs", "msbfs") or (kind == "mul" and case["semiring"] != "plus_times"):
        return None
    d = _inputs(case, seed)
    if kind == "mul":
        t, seen = _times(d, m, d["x_idx"], d["x_val"])
        if d["member"] is not None:
            seen &= ~d["member"]
        rows = seen.nonzero().flatten()
        return _whole(m, rows, t[rows]) + [rows.numel()]
    if kind == "graphblas":
        t, seen = _times(d, m, d["x_idx"], d["x_val"])
        inside = torch.zeros(m, dtype=torch.bool, device="cuda")
        inside[d["mask_idx"].long()] = True
        if case["complement"]:
            inside = ~inside
        w = torch.zeros(m, dtype=torch.float64, device="cuda")
        w[d["w_idx"].long()] = d["w_val"].double()
        has_w = torch.zeros(m, dtype=torch.bool, device="cuda")
        has_w[d["w_idx"].long()] = True
        seen &= inside
        out = seen | (has_w & inside if case["replace"] else has_w)
        rows = out.nonzero().flatten()
        return _whole(m, rows, (w + torch.where(seen, t, torch.zeros_like(t)))[rows]) + [rows.numel()]
    if kind == "batch":
        off = d["x_off"].tolist()
        idx, val, starts = [], [], [0]
        for b in range(case["nbatch"]):
            t, seen = _times(d, m, d["x_idx"][off[b]:off[b + 1]], d["x_val"][off[b]:off[b + 1]])
            rows = seen.nonzero().flatten()
            idx.append(rows)
            val.append(t[rows])
            starts.append(starts[-1] + rows.numel())
        return [torch.tensor(starts)] + _whole(m * case["nbatch"], torch.cat(idx), torch.cat(val))
    # PageRank in its delta form, vertices leaving once converged
    degree = (d["colptr"][1:] - d["colptr"][:-1]).long()
    rows, cols = d["rowids"].long(), torch.repeat_interleave(torch.arange(n, device="cuda"), degree)
    damping = 0.85
    rank = torch.zeros(n, dtype=torch.float64, device="cuda")
    delta = torch.full((n,), (1 - damping) / n, dtype=torch.float64, device="cuda")
    active = torch.ones(n, dtype=torch.bool, device="cuda")
    share = damping / degree.clamp(min=1).double()
    for it in range(101):
        rank += delta
        send = torch.where(active & (degree > 0), delta * share, torch.zeros_like(delta))
        if it == 100 or not bool((active & (degree > 0)).any()):
            break
        delta = torch.zeros_like(delta).index_add_(0, rows, send[cols])
        active = delta > case["tol"] * rank
    return [rank, it]


def work(case):
    """Bytes and operations of one pass: the inputs it selects read once, its outputs written once."""
    kind, m, n = case["kind"], case["m"], case["n"]
    d = _inputs(case, 1)
    nnz = d["rowids"].numel()
    if kind in ("mul", "graphblas"):
        f = d["x_idx"].numel()
        entry, _ = _products(d, d["x_idx"])
        seen = torch.zeros(m, dtype=torch.bool, device="cuda")
        seen[d["rowids"][entry].long()] = True
        products, touched = entry.numel(), int(seen.sum())
        per = 8 if case.get("semiring", "plus_times") == "plus_times" else 4
        nbytes = f * 16 + products * per + touched * 8
        if kind == "graphblas":
            nbytes += 4 * d["mask_idx"].numel() + 8 * d["w_idx"].numel()
        elif case["masked"]:
            nbytes += m // 8
        return {"bytes": nbytes, "flops": 2 * products}
    if kind == "batch":
        entry, _ = _products(d, d["x_idx"])
        off, touched = d["x_off"].tolist(), 0
        for b in range(case["nbatch"]):
            at, _ = _products(d, d["x_idx"][off[b]:off[b + 1]])
            seen = torch.zeros(m, dtype=torch.bool, device="cuda")
            seen[d["rowids"][at].long()] = True
            touched += int(seen.sum())
        return {"bytes": d["x_idx"].numel() * 16 + entry.numel() * 8 + touched * 8, "flops": 2 * entry.numel()}
    if kind in ("bfs", "msbfs"):
        # levels and parents, and per vertex its column bounds and one edge
        # that shows its parent (a search that has to walk the edges forward
        # reads all of them)
        edges = nnz if case.get("how") in ("push", "persistent") else n
        return {"bytes": 8 * n * case.get("nsrc", 1) + 4 * n + 4 * edges, "flops": 0}
    iters = math.ceil(math.log(case["tol"]) / math.log(0.85))
    return {"bytes": iters * (4 * nnz + 4 * n + 12 * n), "flops": 2 * iters * nnz}
