"""Performance cases of libcmg: what a user of the library has it do.

Every case makes seeded graphs on the GPU, calls the public entry points of
``paper_1412_0565_amd.cmg`` as a user's program does, and returns whole
results (eigenvalue, vector, residual; parts and cut).  ``exact`` computes
the same method in 64 bits with plain torch.

A case is a dict of plain values:
  call       noalloc   cmg_fiedler_noalloc: one small graph, nothing allocated
             solve     cmg_setup + cmg_fiedler + cmg_free, arrays on the device
             host      the same as a server does it: numpy arrays in and out,
                       cmg_fiedler_batch of one
             resident  cmg_fiedler on a kept hierarchy
             schedule  the same with the fixed smoothing schedule, replayed as
                       a HIP graph
             batch     cmg_fiedler_batch on several kept hierarchies
             block     cmg_fiedler_block on a kept hierarchy
             bisect    cmg_bisect, arrays on the device
  family     grid2d, grid3d (with sides a, b, c), rgg (mean degree 10),
             chunglu (gamma, deg, cap) of n vertices, each component joined
             to the others by an edge
  weights    unit, int (1..8), real (in [0.5, 1.5))
  values     f64 or f32 (the type of the weight array)
  precision  fp64 or mixed
"""
from __future__ import annotations

import ctypes as C
import math

import numpy as np
import torch

from paper_1412_0565_amd import cmg


# ------------------------------------------------------------------ the cases

def _case(name, call, family, **kw):
    c = {"call": call, "family": family, "weights": "int", "values": "f64", "precision": "fp64"}
    if name:
        c = {"name": name, **c}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one graph of a thousand vertices from a caller that may not allocate
        _case("noalloc grid 32x31", "noalloc", "grid2d", a=32, b=31),
        # a small mesh solved once (the 128 x 128 five-point grid workload)
        _case("solve grid 128x128", "solve", "grid2d", a=128, b=128, weights="unit"),
        # a served request of middle size: host arrays, mixed precision
        _case("host rgg 40k mixed", "host", "rgg", n=40000, precision="mixed"),
        # a served request of the power-law family (exponent 2.5, mean degree 8, cap sqrt(8 n))
        _case("host chunglu 120k", "host", "chunglu", n=120011, gamma=2.5, deg=8.0, cap=980.0),
        # the random geometric graph workload, 1M points, solved once
        _case("solve rgg 1M", "solve", "rgg", n=1000000),
        # the same graph family kept resident and solved again, mixed precision
        _case("resident rgg 300k mixed", "resident", "rgg", n=299993, precision="mixed"),
        # a weighted box of odd sides kept resident: real conductances, FP64 storage throughout
        _case("resident grid 97x101x113 real", "resident", "grid3d", a=97, b=101, c=113, weights="real"),
        # the benchmark: 256^3 seven-point grid, unit weights given as FP32
        _case("solve grid 256^3", "solve", "grid3d", a=256, b=256, c=256, weights="unit", values="f32"),
        # the largest power-law graph: 4M vertices, exponent 2.1, mean degree 16, cap 50000
        _case("solve chunglu 4M", "solve", "chunglu", n=4000000, gamma=2.1, deg=16.0, cap=50000.0, weights="unit",
              values="f32"),
        # a server's packed launch: twelve kept hierarchies of 1k to 60k vertices of the three families
        _case("batch of 12", "batch", "mixed", n=60000, n0=1000, count=12, precision="mixed"),
        # four eigenpairs on a kept hierarchy
        _case("block p=4 rgg 200k", "block", "rgg", n=200000, p=4),
        # recursive bisection of a mesh-like graph into 16 parts
        _case("bisect rgg 60k into 16", "bisect", "rgg", n=60000, depth=4),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["noalloc", "solve", "solve", "host", "host", "resident", "resident", "schedule", "batch",
                       "block", "bisect"])
    if call == "batch":
        n = _log_uniform(rng, 4000, 100000)
        return _case(None, "batch", "mixed", n=n, n0=1000, count=rng.randint(2, 14),
                     precision=rng.choice(["fp64", "mixed"]))
    top = {"noalloc": 30000, "solve": 4000000, "host": 1000000, "resident": 4000000, "schedule": 4000000,
           "block": 300000, "bisect": 100000}[call]
    low = {"solve": 1000, "bisect": 2000, "block": 2000}.get(call, 1000)
    families = ["grid2d", "grid3d", "rgg"] if call in ("block", "bisect") else ["grid2d", "grid3d", "rgg", "chunglu"]
    family = rng.choice(families)
    if family in ("rgg", "chunglu"):
        top = min(top, 1000000)
    n = _log_uniform(rng, low, top)
    kw = {"weights": rng.choice(["unit", "int", "int", "real"]) if call not in ("host", "bisect") else "int",
          "values": rng.choice(["f64", "f64", "f32"]), "precision": rng.choice(["fp64", "fp64", "mixed"])}
    if family == "grid2d":
        r = rng.uniform(0.7, 1.4)
        kw.update(a=max(3, round(math.sqrt(n) * r)), b=max(3, round(math.sqrt(n) / r)))
    elif family == "grid3d":
        s, t = rng.uniform(0.8, 1.25), rng.uniform(0.8, 1.25)
        kw.update(a=max(3, round(n ** (1 / 3) * s)), b=max(3, round(n ** (1 / 3) * t)),
                  c=max(3, round(n ** (1 / 3) / (s * t))))
    else:
        kw["n"] = n
    if family == "chunglu":
        kw.update(gamma=2.5, deg=8.0, cap=round(math.sqrt(8.0 * n), 3))
    if call == "block":
        kw.update(p=rng.randint(1, 4), precision="fp64")
    if call == "bisect":
        kw.update(depth=rng.randint(1, 5), precision="fp64", values="f64")
    return _case(None, call, family, **kw)


# ----------------------------------------------------------------- the graphs

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _mix(z):
    """An integer hash of int64 tensors (wrapping arithmetic, logical shifts)."""
    def shr(x, k):
        return (x >> k) & ((1 << (64 - k)) - 1)

    z = (z ^ shr(z, 30)) * -4658895280553007687
    z = (z ^ shr(z, 27)) * -7723592293110705685
    return z ^ shr(z, 31)


def _weights(kind, rows, col, seed):
    """Symmetric weights of the entries: a hash of (smaller end, larger end, seed)."""
    if kind == "unit":
        return torch.ones(col.numel(), dtype=torch.float64, device=col.device)
    a, b = torch.minimum(rows, col).long(), torch.maximum(rows, col).long()
    fold = (seed * 0x9E3779B1 + 12345) & ((1 << 64) - 1)
    h = _mix(_mix((a << 32) | b) ^ (fold - (1 << 64) if fold >> 63 else fold))
    if kind == "int":
        return ((h >> 20) & 7).double() + 1.0
    return 0.5 + ((h >> 12) & ((1 << 40) - 1)).double() * 2.0 ** -40


def _grid(dims):
    """Grid graph CSR: vertex id with the last side running fastest."""
    dev = _device()
    n = math.prod(dims)
    idx = torch.arange(n, dtype=torch.int32, device=dev)
    strides = [math.prod(dims[k + 1:]) for k in range(len(dims))]
    lower, upper = [], []
    for d, s in zip(dims, strides):
        x = (idx // s) % d
        lower.append((-s, x > 0))
        upper.append((s, x < d - 1))
    offs = lower + upper[::-1]  # ascending neighbour indices
    keep = torch.stack([m for _, m in offs], 1)
    cols = torch.stack([idx + o for o, _ in offs], 1)
    rp = torch.zeros(n + 1, dtype=torch.int32, device=dev)
    rp[1:] = keep.sum(1).cumsum(0).int()
    return n, rp, cols[keep]


def _components(n, rows, cols):
    """Smallest vertex of each vertex's component."""
    lab = torch.arange(n, device=cols.device)
    while True:
        best = lab.clone()
        best.scatter_reduce_(0, lab[rows], lab[cols], "amin")  # every root hooks to its smallest neighbour
        while True:
            nxt = best[best]
            if torch.equal(nxt, best):
                break
            best = nxt
        new = best[lab]
        if torch.equal(new, lab):
            return lab
        lab = new


def _connected(n, rows, cols, join):
    """CSR of the entries (rows, cols, in order) with every component but
    vertex 0's joined by one edge from its smallest vertex v to the vertex
    join(v) < v, so that the graph is connected and keeps n vertices."""
    lab = _components(n, rows, cols)
    v = torch.nonzero(lab == torch.arange(n, device=cols.device)).reshape(-1)[1:]
    if v.numel():
        to = join(v)
        key = torch.sort(torch.cat([rows * n + cols, v * n + to, to * n + v])).values
        rows, cols = key // n, key % n
    rp = torch.zeros(n + 1, dtype=torch.int32, device=cols.device)
    rp[1:] = torch.bincount(rows, minlength=n).cumsum(0).int()
    return n, rp, cols.int()


def _rgg(n, seed, deg=10.0):
    """Random geometric graph in the unit square, vertices in cell order."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed * 7919 + 17)
    r = math.sqrt(deg / (math.pi * n))
    x, y = torch.rand(2, n, dtype=torch.float64, device=dev, generator=g)
    m = max(1, int(1.0 / r))
    cx, cy = (x * m).long().clamp_(max=m - 1), (y * m).long().clamp_(max=m - 1)
    cell, order = torch.sort(cy * m + cx, stable=True)
    x, y, cx, cy = x[order], y[order], cx[order], cy[order]
    first = torch.zeros(m * m + 1, dtype=torch.int64, device=dev)
    first[1:] = torch.bincount(cell, minlength=m * m).cumsum(0)
    lo, hi = [], []
    for dy in (-1, 0, 1):  # the three cells of a row are one range of vertices
        yy = cy + dy
        ok = (yy >= 0) & (yy < m)
        yy = yy.clamp(0, m - 1)
        a = first[yy * m + (cx - 1).clamp(min=0)]
        b = first[yy * m + (cx + 1).clamp(max=m - 1) + 1]
        lo.append(torch.where(ok, a, 0))
        hi.append(torch.where(ok, b, 0))
    lo, hi = torch.stack(lo, 1).reshape(-1), torch.stack(hi, 1).reshape(-1)
    cnt = hi - lo
    start = cnt.cumsum(0) - cnt
    seg = torch.repeat_interleave(torch.arange(cnt.numel(), device=dev), cnt)
    cand = torch.arange(seg.numel(), device=dev) - start[seg] + lo[seg]
    row = seg // 3
    keep = (row != cand) & ((x[row] - x[cand]) ** 2 + (y[row] - y[cand]) ** 2 < r * r)
    return _connected(n, row[keep], cand[keep], lambda v: v - 1)


def _chung_lu(n, gamma, deg, cap, seed):
    """Chung-Lu graph: n deg / 2 endpoint pairs drawn by expected degree, hubs first."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed * 104729 + 29)
    base = torch.arange(1, n + 1, dtype=torch.float64, device=dev) ** (-1.0 / (gamma - 1.0))
    lo, hi = 0.0, 1.0
    while float((hi * base).clamp(max=cap).mean()) < deg and hi < 1e9:
        hi *= 2.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if float((mid * base).clamp(max=cap).mean()) < deg else (lo, mid)
    cdf = (hi * base).clamp(max=cap).cumsum(0)
    cdf = cdf / cdf[-1].clone()
    u = torch.rand(2, int(n * deg / 2), dtype=torch.float64, device=dev, generator=g)
    e = torch.searchsorted(cdf, u, right=True).clamp_(max=n - 1)
    e = e[:, e[0] != e[1]]
    key = torch.unique(torch.minimum(e[0], e[1]) * n + torch.maximum(e[0], e[1]))
    del e, u
    a, b = key // n, key % n
    key = torch.sort(torch.cat([a * n + b, b * n + a])).values

    def join(v):  # by expected degree among the vertices before v
        r = torch.rand(v.numel(), dtype=torch.float64, device=dev, generator=g)
        return torch.minimum(torch.searchsorted(cdf, r * cdf[v - 1]), v - 1)

    return _connected(n, key // n, key % n, join)


def _graph(case, seed):
    """(n, row_ptr, col, w) on the device; w in the case's value type."""
    if case["family"] == "grid2d":
        n, rp, col = _grid((case["a"], case["b"]))
    elif case["family"] == "grid3d":
        n, rp, col = _grid((case["a"], case["b"], case["c"]))
    elif case["family"] == "rgg":
        n, rp, col = _rgg(case["n"], seed)
    else:
        n, rp, col = _chung_lu(case["n"], case["gamma"], case["deg"], case["cap"], seed)
    if case["weights"] == "unit":
        w = torch.ones(col.numel(), dtype=torch.float64, device=col.device)
    else:
        rows = torch.repeat_interleave(torch.arange(n, dtype=torch.int32, device=col.device), rp[1:] - rp[:-1])
        w = _weights(case["weights"], rows, col, seed)
    return n, rp, col, w.float() if case["values"] == "f32" else w


def _members(case):
    """The graphs of a batch: sizes spread evenly over their logarithm, the three families in turn."""
    k = case["count"]
    out = []
    for i in range(k):
        n = int(case["n0"] * (case["n"] / case["n0"]) ** ((i + 0.5) / k))
        c = _case(None, "solve", ("grid2d", "rgg", "chunglu")[i % 3], n=n, precision=case["precision"])
        if c["family"] == "grid2d":
            c["a"] = c["b"] = max(3, round(math.sqrt(n)))
        elif c["family"] == "chunglu":
            c.update(gamma=2.5, deg=8.0, cap=round(math.sqrt(8.0 * n), 3))
        out.append(c)
    return out


# -------------------------------------------------------------------- a state

def _hec_seed(seed):
    return (14120565 + 7 * seed) & 0xFFFFFFFF


def _options(case, seed, alloc):
    kw = {"precision": cmg.CMG_MIXED if case["precision"] == "mixed" else cmg.CMG_FP64, "seed": _hec_seed(seed),
          "stream": C.c_void_p(torch.cuda.current_stream().cuda_stream), "allocator": C.pointer(alloc)}
    if case["call"] == "schedule":
        kw.update(fixed_k0=3, fixed_beta=1.6, graph=1)
    return kw


class _Kept:
    """A kept hierarchy, freed with the state that holds it."""

    def __init__(self, g, options):
        self.n = g[0]
        self.handle = cmg.cmg_setup(*g, cmg.cmg_options_default(**options))

    def __del__(self):
        cmg.cmg_free(self.handle)


_ALLOCATOR = None


def _allocator():
    global _ALLOCATOR
    if _ALLOCATOR is None:
        _ALLOCATOR = cmg.torch_allocator()
    return _ALLOCATOR


def _stats():
    st = cmg.cmg_stats()
    st.struct_size = C.sizeof(cmg.cmg_stats)
    return st


def prepare(case, seed):
    alloc = _allocator()
    call = case["call"]
    options = _options(case, seed, alloc)
    state = {"call": call}
    if call == "batch":
        state["kept"] = [_Kept(_graph(c, seed * 64 + i), options) for i, c in enumerate(_members(case))]
        state["x"] = [torch.zeros(k.n, dtype=torch.float64, device="cuda") for k in state["kept"]]
        return state
    g = _graph(case, seed)
    n = g[0]
    if call == "host":
        state["graph"] = (n, *(t.cpu().numpy() for t in g[1:]))
        state["opt"] = cmg.cmg_options_default(**options)
    elif call in ("resident", "schedule", "block"):
        state["kept"] = _Kept(g, options)
        state["p"] = case.get("p", 1)
        state["x"] = torch.zeros(state["p"] * n, dtype=torch.float64, device="cuda")
    else:
        state["graph"] = g
        state["opt"] = cmg.cmg_options_default(**options)
        state["depth"] = case.get("depth", 0)
        state["x"] = torch.zeros(n, dtype=torch.int32 if call == "bisect" else torch.float64, device="cuda")
    return state


def run(state):
    call = state["call"]
    if call == "batch":
        lams, _ = cmg.cmg_fiedler_batch([k.handle for k in state["kept"]], state["x"])
        return {"lambda": np.array(lams), "x": state["x"]}
    if call in ("resident", "schedule"):
        st = _stats()
        lam, _ = cmg.cmg_fiedler(state["kept"].handle, state["x"], st)
        return {"lambda": lam, "x": state["x"], "residual": st.residual}
    if call == "block":
        lams, res, _, _ = cmg.cmg_fiedler_block(state["kept"].handle, state["p"], state["x"])
        return {"lambda": lams, "x": state["x"], "residual": res}
    n, rp, col, w = state["graph"]
    if call == "bisect":
        part, cut = cmg.cmg_bisect(n, rp, col, w, state["depth"], part=state["x"], opt=state["opt"])
        return {"part": part, "cut": cut}
    if call == "noalloc":
        st = _stats()
        lam, _ = cmg.cmg_fiedler_noalloc(n, rp, col, w, state["x"], state["opt"], st)
        return {"lambda": lam, "x": state["x"], "residual": st.residual}
    h = cmg.cmg_setup(n, rp, col, w, state["opt"])
    try:
        if call == "host":
            x = np.zeros(n)
            lams, _ = cmg.cmg_fiedler_batch([h], [x])
            return {"lambda": lams[0], "x": x}
        st = _stats()
        lam, _ = cmg.cmg_fiedler(h, state["x"], st)
    finally:
        cmg.cmg_free(h)
    return {"lambda": lam, "x": state["x"], "residual": st.residual}


# ----------------------------------------------------------------- the demand

def _size(case):
    """(vertices, stored entries) to within the randomness of the family."""
    if case["family"] == "grid2d":
        a, b = case["a"], case["b"]
        return a * b, 2 * (2 * a * b - a - b)
    if case["family"] == "grid3d":
        a, b, c = case["a"], case["b"], case["c"]
        return a * b * c, 2 * (3 * a * b * c - a * b - b * c - a * c)
    if case["family"] == "rgg":
        return case["n"], 10 * case["n"]
    return case["n"], int(0.97 * case["deg"] * case["n"])


def work(case):
    """One pass reads each graph (or the kept hierarchy's finest level) once
    and writes the vectors once; one multiply-add and one subtraction per
    entry for the product with the Laplacian that the residual needs."""
    if case["call"] == "batch":
        parts = [work({**c, "call": "resident"}) for c in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, nnz = _size(case)
    p = case.get("p", 1)
    given = 8 if case["values"] == "f64" else 4
    w = 0 if case["weights"] == "unit" and case["call"] in ("resident", "schedule", "block") else given
    out = 4 * n if case["call"] == "bisect" else 8 * n * p
    return {"bytes": 4 * (n + 1) + nnz * (4 + w) + out, "flops": 3 * nnz * p * max(1, case.get("depth", 1))}


# ------------------------------------------------- the method in plain 64 bits

def _keys(seed, level, n, dev):
    """Visit-order keys (SplitMix64's output function), as signed integers in
    the order of the unsigned ones."""
    v = torch.arange(n, dtype=torch.int64, device=dev)
    return _mix(v ^ (level << 40) ^ seed) ^ (-1 << 63)


def _uniform(seed, n, dev):
    h = _mix(torch.arange(n, dtype=torch.int64, device=dev) ^ ((seed ^ 0x9E3779B97F4A7C15) - (1 << 64)
             if (seed ^ 0x9E3779B97F4A7C15) >= 1 << 63 else seed ^ 0x9E3779B97F4A7C15))
    return ((h >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53


def _segments(t, offsets, how, most=1 << 22):
    """Reduction of t over segments, in pieces that one call can take."""
    k = offsets.numel() - 1
    if k <= most:
        return torch.segment_reduce(t, how, offsets=offsets)
    out = []
    for a in range(0, k, most):
        o = offsets[a:min(a + most, k) + 1]
        out.append(torch.segment_reduce(t[int(o[0]):int(o[-1])], how, offsets=o - o[0]))
    return torch.cat(out)


class _Level:
    def __init__(self, n, rp, col, w):
        self.n, self.rp, self.col, self.w = n, rp.long(), col.long(), w
        self.rows = torch.repeat_interleave(torch.arange(n, device=col.device), self.rp[1:] - self.rp[:-1])
        self.agg = None

    def sums(self, t):
        return _segments(t, self.rp, "sum")

    def laplacian(self, y):
        return self.sums(self.w * (y[self.rows] - y[self.col]))


def _heavy_edge(L, seed, level):
    """Heavy edge coarsening as rounds of locally first candidates, equal to
    the visit in key order; aggregates numbered by their opening vertex."""
    dev, n = L.col.device, L.n
    wmax = _segments(L.w, L.rp, "max")
    cand = torch.where(L.w == wmax[L.rows], L.col, n)
    h = torch.full((n,), n, dtype=torch.int64, device=dev).scatter_reduce_(0, L.rows, cand, "amin")
    key = _keys(seed, level, n, dev)
    ids = torch.arange(n, device=dev)
    opened = torch.full((n,), -1, dtype=torch.int64, device=dev)  # the opening vertex of a matched vertex's pair
    live = ids[key < key[h]]
    last = (1 << 63) - 1
    while live.numel():
        slot = torch.full((n,), last, dtype=torch.int64, device=dev)
        slot.scatter_reduce_(0, live, key[live], "amin")
        slot.scatter_reduce_(0, h[live], key[live], "amin")
        won = live[(slot[live] == key[live]) & (slot[h[live]] == key[live])]
        opened[won] = won
        opened[h[won]] = won
        live = live[(opened[live] < 0) & (opened[h[live]] < 0)]
    root = torch.where(opened >= 0, ids, h)  # the rest follow h to a matched vertex
    while True:
        nxt = root[root]
        if torch.equal(nxt, root):
            break
        root = nxt
    root = opened[root]
    rank = (root == ids).long().cumsum(0) - 1
    return rank[root], int(rank[-1]) + 1


def _hierarchy(n, rp, col, w, seed):
    levels = [_Level(n, rp, col, w.double())]
    while levels[-1].n > 25 and len(levels) < 64:
        L = levels[-1]
        agg, nc = _heavy_edge(L, seed, len(levels) - 1)
        if nc < 2:
            break
        key = agg[L.rows] * nc + agg[L.col]
        off = key // nc != key % nc
        key, order = torch.sort(key[off], stable=True)
        uniq, cnt = torch.unique_consecutive(key, return_counts=True)
        first = torch.zeros(cnt.numel() + 1, dtype=torch.int64, device=col.device)
        first[1:] = cnt.cumsum(0)
        wc = _segments(L.w[off][order], first, "sum")
        rpc = torch.zeros(nc + 1, dtype=torch.int64, device=col.device)
        rpc[1:] = torch.bincount(uniq // nc, minlength=nc).cumsum(0)
        L.agg = agg
        levels.append(_Level(nc, rpc, uniq % nc, wc))
    return levels


def _dense(L):
    A = torch.zeros(L.n, L.n, dtype=torch.float64)
    rows, col, w = L.rows.cpu(), L.col.cpu(), L.w.cpu()
    A[rows, col] = -w
    A += torch.diag(-A.sum(1))
    ev, V = np.linalg.eigh(A.numpy())
    return ev, V, float(torch.linalg.norm(A))


def _deflated(y):
    y = y - y.mean(0)
    return y / y.norm()


def _start(L, seed):
    ev, V, fro = _dense(L)
    n = L.n
    E = V[:, 1:][:, np.abs(ev[1:] - ev[1]) <= 1e-10 * fro]
    z = np.arange(n) - 0.5 * (n - 1)
    y = E @ (E.T @ z)
    if np.linalg.norm(y) < 1e-8 * np.linalg.norm(z):
        y = E @ (E.T @ (_uniform(seed, n, "cpu").numpy() - 0.5))
    return torch.from_numpy(y / np.linalg.norm(y)).to(L.col.device)


def _orthonormal(V):
    cols = []
    for c in range(V.shape[1]):
        v = V[:, c] - V[:, c].mean()
        for u in cols:
            v = v - (u @ v) * u
        cols.append(v / v.norm())
    return torch.stack(cols, 1)


def _rayleigh(L, y):
    d = y[L.rows] - y[L.col]
    lam = 0.5 * float((L.w * d * d).sum()) / float(y @ y)
    return lam, float((L.laplacian(y) - lam * y).norm() / y.norm())


def _fiedler(levels, seed, tol=1e-8, k0=0, beta=0.0):
    J = len(levels) - 1
    L = levels[J]
    if L.n > 128:
        return None  # a collapsed coarsening: the start is not the dense one
    y = _start(L, seed)
    for j in range(J - 1, -1, -1):
        L = levels[j]
        g = 2.0 * float(L.sums(L.w).max())
        y = _deflated(y[L.agg])
        steps = math.ceil(k0 * math.prod([beta] * j)) if k0 else 100000
        for _ in range(steps):
            v, y = y, _deflated(g * y - L.laplacian(y))
            if not k0 and float(y @ v) >= 1.0 - tol:
                break
    y = _deflated(y)
    return (y, *_rayleigh(levels[0], y))


def _block(levels, seed, p, tol=1e-8):
    J = len(levels) - 1
    L = levels[J]
    if L.n > 128 or p > L.n - 1:
        return None
    ev, V, fro = _dense(L)
    E = V[:, 1:][:, ev[1:] <= ev[p] + 1e-10 * fro]
    z = [_uniform(seed ^ ((c + 1) * 0xD1B54A32D192ED03 & (1 << 64) - 1), L.n, "cpu").numpy() - 0.5 for c in range(p)]
    Y = _orthonormal(torch.from_numpy(np.stack([E @ (E.T @ v) for v in z], 1)).to(L.col.device))
    for j in range(J - 1, -1, -1):
        L = levels[j]
        g = 2.0 * float(L.sums(L.w).max())
        Y = _orthonormal(Y[L.agg])
        for _ in range(100000):
            V = Y
            Y = _orthonormal(torch.stack([g * V[:, c] - L.laplacian(V[:, c].contiguous()) for c in range(p)], 1))
            if float((Y * V).sum(0).min()) >= 1.0 - tol:
                break
    Y = _orthonormal(Y)
    rr = [_rayleigh(levels[0], Y[:, c].contiguous()) for c in range(p)]
    return Y.T.reshape(-1).contiguous(), np.array([r[0] for r in rr]), np.array([r[1] for r in rr])


def exact(case, seed):
    call = case["call"]
    hs = _hec_seed(seed)
    if call == "bisect":
        return None  # whole numbers
    if call == "batch":
        got = [_fiedler(_hierarchy(*_graph(c, seed * 64 + i), hs), hs) for i, c in enumerate(_members(case))]
        if any(g is None for g in got):
            return None
        return {"lambda": np.array([g[1] for g in got]), "x": [g[0] for g in got]}
    levels = _hierarchy(*_graph(case, seed), hs)
    if call == "block":
        got = _block(levels, hs, case["p"])
    elif call == "schedule":
        got = _fiedler(levels, hs, k0=3, beta=1.6)
    else:
        got = _fiedler(levels, hs)
    if got is None:
        return None
    out = {"lambda": got[1], "x": got[0], "residual": got[2]}
    if call == "host":
        del out["residual"]
    return out
