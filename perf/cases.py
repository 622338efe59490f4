"""The library's measured cases: what users of the 1-WL stable colouring run.

Every case is one call of a public entry point on a graph that a program
already holds (a device CSR, or a host CSR for the out-of-core entry points),
with the workspace such a program keeps between calls.  The graphs are the
families of the repository's own benchmark and tests (Erdos-Renyi, grid,
Chung-Lu, R-MAT, directed weighted web-like graphs, unions of small labelled
graphs), made on the GPU from the seed; the seed also picks the random values
of the colouring itself.  Colour ids are whole numbers and must agree exactly.

    listed()             the fixed cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, workspace and output buffer
    run(state)           one call
    work(case)           bytes and additions no implementation can avoid
    tolerance(case)      "exact": ids, counts and rounds are integers
    exact(case, seed)    the same result from numpy, for the cases it can do
"""
import math

import numpy as np
import torch

import paper_2607_02603_amd as wl
from paper_2607_02603_amd import inputs

DEV = "cuda:0"
P61 = (1 << 61) - 1


def listed():
    return [
        # one small graph per call, without a workspace: a serving loop, or a
        # data set walked graph by graph; launches and waits decide
        {"name": "er_small_noalloc", "kind": "er", "n": 1500, "m": 6000,
         "call": "noalloc", "ring": False},
        # the repository's first configuration: a sparse random graph
        {"name": "er_20k", "kind": "er", "n": 20000, "m": 80000,
         "call": "stable", "ring": False},
        # a data set of small labelled graphs taken as one disjoint union, as
        # an expressiveness analysis of graph networks does; odd sizes
        {"name": "molecules_union", "kind": "molecules", "graphs": 9001,
         "call": "stable", "ring": False},
        # a mesh: 512 short rounds, the per-round overhead
        {"name": "grid_1024", "kind": "grid", "a": 1024, "b": 1024,
         "call": "stable", "ring": False},
        # a power-law graph of a few million nodes (social network)
        {"name": "chunglu_4m", "kind": "chunglu", "n": 4000000, "samples": 64000000,
         "call": "stable", "ring": False},
        # directed, weighted, labelled, not symmetric: a web-like graph whose
        # rows are gathered
        {"name": "web_20", "kind": "web", "scale": 20, "factor": 16, "pad": 77,
         "call": "stable", "ring": False},
        # the paper's own arithmetic Z/2^64 on a skewed graph of medium size
        {"name": "rmat_20_ring", "kind": "rmat", "scale": 20, "factor": 16, "pad": 0,
         "call": "stable", "ring": True},
        # the headline: 4.2e9 entries in HBM, 64-bit row pointers
        {"name": "rmat_27", "kind": "rmat", "scale": 27, "factor": 16, "pad": 0,
         "call": "stable", "ring": False},
        # a program that drives the rounds itself: one round from a colouring
        # with many classes
        {"name": "round_22", "kind": "rmat", "scale": 22, "factor": 16, "pad": 1001,
         "call": "round", "ring": False},
        # a colouring with its exact certificate, which makes the randomized
        # result certain
        {"name": "verify_22", "kind": "rmat", "scale": 22, "factor": 16, "pad": 0,
         "call": "verify", "ring": False},
        # edge arrays in page-locked host memory, streamed through the device
        {"name": "streamed_22", "kind": "rmat", "scale": 22, "factor": 16, "pad": 0,
         "call": "streamed", "ring": False},
        # Algorithm 2 in four batches, edge arrays in host memory
        {"name": "batched_18", "kind": "rmat", "scale": 18, "factor": 16, "pad": 333,
         "call": "batched", "ring": False, "batches": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["er", "er", "molecules", "grid", "chunglu", "rmat", "rmat", "web",
                       "round", "verify", "streamed", "batched"])
    ring = rng.random() < 0.25
    if kind == "er":
        n = _log(rng, 100, 300000)
        call = rng.choice(["stable", "noalloc"])
        return {"kind": "er", "n": n, "m": int(n * rng.uniform(0.6, 8.0)), "call": call,
                "ring": ring}
    if kind == "molecules":
        return {"kind": "molecules", "graphs": _log(rng, 3, 30000), "call": "stable",
                "ring": ring}
    if kind == "grid":
        return {"kind": "grid", "a": _log(rng, 3, 900), "b": _log(rng, 3, 900),
                "call": "stable", "ring": ring}
    if kind == "chunglu":
        n = _log(rng, 2000, 4000000)
        return {"kind": "chunglu", "n": n, "samples": int(n * rng.uniform(2.0, 16.0)),
                "call": "stable", "ring": ring}
    scale = rng.randint(10, 24)
    if kind in ("streamed", "batched", "web"):
        scale = min(scale, {"streamed": 22, "batched": 18, "web": 20}[kind])
    case = {"kind": "web" if kind == "web" else "rmat", "scale": scale,
            "factor": rng.choice([8, 16]), "pad": rng.randint(0, 3000),
            "call": kind if kind in ("round", "verify", "streamed", "batched") else "stable",
            "ring": ring}
    if kind == "batched":
        case["batches"] = rng.randint(1, 5)
    return case


# ---------------------------------------------------------------------------
# Graphs
# ---------------------------------------------------------------------------

def _csr(n, u, v, gen, weighted=False, symmetric=True):
    """CSR of the entries (u, v) (both directions when symmetric), sorted,
    without duplicates and self-loops; row pointers int32."""
    keep = u != v
    u, v = u[keep], v[keep]
    keys = (u << 32) | v
    if symmetric:
        keys = torch.cat([keys, (v << 32) | u])
    keys = torch.unique(keys)
    cnt = torch.bincount(keys >> 32, minlength=n)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=keys.device)
    rp[1:] = torch.cumsum(cnt, 0)
    col = (keys & 0xFFFFFFFF).to(torch.int32)
    wt = None
    if weighted:
        # small counts with a heavy tail, as link multiplicities have
        x = torch.rand(col.numel(), device=keys.device, generator=gen)
        wt = (1.0 / (x * 0.999 + 0.001)).to(torch.int32)
    return rp.to(torch.int32), col, wt


def _padded(rp, pad):
    if not pad:
        return rp
    return torch.cat([rp, rp[-1:].expand(pad)])


def _graph(case, seed):
    """(Graph on the device, labels or None)."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "er":
        n, m = case["n"], case["m"]
        u = torch.randint(0, n, (m,), device=DEV, generator=gen)
        v = torch.randint(0, n, (m,), device=DEV, generator=gen)
        rp, col, _ = _csr(n, u, v, gen)
        return wl.Graph(n, rp, col, symmetric=True), None
    if kind == "molecules":
        # chains with branches and rings of 8 to 40 atoms, five atom labels;
        # four or five copies of every molecule, numbered in random order
        g = case["graphs"]
        t = max(1, g // 4)
        size = 8 + torch.arange(t, device=DEV) * 7 % 33
        back = torch.randint(1, 4, (t, 40), device=DEV, generator=gen)
        ring = torch.rand(t, 40, device=DEV, generator=gen) < 0.15
        label = (torch.rand(t, 40, device=DEV, generator=gen) ** 3 * 5).to(torch.int32)
        pick = torch.randperm(g, device=DEV, generator=gen) % t
        sz = size[pick]
        start = torch.cumsum(sz, 0) - sz
        n = int(sz.sum())
        mol = torch.repeat_interleave(torch.arange(g, device=DEV), sz)
        at = torch.arange(n, device=DEV) - start[mol]
        tm = pick[mol]
        ids = torch.arange(n, device=DEV)
        b = torch.minimum(back[tm, at], at)
        r5 = ring[tm, at] & (at >= 5)
        u = torch.cat([ids, ids[r5]])
        v = torch.cat([ids - b, ids[r5] - 5])
        rp, col, _ = _csr(n, u, v, gen)
        return wl.Graph(n, rp, col, symmetric=True), label[tm, at].contiguous()
    if kind == "grid":
        # row-major ids, as a mesh is stored, counted from a random node on
        a, b = case["a"], case["b"]
        n = a * b
        off = int(torch.randint(0, n, (1,), device=DEV, generator=gen))
        ids = torch.arange(n, device=DEV).reshape(a, b)
        u = torch.cat([ids[:, :-1].reshape(-1), ids[:-1].reshape(-1)])
        v = torch.cat([ids[:, 1:].reshape(-1), ids[1:].reshape(-1)])
        rp, col, _ = _csr(n, (u + off) % n, (v + off) % n, gen)
        return wl.Graph(n, rp, col, symmetric=True), None
    if kind == "chunglu":
        g = inputs.chung_lu(case["n"], case["samples"], seed=seed, device=DEV)
        return wl.Graph(g.n, g.row_ptr.to(torch.int32), g.col, symmetric=True), None
    if kind == "rmat":
        g = inputs.rmat(case["scale"], case["factor"], seed=seed, device=DEV)
        rp = g.row_ptr if g.nnz >= 1 << 31 else g.row_ptr.to(torch.int32)
        return wl.Graph(g.n + case["pad"], _padded(rp, case["pad"]), g.col,
                        symmetric=True), None
    # web: R-MAT endpoints drawn level by level, one entry per sample,
    # weights and a few page labels
    scale, n = case["scale"], (1 << case["scale"]) + case["pad"]
    m = case["factor"] << scale
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        x = torch.rand(m, device=DEV, generator=gen)
        u = 2 * u + (x >= 0.76)
        v = 2 * v + (((x >= 0.57) & (x < 0.76)) | (x >= 0.95))
    perm = torch.randperm(n, device=DEV, generator=gen)
    rp, col, wt = _csr(n, perm[u], perm[v], gen, weighted=True, symmetric=False)
    label = (torch.rand(n, device=DEV, generator=gen) ** 4 * 7).to(torch.int32)
    return wl.Graph(n, rp, col, wt), label


def _host(t):
    return None if t is None else t.cpu().pin_memory()


def prepare(case, seed):
    g, label = _graph(case, seed)
    s = {"call": case["call"], "g": g, "label": label, "seed": seed * 1000003 + 17,
         "q": wl.WL_PRECISION_RING64 if case["ring"] else wl.WL_PRECISION_FP}
    if case["call"] in ("stable", "noalloc", "round", "verify"):
        s["out"] = torch.empty(g.n, dtype=torch.int32, device=DEV)
    if case["call"] in ("stable", "round", "verify"):
        s["ws"] = wl.workspace(wl.wl_workspace_size(g), g.device)
    if case["call"] == "round":
        # many classes that the round splits further: a node's degree with the
        # degree of its first neighbour, as dense ids
        s["color"], s["k"] = _start_colors(g)
    elif case["call"] == "verify":
        s["ws2"] = wl.workspace(wl.wl_verify_workspace_size(g), g.device)
    elif case["call"] in ("streamed", "batched"):
        h = wl.Graph(g.n, _host(g.row_ptr), _host(g.col_idx), _host(g.weight))
        s["g"], s["label"] = h, _host(label)
        if case["call"] == "streamed":
            s["ws"] = wl.workspace(wl.wl_streamed_workspace_size(h), DEV)
        else:
            s["cap"] = max(1, -(-h.nnz // case["batches"]))
            s["ws"] = wl.workspace(wl.wl_batched_workspace_size(h, s["cap"]), DEV)
    return s


def _start_colors(g):
    rp = g.row_ptr.to(torch.int64)
    deg = rp[1:] - rp[:-1]
    first = torch.full((g.n,), -1, dtype=torch.int64, device=DEV)
    some = deg > 0
    first[some] = deg[g.col_idx[rp[:-1][some]].to(torch.int64)]
    key, color = torch.unique(deg * g.n + first + 1, return_inverse=True)
    return color.to(torch.int32), int(key.numel())


def run(state):
    s = state
    with wl.precision(s["q"]):
        if s["call"] == "stable":
            return wl.wl_stable_coloring(s["g"], s["label"], s["seed"], color_out=s["out"],
                                         ws=s["ws"])
        if s["call"] == "noalloc":
            return wl.wl_stable_coloring_noalloc(s["g"], s["label"], s["seed"],
                                                 color_out=s["out"])
        if s["call"] == "round":
            return wl.wl_refine_round(s["g"], s["color"], s["k"], s["seed"], 1,
                                      color_out=s["out"], ws=s["ws"])
        if s["call"] == "verify":
            c, k, rounds = wl.wl_stable_coloring(s["g"], s["label"], s["seed"],
                                                 color_out=s["out"], ws=s["ws"])
            return c, k, rounds, int(wl.wl_verify_stable(s["g"], c, k, ws=s["ws2"]))
        if s["call"] == "streamed":
            return wl.wl_stable_coloring_streamed(s["g"], s["label"], s["seed"], ws=s["ws"])
        c, k, rounds, outer, coarsest = wl.wl_stable_coloring_batched(
            s["g"], s["label"], s["seed"], s["cap"], ws=s["ws"])
        return c, k, rounds, outer, int(coarsest)


# ---------------------------------------------------------------------------
# Work, tolerance, reference
# ---------------------------------------------------------------------------

def work(case):
    """Each input read once and each output written once; one addition per
    entry, which one image of the graph takes.  Entry counts of the random
    families are the expected ones (samples less duplicates and loops)."""
    kind = case["kind"]
    rp = 4
    if kind == "er":
        n, nnz = case["n"], 2 * case["m"]
    elif kind == "molecules":
        n = 24 * case["graphs"]
        nnz = int(2.2 * n)
    elif kind == "grid":
        n = case["a"] * case["b"]
        nnz = 4 * n - 2 * (case["a"] + case["b"])
    elif kind == "chunglu":
        n, nnz = case["n"], int(1.6 * case["samples"])
    else:
        n = (1 << case["scale"]) + case["pad"]
        per = 1 if kind == "web" else 2
        lost = 0.07 * 2.0 ** ((20 - case["scale"]) * 0.25)
        nnz = int(per * (case["factor"] << case["scale"]) * max(0.3, 1 - lost))
        rp = 8 if nnz >= 1 << 31 else 4
    b = rp * (n + 1) + 4 * nnz
    if kind in ("molecules", "web"):
        b += 4 * n                       # labels
    if kind == "web":
        b += 4 * nnz                     # weights
    if case["call"] == "round":
        b += 4 * n                       # the colouring handed in
    b += 4 * n
    return {"bytes": b, "flops": nnz}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """Algorithm 1 in numpy for the in-core calls on graphs of up to a few
    million entries and few rounds: the image in exact integers, the new
    colour of a node the rank of its pair (colour, image)."""
    if case["call"] not in ("stable", "noalloc") or case["kind"] == "grid":
        return None
    if work(case)["flops"] > 4000000:
        return None
    g, label = _graph(case, seed)
    rp = g.row_ptr.cpu().numpy().astype(np.int64)
    col = g.col_idx.cpu().numpy().astype(np.int64)
    wt = None if g.weight is None else g.weight.cpu().numpy().astype(np.uint64)
    c = np.zeros(g.n, dtype=np.int64)
    if label is not None:
        c = np.unique(label.cpu().numpy(), return_inverse=True)[1].astype(np.int64)
    k, rounds = int(c.max()) + 1, 0
    while True:
        z = _image(rp, col, wt, _values(seed * 1000003 + 17, rounds, k, case["ring"])[c],
                   case["ring"])
        order = np.lexsort((z, c))
        new = np.ones(g.n, dtype=np.int64)
        new[1:] = (c[order][1:] != c[order][:-1]) | (z[order][1:] != z[order][:-1])
        rank = np.cumsum(new) - 1
        c = np.empty_like(c)
        c[order] = rank
        rounds += 1
        k, before = int(rank[-1]) + 1, k
        if k == before:
            return torch.from_numpy(c.astype(np.int32)), k, rounds


def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _fold(v):
    t = (v & np.uint64(P61)) + (v >> np.uint64(61))
    return np.where(t >= P61, t - np.uint64(P61), t)


def _values(seed, rnd, k, ring):
    with np.errstate(over="ignore"):
        gamma = np.uint64(0x9E3779B97F4A7C15)
        s = _mix(np.array([seed], dtype=np.uint64) + gamma)
        key = _mix(s + np.uint64(rnd + 1) * gamma)
        w = _mix(key + np.arange(1, k + 1, dtype=np.uint64) * gamma)
    return w if ring else _fold(w)


def _image(rp, col, wt, x, ring):
    """Row sums of wt * x[col], mod 2^64 or mod 2^61 - 1.  In F_p the values
    are summed as two 31-bit halves, whose products with a weight below 2^11
    leave room for 2^22 entries of a row."""
    def rows(v):
        s = np.concatenate([np.zeros(1, np.uint64), np.cumsum(v, dtype=np.uint64)])
        return s[rp[1:]] - s[rp[:-1]]      # exact: wraps cancel
    v = x[col]
    w = np.uint64(1) if wt is None else wt
    with np.errstate(over="ignore"):
        if ring:
            return rows(v * w)
        lo = rows((v & np.uint64(0x7FFFFFFF)) * w)
        hi = _fold(rows((v >> np.uint64(31)) * w))
        # hi * 2^31 mod p: the top 31 bits of hi wrap round to the bottom
        t = ((hi & np.uint64((1 << 30) - 1)) << np.uint64(31)) + (hi >> np.uint64(30))
        return _fold(_fold(t) + _fold(lo))
