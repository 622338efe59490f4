"""GPU parity: the HIP path (through the C ABI) against the CPU oracle.

Bit-exact: colour ids, colour count and round count (Algorithm 1 with the
readings of the oracle).  Partition equality with classic refinement.
Inputs are seeded and synthetic; no oracle input comes from the GPU.
"""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2607_02603_amd as wl
from oracle import bruteforce as bf
from paper_2607_02603_amd import inputs

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _dev_graph(rp, col, wt=None, rp64=False):
    n = len(rp) - 1
    rp = np.asarray(rp, dtype=np.uint64 if rp64 else np.uint64)
    if not rp64:
        assert rp[-1] < 2**32
        rp = rp.astype(np.uint32)
    return wl.Graph.from_numpy(n, rp, col, wt, device="cuda")


def _gpu_stable(g, init=None, seed=0, max_rounds=0):
    init_t = None
    if init is not None:
        init_t = torch.from_numpy(np.asarray(init, np.uint32).view(np.int32)).cuda()
    c, k, r = wl.wl_stable_coloring(g, init_t, seed, max_rounds)
    torch.cuda.synchronize()
    return c.cpu().numpy().view(np.uint32), k, r


def _check_exact(rp, col, wt=None, init=None, seed=0, rp64=False, classic=True):
    g = _dev_graph(rp, col, wt, rp64)
    cg, kg, rg = _gpu_stable(g, init, seed)
    co, ko, ro, _, st = oracle.stable_coloring(rp, col, wt, init, seed)
    assert st == 0
    assert (kg, rg) == (ko, ro)
    assert np.array_equal(cg, co)
    if classic:
        cb = oracle.classic_coloring(rp, col, wt, init)[0]
        assert np.array_equal(oracle.first_occurrence(cg)[0],
                              oracle.first_occurrence(cb)[0])
    return cg, kg, rg


# ---------------------------------------------------------------------------
# small graphs, every shape of row and class
# ---------------------------------------------------------------------------

@pytest.mark.usefixtures("in_core_path")
@pytest.mark.parametrize("trial", range(24))
def test_random_small_graphs(trial):
    rng = random.Random(trial)
    n = rng.randint(1, 300)
    directed = trial % 2 == 1
    weighted = trial % 3 == 2
    edges = []
    for _ in range(rng.randint(0, 4 * n)):
        u, v = rng.randrange(n), rng.randrange(n)
        if trial % 5 != 0 and u == v:
            continue
        edges.append((u, v))
    rp, col = bf.to_csr(n, edges, directed=directed)
    wt = None
    if weighted:
        wt = np.array([rng.choice([1, 2, 3, 0xFFFFFFFF]) for _ in range(col.size)],
                      np.uint32)
    init = None
    if trial % 4 == 3:
        init = np.array([rng.choice([7, 100, 2**31 + 5]) for _ in range(n)], np.uint32)
    _say(f"trial {trial} n={n} m={col.size}")
    _check_exact(rp, col, wt, init, seed=trial, rp64=trial % 2 == 0)


@pytest.mark.usefixtures("in_core_path")
@pytest.mark.parametrize("n", [1, 2, 3, 17])
def test_edgeless(n):
    rp = np.zeros(n + 1, np.uint64)
    col = np.zeros(0, np.uint32)
    cg, kg, rg = _check_exact(rp, col)
    assert kg == 1 and rg == 1


def test_empty_graph():
    g = _dev_graph(np.zeros(1, np.uint64), np.zeros(0, np.uint32))
    c, k, r = wl.wl_stable_coloring(g)
    assert (k, r) == (0, 0)


@pytest.mark.usefixtures("in_core_path")
def test_path_and_grid_closed_forms():
    for n in (2, 5, 12, 101):
        rp, col = bf.to_csr(n, [(i, i + 1) for i in range(n - 1)])
        _, k, r = _check_exact(rp, col)
        assert k == (n + 1) // 2 == r
    g = inputs.grid_graph(40)
    _, k, r = _check_exact(g.row_ptr, g.col)
    assert (k, r) == (210, 20)


def test_heavy_rows_and_large_classes():
    # star with 10000 leaves (a heavy row of 10000 > 4096 entries and one
    # class of 10000 leaves), plus 3000 pendant paths of random lengths hung
    # on hubs of different degrees (many distinct images in big classes).
    rng = random.Random(11)
    edges = [(0, i) for i in range(1, 10001)]
    n = 10001
    hubs = []
    for h in range(40):
        hub = n
        n += 1
        hubs.append(hub)
        for _ in range(h * 50 + 3):
            edges.append((hub, n))
            n += 1
    for _ in range(3000):
        a = rng.choice(hubs)
        ln = rng.randint(1, 4)
        prev = a
        for _ in range(ln):
            edges.append((prev, n))
            prev = n
            n += 1
    rp, col = bf.to_csr(n, edges)
    _check_exact(rp, col, seed=3)
    _check_exact(rp, col, seed=4, rp64=True)


def test_msd_passes_many_distinct_in_one_class():
    # 20000 leaves each attached to its own hub; hub degrees all distinct up
    # to 200: in round 1 the leaf class (> 2048 nodes) splits by hub degree.
    edges = []
    n = 0
    leaves = []
    for h in range(200):
        hub = n
        n += 1
        for _ in range(h + 1):
            edges.append((hub, n))
            leaves.append(n)
            n += 1
    rp, col = bf.to_csr(n, edges)
    _check_exact(rp, col, seed=5)


def test_initial_colours_large_labels():
    g = inputs.er_graph(5000, 12000, seed=7)
    rng = np.random.default_rng(0)
    init = rng.integers(0, 2**32, size=g.n, dtype=np.uint64).astype(np.uint32)
    init[::3] = 4000000000
    _check_exact(g.row_ptr, g.col, init=init, seed=2)


@pytest.mark.usefixtures("in_core_path")
def test_weighted_quotient_like_graph():
    rng = random.Random(8)
    n = 3000
    edges = [(rng.randrange(n), rng.randrange(n)) for _ in range(20000)]
    rp, col = bf.to_csr(n, edges, directed=True)
    wt = np.array([rng.randint(1, 2**32 - 1) for _ in range(col.size)], np.uint32)
    _check_exact(rp, col, wt, seed=9)


# ---------------------------------------------------------------------------
# wl_refine_round: every round of the oracle's trace, inputs from the oracle
# ---------------------------------------------------------------------------

def test_refine_round_each_round_bit_exact():
    g = inputs.rmat(13, 8, seed=1)
    dg = _dev_graph(g.row_ptr, g.col)
    c, k = oracle.canonicalize(None, g.n)
    r = 0
    while True:
        cin = torch.from_numpy(c.view(np.int32)).cuda()
        cout, kg = wl.wl_refine_round(dg, cin, k, 17, r)
        c2, k2, _ = oracle.refine_round(g.row_ptr, g.col, None, c, k, 17, r)
        assert kg == k2
        assert np.array_equal(cout.cpu().numpy().view(np.uint32), c2)
        # in place (color_out aliases color_in)
        cin2 = cin.clone()
        _, kg2 = wl.wl_refine_round(dg, cin2, k, 17, r, color_out=cin2)
        assert kg2 == k2 and np.array_equal(cin2.cpu().numpy().view(np.uint32), c2)
        r += 1
        if k2 == k:
            break
        c, k = c2, k2
    assert r >= 3


def test_refine_round_sparse_colour_ids():
    # colours need not be dense: ids drawn from [0, k_in) with gaps
    g = inputs.er_graph(4000, 9000, seed=2)
    rng = np.random.default_rng(3)
    c = (rng.integers(0, 50, size=g.n) * 7).astype(np.uint32)
    dg = _dev_graph(g.row_ptr, g.col)
    cin = torch.from_numpy(c.view(np.int32)).cuda()
    cout, kg = wl.wl_refine_round(dg, cin, 400, 5, 3)
    c2, k2, _ = oracle.refine_round(g.row_ptr, g.col, None, c, 400, 5, 3)
    assert kg == k2 and np.array_equal(cout.cpu().numpy().view(np.uint32), c2)


@pytest.mark.parametrize("n", [1, 2, 255, 1023, 1024, 1025, 2049, 9001])
@pytest.mark.parametrize("shape", ["one", "half", "discrete"])
def test_refine_round_class_sizes(n, shape):
    # one class, one class with half of the nodes beside classes of one node
    # each, and only those: the grouping by colour takes tiles of 1024 nodes
    g = inputs.csr_from_edges(n, np.arange(n - 1), np.arange(1, n))
    rng = np.random.default_rng(n)
    c = rng.permutation(n).astype(np.uint32)
    if shape != "discrete":
        c[rng.random(n) < (2 if shape == "one" else 0.5)] = n // 2
    _say(f"n={n} {shape}")
    dg = _dev_graph(g.row_ptr, g.col)
    cin = torch.from_numpy(c.view(np.int32)).cuda()
    cout, kg = wl.wl_refine_round(dg, cin, n, 11, 1)
    c2, k2, _ = oracle.refine_round(g.row_ptr, g.col, None, c, n, 11, 1)
    assert kg == k2 and np.array_equal(cout.cpu().numpy().view(np.uint32), c2)


@pytest.mark.parametrize("step", [1, 63, 64, 65, 2048, 4096])
@pytest.mark.parametrize("k", [16, 1000, 9001])
def test_refine_round_colour_spacing(k, step):
    # colours that the tiles' hash tables keep in a row, and colours whose
    # distance is that of a group of slots, of a table, or beside them
    n = 70001
    g = inputs.csr_from_edges(n, np.arange(n - 1), np.arange(1, n))
    c = (np.arange(n) % k * step % n).astype(np.uint32)
    _say(f"k={k} step={step}")
    dg = _dev_graph(g.row_ptr, g.col)
    cout, kg = wl.wl_refine_round(dg, torch.from_numpy(c.view(np.int32)).cuda(), n, 11, 1)
    c2, k2, _ = oracle.refine_round(g.row_ptr, g.col, None, c, n, 11, 1)
    assert kg == k2 and np.array_equal(cout.cpu().numpy().view(np.uint32), c2)


# ---------------------------------------------------------------------------
# configurations
# ---------------------------------------------------------------------------

def test_config_er():
    g = inputs.er_graph()
    _say("ER 20000/80000")
    _, k, r = _check_exact(g.row_ptr, g.col)
    assert k == 19993 and r == 4


def test_config_grid_1024():
    g = inputs.grid_graph(1024)
    _say("grid 1024")
    cg, kg, rg = _check_exact(g.row_ptr, g.col, classic=False)
    assert (kg, rg) == (131328, 512)
    assert bf.partition_of(cg) == bf.partition_of(bf.grid_orbits(1024, 1024))


# ---------------------------------------------------------------------------
# errors
# ---------------------------------------------------------------------------

@pytest.mark.usefixtures("in_core_path")
def test_errors():
    g = inputs.er_graph(1000, 3000, seed=1)
    dg = _dev_graph(g.row_ptr, g.col)
    need = wl.wl_workspace_size(dg)
    small = wl.workspace(need - 1024)
    with pytest.raises(wl.WlError) as e:
        wl.wl_stable_coloring(dg, ws=small)
    assert e.value.code == wl.WL_EBUDGET
    c, k, r = wl.wl_stable_coloring(dg, max_rounds=2, allow_max_rounds=True)
    assert r == 2
    with pytest.raises(wl.WlError) as e:
        wl.wl_stable_coloring(dg, max_rounds=2)
    assert e.value.code == wl.WL_EMAXROUNDS
    bad = torch.full((g.n,), 9, dtype=torch.int32, device="cuda")
    with pytest.raises(wl.WlError) as e:
        wl.wl_refine_round(dg, bad, 5, 0, 0)
    assert e.value.code == wl.WL_EINVAL
    # WL_VALIDATE=1: a column index out of range is reported, not used
    col = g.col.copy()
    col[17] = g.n + 5
    bg = _dev_graph(g.row_ptr, col)
    import os
    os.environ["WL_VALIDATE"] = "1"
    try:
        with pytest.raises(wl.WlError) as e:
            wl.wl_stable_coloring(bg)
        assert e.value.code == wl.WL_EINVAL
        c, k, r = wl.wl_stable_coloring(dg)  # a valid graph still passes
    finally:
        del os.environ["WL_VALIDATE"]
