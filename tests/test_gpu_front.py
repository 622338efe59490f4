"""Frontier rounds (symmetric graphs of short rows): the oracle's colours,
colour count and rounds bit for bit, entered after every early round
(WL_FRONT), on graphs whose rounds mark few members of a class (one wave),
many (a workgroup), all of them, and more than a workgroup takes (the round
goes back to a full one), under a round cap, with labels and weights, with
rows of every length that qualifies, in F_p and in Z/2^64."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_02603_amd as wl
from paper_2607_02603_amd import inputs
from weight_seeds import G, M, unmix

pytestmark = pytest.mark.gpu


def _csr(n, u, v):
    return inputs.csr_from_edges(n, np.asarray(u), np.asarray(v))


def _check(g, wt=None, init=None, seed=0, rp64=False, ring=False, max_rounds=0):
    ref, kr, rr, _, st = oracle.stable_coloring(g.row_ptr, g.col, wt, init, seed, max_rounds,
                                                q=64 if ring else 0)
    rp = np.asarray(g.row_ptr, np.uint64)
    dg = wl.Graph.from_numpy(g.n, rp if rp64 else rp.astype(np.uint32), g.col, wt,
                             device="cuda", symmetric=True)
    it = None if init is None else torch.from_numpy(
        np.asarray(init, np.uint32).view(np.int32)).cuda()
    print(f"n={g.n} nnz={g.nnz} colours={kr} rounds={rr}", flush=True)
    with wl.precision(wl.WL_PRECISION_RING64 if ring else wl.WL_PRECISION_FP):
        c, k, r = wl.wl_stable_coloring(dg, it, seed, max_rounds, allow_max_rounds=True)
    assert (k, r) == (kr, rr)
    assert np.array_equal(c.cpu().numpy().view(np.uint32), ref)


def _tree(n, seed, window):
    rng = np.random.default_rng(seed)
    i = np.arange(1, n)
    return _csr(n, i, i - 1 - (rng.random(n - 1) * np.minimum(i, window)).astype(np.int64))


def _spider(legs, length):
    """'legs' equal paths from one centre through a binary tree (short rows)."""
    u, v = [], []
    ids = list(range(legs))
    nxt = legs
    while len(ids) > 1:
        new = []
        for a in range(0, len(ids), 2):
            for x in ids[a:a + 2]:
                u.append(x)
                v.append(nxt)
            new.append(nxt)
            nxt += 1
        ids = new
    base = nxt
    for t in range(length):
        for x in range(legs):
            u.append(x if t == 0 else base + (t - 1) * legs + x)
            v.append(base + t * legs + x)
    return _csr(base + legs * length, u, v)


GRAPHS = {
    "grid": lambda: inputs.grid_graph(70, 90),
    "grid_thin": lambda: inputs.grid_graph(2, 4000),
    "path": lambda: inputs.grid_graph(1, 5001),
    "tree": lambda: _tree(6000, 1, 3),
    "tree_bushy": lambda: _tree(9000, 2, 40),
    "spider": lambda: _spider(128, 70),
    "er": lambda: inputs.er_graph(6000, 9000, seed=4),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("front", [0, 1, 2, 5])
def test_entered_after_every_early_round(monkeypatch, name, front):
    monkeypatch.setenv("WL_FRONT", str(front))
    _check(GRAPHS[name](), seed=front, rp64=front == 2)


@pytest.mark.parametrize("name", ["grid", "tree", "spider"])
def test_default_entry_weights_labels_ring(name):
    g = GRAPHS[name]()
    _check(g, seed=1)
    _check(g, seed=1, ring=True)
    _check(g, init=(np.arange(g.n) % 997 == 0), seed=2)
    # symmetric weights, zeros among them: a value of the unordered pair
    u = np.repeat(np.arange(g.n), np.diff(np.asarray(g.row_ptr, np.int64)))
    lo, hi = np.minimum(u, g.col), np.maximum(u, g.col)
    wt = ((lo * 7 + hi * 7) % 5 % 3).astype(np.uint32)
    _check(g, wt, seed=3)
    _check(g, wt, seed=3, ring=True)  # weighted: full rounds in Z/2^64


@pytest.mark.parametrize("cap", [3, 4, 9, 17, 34])
def test_round_cap(monkeypatch, cap):
    monkeypatch.setenv("WL_FRONT", "2")
    _check(inputs.grid_graph(70, 90), seed=1, max_rounds=cap)


@pytest.mark.parametrize("legs,length", [(63, 100), (64, 100), (65, 100), (2000, 12), (8192, 6),
                                         (8300, 6)])
def test_marked_members_of_one_class(monkeypatch, legs, length):
    # every round marks all members of classes of 'legs' nodes: one wave up
    # to 64, a workgroup up to 8192, and beyond that the full rounds
    monkeypatch.setenv("WL_FRONT", "1")
    _check(_spider(legs, length), seed=legs)


@pytest.mark.parametrize("deg", [4, 5, 8, 9, 16, 63, 64, 65])
def test_row_lengths(monkeypatch, deg):
    # a path whose every 50th node carries pendant nodes up to degree 'deg'
    monkeypatch.setenv("WL_FRONT", "1")
    n0 = 3000
    hubs = np.arange(0, n0, 50)
    pend = deg - 2
    u = np.concatenate([np.arange(n0 - 1), np.repeat(hubs, pend)])
    v = np.concatenate([np.arange(1, n0), n0 + np.arange(hubs.size * pend)])
    g = _csr(n0 + hubs.size * pend + 2000, u, v)  # and isolated nodes
    _check(g, seed=deg)
    _check(g, seed=deg, ring=True)


def test_wide_grid_goes_back_to_full_rounds(monkeypatch):
    # 2 x (300 + 9000) outline: more than 8192 members are marked at once
    monkeypatch.setenv("WL_FRONT", "2")
    _check(inputs.grid_graph(12, 9000), seed=5)


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("rnd", [2, 3, 4, 11, 20])
def test_degenerate_value_in_a_round(monkeypatch, rnd, ring):
    # a seed that makes one colour's value 0 (in Z/2^64: 2^60 or 0) in a round
    # before, at and after the change to frontier rounds: the round is left to
    # the full rounds
    monkeypatch.setenv("WL_FRONT", "2")
    g = inputs.grid_graph(70, 90)
    for b in (0, 1, 5):
        for w in (0, 1 << 60) if ring else (0,):
            _check(g, seed=_seed_for_weight(w, rnd, b), ring=ring)


def _seed_for_weight(w, rnd, b):
    key = (unmix(w) - (b + 1) * G) & M
    s1 = (unmix(key) - (rnd + 1) * G) & M
    return (unmix(s1) - G) & M


def test_full_round_after_device_driven_rounds(monkeypatch):
    # The positions that the one-colour round records hold for the round after
    # it only.  With that round device-driven, a later host-driven one (the
    # full round before frontier rounds) must not take its image from them.
    # Rows of 17 to 64 entries: no other round keeps the positions up to date.
    monkeypatch.setenv("WL_HOST_ROUNDS", "1")
    monkeypatch.setenv("WL_FRONT", "4")
    monkeypatch.setenv("WL_PB", "force")
    n0, pend = 9000, 18  # enough nodes for the one-colour round's tables
    hubs = np.arange(0, n0, 50)
    u = np.concatenate([np.arange(n0 - 1), np.repeat(hubs, pend)])
    v = np.concatenate([np.arange(1, n0), n0 + np.arange(hubs.size * pend)])
    g = _csr(n0 + hubs.size * pend, u, v)
    _check(g, seed=3)
    _check(g, seed=3, ring=True)


def _strip(width, layers, deg):
    """Layers of 'width' nodes; node j of a layer has the deg / 2 neighbours
    j .. j + deg / 2 - 1 (mod width) in the next one."""
    j = np.arange(width)
    u, v = [], []
    for t in range(layers - 1):
        for d in range(deg // 2):
            u.append(t * width + j)
            v.append((t + 1) * width + (j + d) % width)
    return _csr(width * layers, np.concatenate(u), np.concatenate(v))


def test_image_of_a_later_full_round_is_chosen_by_its_own_rows():
    # Labels of their own on the first layer: a layer of 8400 nodes becomes
    # singletons in every round, more at once than a workgroup splits, so both
    # attempts at frontier rounds (from round 16 on, and 17 rounds later) go
    # back at once.  The propagation-blocking image serves rounds 0 to 7 and the
    # full round of the first attempt, while at least half of the entries feed
    # rows that need one; by the second attempt fewer do.
    width, layers = 8400, 50
    g = _strip(width, layers, 16)
    assert g.nnz >= 1 << 22
    init = np.zeros(g.n, np.uint32)
    init[:width] = 1 + np.arange(width)
    wl.wl_stats_enable(wl.WL_STATS_TIME)
    try:
        _check(g, init=init, seed=1)
        st = wl.wl_stats_get()
    finally:
        wl.wl_stats_enable(0)
    assert st["rounds"] > 40
    assert st["pb"]["launches"] == 9


@pytest.mark.parametrize("front", [None, 2])
@pytest.mark.parametrize("legs,length", [(255, 40), (256, 40), (257, 40), (2000, 40), (4096, 30),
                                         (8192, 30)])
def test_many_images_in_one_class(monkeypatch, legs, length, front):
    # Leg ends with labels of their own (the first six share one): every round
    # marks about 'legs' members of the class that the labels have not reached
    # yet, with as many images and one more (from the tree's side), and from
    # the meeting of the two sides on all members of a class.  256 images and
    # 257, from which on the members are sorted; 8192 is the largest class.
    if front:
        monkeypatch.setenv("WL_FRONT", str(front))
    g = _spider(legs, length)
    ends = np.arange(g.n - legs, g.n)
    init = np.zeros(g.n, np.uint32)
    init[ends] = 1 + np.maximum(np.arange(legs) - 5, 0)
    _check(g, init=init, seed=legs)
    _check(g, init=init, seed=legs, ring=True)
    # weights of 0 across the middle of every seventh leg: members that are
    # marked and have the image of the unmarked ones
    u = np.repeat(np.arange(g.n), np.diff(np.asarray(g.row_ptr, np.int64)))
    lo, hi = np.minimum(u, g.col), np.maximum(u, g.col)
    cut = g.n - legs * (length // 2 + 5)  # first node of a layer
    wt = np.where((lo < cut) & (hi >= cut) & ((hi - cut) % 7 == 0), 0, 1).astype(np.uint32)
    _check(g, wt, init=init, seed=legs)


@pytest.mark.parametrize("species,copies,length", [(17, 40, 60), (300, 33, 24)])
def test_many_classes_for_a_workgroup(monkeypatch, species, copies, length):
    # Copies of labelled paths: every round marks 2 * copies > 64 members in a
    # class of every label, in more classes than the workgroups set aside for
    # such classes, and than there are workgroups.
    monkeypatch.setenv("WL_FRONT", "1")
    m = species * copies
    ids = np.random.default_rng(species).permutation(m * length).reshape(m, length)
    g = _csr(m * length, ids[:, :-1].ravel(), ids[:, 1:].ravel())
    init = np.empty(g.n, np.uint32)
    init[ids] = (np.arange(m) % species)[:, None]
    _check(g, init=init, seed=species)
    _check(g, init=init, seed=species, ring=True)


@pytest.mark.parametrize("front", [None, 1])
@pytest.mark.parametrize("copies", [4096, 4097])
def test_copies_of_a_path(monkeypatch, copies, front):
    # every class has 2 * copies nodes: as many as a workgroup splits, and
    # more, for which the change to frontier rounds is not made
    if front:
        monkeypatch.setenv("WL_FRONT", str(front))
    ids = np.arange(copies * 44).reshape(copies, 44)
    _check(_csr(ids.size, ids[:, :-1].ravel(), ids[:, 1:].ravel()), seed=copies)


@pytest.mark.parametrize("flags", [0, wl.WL_STATS_TIME])
def test_image_launches_count_every_round(flags):
    # timed or not, a call has one image launch for every round that ran
    g = inputs.grid_graph(70, 90)
    wl.wl_stats_enable(flags)
    try:
        _check(g, seed=1)
        st = wl.wl_stats_get()
    finally:
        wl.wl_stats_enable(0)
    assert st["rounds"] > 40
    assert sum(st[kd]["launches"] for kd in ("gather", "pb", "uniform")) == st["rounds"]
