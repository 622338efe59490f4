"""The one-workgroup path of the in-core colouring (graphs of at most 4096
nodes and 2^17 entries): bit for bit the oracle's result, and the general
path's (WL_SMALL=0), at the edges of its bounds, of its row kinds (one
thread, 16 lanes, a wave; columns in LDS or in memory) and of its sort."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_02603_amd as wl
from paper_2607_02603_amd import inputs

pytestmark = pytest.mark.gpu


def _dev(rp, col, wt=None, rp64=False):
    rp = np.asarray(rp, np.uint64)
    return wl.Graph.from_numpy(len(rp) - 1, rp if rp64 else rp.astype(np.uint32), col, wt,
                               device="cuda")


def _csr(n, u, v, directed=False):
    """Multigraph CSR (duplicates and loops kept)."""
    u, v = np.asarray(u, np.int64), np.asarray(v, np.int64)
    if not directed:
        u, v = np.concatenate([u, v]), np.concatenate([v, u])
    o = np.argsort(u, kind="stable")
    rp = np.zeros(n + 1, np.uint64)
    rp[1:] = np.cumsum(np.bincount(u, minlength=n))
    return rp, v[o].astype(np.uint32)


def _check(monkeypatch, rp, col, wt=None, init=None, seed=0, rp64=False, ring=False):
    q = wl.WL_PRECISION_RING64 if ring else wl.WL_PRECISION_FP
    ref, kr, rr, _, st = oracle.stable_coloring(rp, col, wt, init, seed, q=64 if ring else 0)
    assert st == 0
    g = _dev(rp, col, wt, rp64)
    it = None if init is None else torch.from_numpy(
        np.asarray(init, np.uint32).view(np.int32)).cuda()
    print(f"n={g.n} nnz={g.nnz} weighted={wt is not None} ring={ring}", flush=True)
    with wl.precision(q):
        got = [wl.wl_stable_coloring(g, it, seed), wl.wl_stable_coloring_noalloc(g, it, seed)]
        monkeypatch.setenv("WL_SMALL", "0")
        got.append(wl.wl_stable_coloring(g, it, seed))
        monkeypatch.delenv("WL_SMALL")
    for c, k, r in got:
        assert (k, r) == (kr, rr)
        assert np.array_equal(c.cpu().numpy().view(np.uint32), ref)


@pytest.mark.parametrize("n", [1, 2, 33, 1023, 1024, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("ring", [False, True])
def test_random_sizes(monkeypatch, n, ring):
    rng = np.random.default_rng(n)
    m = 3 * n
    rp, col = _csr(n, rng.integers(0, n, m), rng.integers(0, n, m))
    _check(monkeypatch, rp, col, seed=n, ring=ring, rp64=n % 2 == 0)
    wt = rng.choice(np.array([0, 1, 2, 2**31, 2**32 - 1 if not ring else 3], np.uint32), col.size)
    if ring:
        # Theorem 1's bound on the row sums
        wt = np.minimum(wt, 1 << 20).astype(np.uint32)
    _check(monkeypatch, rp, col, wt, rng.integers(0, 5, n), seed=n, ring=ring)


@pytest.mark.parametrize("entries", [16383, 16384, 16385, 131071, 131072, 131073])
def test_entry_bounds(monkeypatch, entries):
    rng = np.random.default_rng(entries)
    n = 3000
    rp, col = _csr(n, (rng.random(entries) ** 3 * n).astype(np.int64),
                   rng.integers(0, n, entries), directed=True)
    assert col.size == entries
    _check(monkeypatch, rp, col, seed=1)


@pytest.mark.parametrize("deg", [31, 32, 33, 511, 512, 513, 4000])
def test_row_kinds(monkeypatch, deg):
    # 40 rows of the same length in one class beside short rows
    rng = np.random.default_rng(deg)
    n = 4096
    u = np.concatenate([np.repeat(np.arange(40), deg), np.arange(40, n)])
    v = rng.integers(0, n, u.size)
    rp, col = _csr(n, u, v, directed=True)
    _check(monkeypatch, rp, col, seed=2)


@pytest.mark.parametrize("kind", ["path", "edgeless", "cycle", "complete", "star", "labels"])
def test_shapes(monkeypatch, kind):
    init = None
    if kind == "path":
        rp, col = _csr(2000, np.arange(1999), np.arange(1, 2000))
    elif kind == "edgeless":
        rp, col = _csr(700, [], [])
    elif kind == "cycle":
        rp, col = _csr(4096, np.arange(4096), (np.arange(4096) + 1) % 4096)
    elif kind == "complete":
        u, v = np.triu_indices(300, 1)
        rp, col = _csr(300, u, v)
    elif kind == "star":
        rp, col = _csr(4096, np.zeros(4095, np.int64), np.arange(1, 4096))
    else:
        rp, col = _csr(4096, np.arange(4095), np.arange(1, 4096))
        init = np.where(np.arange(4096) % 2, 0xFFFFFFFF, np.arange(4096) % 40)
    _check(monkeypatch, rp, col, None, init, seed=3)


def test_many_equal_images_in_one_class():
    # one class of 4096 nodes with 2 to 4096 distinct images, so that a level
    # of the sort meets buckets of every size: node i points at the leaf
    # class of its group
    for groups in (2, 3, 33, 700):
        n = 4096
        half = n // 2
        u = np.arange(half)
        v = half + u % groups
        rp, col = _csr(n, u, v, directed=True)
        init = np.concatenate([np.zeros(half), 1 + np.arange(n - half) % groups])
        ref, kr, rr, _, st = oracle.stable_coloring(rp, col, None, init, 9)
        c, k, r = wl.wl_stable_coloring(
            _dev(rp, col), torch.from_numpy(init.astype(np.int32)).cuda(), 9)
        assert (k, r) == (kr, rr) and st == 0
        assert np.array_equal(c.cpu().numpy().view(np.uint32), ref)


def test_round_cap_and_errors():
    rp, col = _csr(101, np.arange(100), np.arange(1, 101))
    g = _dev(rp, col)
    full = wl.wl_stable_coloring(g)
    assert (full[1], full[2]) == (51, 51)
    for cap in (1, 7, 50):
        c, k, r = wl.wl_stable_coloring(g, max_rounds=cap, allow_max_rounds=True)
        ref, kr, rr, _, st = oracle.stable_coloring(rp, col, max_rounds=cap)
        assert (k, r) == (kr, rr) and r == cap
        assert np.array_equal(c.cpu().numpy().view(np.uint32), ref)
    bad = _dev(rp, np.concatenate([col, col[:1]]))  # one entry more than row_ptr[n]
    with pytest.raises(wl.WlError) as e:
        wl.wl_stable_coloring(bad)
    assert e.value.code == wl.WL_EINVAL
    wt = np.full(col.size, 0xFFFFFFFF, np.uint32)
    with wl.precision(wl.WL_PRECISION_RING64), pytest.raises(wl.WlError) as e:
        wl.wl_stable_coloring(_dev(rp, col, wt))
    assert e.value.code == wl.WL_EOVERFLOW


@pytest.mark.usefixtures("in_core_path")
@pytest.mark.parametrize("deg", [1, 32, 33, 512, 513, 1025, 130000])
def test_row_sum_bound_by_row_length(deg):
    # three rows of the same length whose weights add up to the bound of
    # Z/2^64, 2^32; one more in one of them is refused
    rng = np.random.default_rng(deg)
    n, rows = (70, 1) if deg > 40000 else (1100, 3)
    rp = np.concatenate([[0], deg * np.minimum(np.arange(1, n + 1), rows)]).astype(np.uint64)
    col = rng.integers(0, n, deg * rows).astype(np.uint32)
    wt = np.full(deg * rows, (1 << 32) // deg if deg > 1 else 0xFFFFFFFF, np.uint32)
    for r in range(rows if deg > 1 else 0):
        wt[r * deg + deg // 2] += (1 << 32) - deg * ((1 << 32) // deg)
        assert int(wt[r * deg:(r + 1) * deg].astype(np.uint64).sum()) == 1 << 32
    print(f"rows of {deg}", flush=True)
    with wl.precision(wl.WL_PRECISION_RING64):
        c, k, r = wl.wl_stable_coloring(_dev(rp, col, wt), None, 3)
        ref, kr, rr, _, st = oracle.stable_coloring(rp, col, wt, None, 3, q=oracle.RING64)
        assert st == 0 and (k, r) == (kr, rr)
        assert np.array_equal(c.cpu().numpy().view(np.uint32), ref)
        if deg > 1:
            wt[(rows - 1) * deg + deg - 1] += 1
            with pytest.raises(wl.WlError) as e:
                wl.wl_stable_coloring(_dev(rp, col, wt), None, 3)
            assert e.value.code == wl.WL_EOVERFLOW
