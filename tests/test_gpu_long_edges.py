"""Calls that want only the matching on instances with edges longer than a
window (2,048 pins), which a whole workgroup takes: at the bound, more of them
than a workgroup keeps, alive over several rounds, winners and losers, few
edges spread over short ranges, single instances and batches; every bitmap
equals the oracle's, and no such call takes several times what the rounds over
all live edges take."""
import time

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _instance(n, sizes, w, seed):
    """Edges of the given sizes, each on random distinct vertices."""
    rng = np.random.default_rng(seed)
    edges = [np.sort(rng.choice(n, s, replace=False)) if s < n else np.arange(n) for s in sizes]
    g = synth.from_edge_lists(0, [], [])
    g.n, g.m = n, len(edges)
    g.e_off = np.concatenate([[0], np.cumsum([e.size for e in edges])]).astype(np.int32)
    g.e_pins = np.concatenate(edges).astype(np.int32)
    ids = np.repeat(np.arange(g.m, dtype=np.int32), np.diff(g.e_off))
    order = np.argsort(g.e_pins, kind="stable")
    g.v_edges = ids[order]
    g.v_off = np.concatenate([[0], np.cumsum(np.bincount(g.e_pins, minlength=n))]).astype(np.int32)
    g.w = np.asarray(w, np.uint32)
    return g


def _exact(g, seed=3):
    return oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, seed)[0]


def _check(hgm, g):
    import torch
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    bare = hgm.DeviceHypergraph(g.n, g.m, dg.e_off, dg.e_pins, none, none, dg.w)
    print(f"n={g.n} m={g.m} kappa={g.e_pins.size}", flush=True)
    for d in (dg, bare):
        for _ in range(2):
            bits, _ = hgm.match(d, 3, hgm.make_opts(solo_max_kappa=-1), want_stats=False)
            assert np.array_equal(bits.cpu().numpy().view(np.uint32), _exact(g))


def _mixed(longs, seed, n=60_000, small=20_000, best=None):
    """Small edges and the long ones among them, whose weights are as the small
    ones', or `best` of the range's top."""
    rng = np.random.default_rng(seed)
    sizes = np.concatenate([rng.integers(1, 6, small), longs])
    w = rng.integers(1, 1000, sizes.size)
    if best:
        w[small:] = 1000 + rng.integers(0, best, len(longs))
    at = rng.permutation(sizes.size)
    return _instance(n, sizes[at], w[at], seed + 1)


@pytest.mark.parametrize("best", [None, 1, 50])
@pytest.mark.parametrize("longs", [[2047, 2048, 2049, 4096, 4097], [30_000], [60_000, 59_999],
                                   [2049] * 300, [2500, 9000] * 40])
def test_among_small_edges(hgm, longs, best):
    _check(hgm, _mixed(longs, len(longs) + sum(longs) % 91, best=best))


def test_more_than_a_workgroup_keeps(hgm):
    """Neighbouring ids: 200 long edges in one workgroup's range, nearly disjoint
    ones (alive until they win) and conflicting ones."""
    for n, size in ((900_000, 2100), (30_000, 2500)):
        g = _instance(n, [3] * 3000 + [size] * 200 + [3] * 3000,
                      np.arange(6200) % 700 + 1, 7)
        _check(hgm, g)


@pytest.mark.parametrize("m,lo,hi", [(5, 9000, 30_000), (63, 2000, 2100), (64, 100, 9000),
                                     (257, 900, 1100), (2000, 9, 11), (2000, 300, 700),
                                     (1500, 1, 30), (3, 1, 3)])
def test_few_edges(hgm, m, lo, hi):
    rng = np.random.default_rng(m)
    _check(hgm, _instance(80_000, rng.integers(lo, hi, m), rng.integers(1, 50, m), m + 1))


@pytest.mark.parametrize("edge_grid", [1, 3, 64, 2000])
def test_edge_grids(hgm, edge_grid):
    g = _mixed([3000, 12_000] * 9, 77)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    for h in (g, _instance(50_000, np.random.default_rng(1).integers(100, 300, 900),
                           np.arange(900) % 50, 2)):
        dg = hgm.DeviceHypergraph.from_host(h, "cuda:0")
        print(f"grid {edge_grid} m={h.m}", flush=True)
        bits, _ = hgm.match(dg, 3, hgm.make_opts(solo_max_kappa=-1, edge_grid=edge_grid),
                            want_stats=False)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), _exact(h))


@pytest.mark.parametrize("solo", [0, -1, 30_000])
def test_batch(hgm, solo):
    gs = [_mixed([2048, 2049, 30_000], 5, small=300), _mixed([20_000] * 3, 6, small=9000),
          _instance(40_000, [2500] * 90, np.arange(90) % 7 + 1, 8), synth.from_edge_lists(3, [], []),
          _mixed([50_000], 9, best=1)]
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    print(f"batch solo={solo}", flush=True)
    bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
    got = bits.cpu().numpy().view(np.uint32)
    for i, g in enumerate(gs):
        assert np.array_equal(got[int(b.word_base[i]):int(b.word_base[i + 1])], _exact(g, 5 + i)), i


@pytest.mark.parametrize("what", ["few", "one among small", "few of a batch"])
def test_time(hgm, what):
    """Against the same call with counts, whose rounds visit all live edges."""
    import torch
    rng = np.random.default_rng(4)
    if what == "few":
        g = _instance(700_000, rng.integers(15_000, 25_000, 64), rng.integers(1, 999, 64), 1)
    else:
        g = _mixed([300_000], 2, n=400_000, small=60_000)
    if what == "few of a batch":
        gs = [_mixed([100_000], 20 + i, n=100_000) for i in range(16)]
        b = hgm.DeviceBatch.from_host(
            synth.batch_from_instances(gs, np.arange(16, dtype=np.uint32)), "cuda:0")
        call = lambda stats: hgm.match_batch(b, want_stats=stats)
    else:
        dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
        ws = hgm.alloc_workspace(dg)
        call = lambda stats: hgm.match(dg, 3, workspace=ws, want_stats=stats)
    best = {}
    for stats in (False, True):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call(stats)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[stats] = min(t)
    print({k: round(v * 1e6) for k, v in best.items()}, flush=True)
    assert best[False] < 1.5 * best[True]
