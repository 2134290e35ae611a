"""GPU parity of the calls that want only the matching (no statistics): their
rounds admit the edges in steps of the order and end in one workgroup, and the
bitmap still equals the oracle's greedy matching, at the edges of a wave's
range, of the flattened windows and of the last workgroup's bounds."""
import numpy as np
import pytest

import oracle
import synth
from tests.fixtures import path_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _check(hgm, g, seed=1, edge_side=False, **kw):
    import torch
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    if edge_side:
        none = torch.empty(0, dtype=torch.int32, device="cuda:0")
        dg = hgm.DeviceHypergraph(g.n, g.m, dg.e_off, dg.e_pins, none, none, dg.w)
    kw.setdefault("solo_max_kappa", -1)   # the grid's rounds at every size
    print(f"n={g.n} m={g.m} kappa={g.kappa} seed={seed} {kw}", flush=True)
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, seed)[0]
    for _ in range(2):                    # a second call on the same workspace size
        bits, st = hgm.match(dg, seed, hgm.make_opts(**kw), want_stats=False)
        assert st is None
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)


SHAPES = [(1, 1), (2, 1), (63, 64), (64, 65), (200, 255), (300, 257), (500, 1024), (700, 1025),
          (900, 2048), (900, 2049), (3000, 9001), (20011, 65537), (70001, 300017)]


@pytest.mark.parametrize("weights", [(1, 1), (0, 3), (1, 1_000_000)])
@pytest.mark.parametrize("n,m", SHAPES)
def test_shapes(hgm, n, m, weights):
    g = synth.random_instance(1000 + m, n, m, 1, 7, *weights, empty_frac=0.02)
    _check(hgm, g, seed=m)
    _check(hgm, g, seed=m, edge_side=True, variant="crcw")


@pytest.mark.parametrize("n,m,lo,hi", [(6000, 300, 1500, 4000), (9000, 40, 2040, 2056),
                                       (3000, 2000, 1, 700), (50_000, 70_000, 60, 68),
                                       (200_000, 3, 60_000, 70_000)])
def test_long_edges(hgm, n, m, lo, hi):
    """Edges below, at and beyond a wave's window of 2048 flattened pins, and
    more live pins than the last workgroup takes."""
    _check(hgm, synth.random_instance(m, n, m, lo, hi, 1, 50))


@pytest.mark.parametrize("m", [1500, 2048, 2049, 20_001])
def test_many_rounds(hgm, m):
    """A path of increasing weights: a match per round, within and beyond the
    edges that the last workgroup takes."""
    _check(hgm, path_graph(m))


def test_disjoint_edges(hgm):
    """Every admitted edge stays live to its test: 120,000 disjoint edges."""
    m = 120_000
    edges = np.arange(3 * m).reshape(m, 3)
    _check(hgm, synth.from_edge_lists(3 * m, edges, np.ones(m, np.uint32)))


@pytest.mark.parametrize("kw", [dict(rounds_per_sync=1), dict(rounds_per_sync=3),
                                dict(edge_grid=1), dict(edge_grid=7), dict(edge_grid=4096)])
def test_schedules(hgm, kw):
    _check(hgm, synth.random_instance(4, 30_000, 80_000, 2, 9, 1, 1000), **kw)
    _check(hgm, synth.shuffle_lists(synth.random_instance(5, 900, 4000, 2, 40, 1, 1), 3), **kw)


def test_hubs(hgm):
    _check(hgm, synth.config_hub_stress(seed=3, n=20_000, m=90_000))
    _check(hgm, synth.config_power_law(seed=4, n=30_000, m=100_000))


@pytest.mark.parametrize("n", [50, 700, 40_000])
@pytest.mark.parametrize("wmax", [1, 1000])
def test_pairs(hgm, n, wmax):
    rng = np.random.default_rng(n + wmax)
    a = rng.integers(0, n, 6 * n)
    b = (a + rng.integers(1, n, 6 * n)) % n
    pairs = synth.gen._unique_pairs(a, b, n)
    g = synth.from_pairs(n, pairs, rng.integers(1, wmax + 1, pairs.shape[0]).astype(np.uint32))
    _check(hgm, g, pairs=True)
    _check(hgm, g, pairs=True, edge_side=True)


@pytest.mark.parametrize("solo", [-1, 3000, 0])
def test_batches(hgm, solo):
    """Batches without statistics: every instance in the grid's rounds, some,
    and by the default bound."""
    import torch
    gs = [synth.random_instance(7 + i, n, 2 * n, 1, 12, 1, 1 if i % 3 == 0 else 1000,
                                empty_frac=0.01)
          for i, n in enumerate([40, 41, 5000, 33, 64, 20_000, 100, 31, 777])]
    gs += [synth.from_edge_lists(0, [], []), path_graph(300), synth.from_edge_lists(4, [], [])]
    b = synth.batch_from_instances(gs, np.arange(50, 50 + len(gs), dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    for vertex_side in (True, False):
        if not vertex_side:
            db.v_off = db.v_edges = None
        bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
        got = bits.cpu().numpy().view(np.uint32)
        for i, g in enumerate(gs):
            exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 50 + i)[0]
            seg = got[int(b.word_base[i]):int(b.word_base[i + 1])]
            assert np.array_equal(seg, exp), f"instance {i}, vertex side {vertex_side}"
