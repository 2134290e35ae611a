"""GPU parity of the instances that one workgroup matches whole: hgm_match on
small instances and the solo part of batches, with and without statistics,
against the oracle's greedy matching and its round simulator."""
import numpy as np
import pytest

import oracle
import synth
from tests.fixtures import disjoint, path_graph, star

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


def _check(hgm, g, seed=1, pairs=False, reseed=True, bound=1 << 22):
    """One instance: the matching alone, with per-round counts, and with
    priorities redrawn every round."""
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    print(f"n={g.n} m={g.m} kappa={g.kappa} seed={seed} pairs={pairs}", flush=True)
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, seed)[0]
    opts = dict(pairs=pairs, solo_max_kappa=bound)
    bits, _ = hgm.match(dg, seed, hgm.make_opts(**opts), want_stats=False)
    assert np.array_equal(_bits(bits), exp)
    bits, st = hgm.match(dg, seed, hgm.make_opts(**opts))
    assert np.array_equal(_bits(bits), exp)
    args = (g.n, g.m, g.e_off, g.e_pins, g.v_off, g.v_edges, g.w, seed)
    _, want = oracle.local_max(*args)
    assert st["rounds"] == want["rounds"]
    for k in ("live_edges", "live_pins", "matched_per_round"):
        assert np.array_equal(st[k], want[k][:st[k].size]), k
    if reseed:
        exp, want = oracle.local_max(*args, reseed=True)
        for stats in (False, True):
            bits, st = hgm.match(dg, seed, hgm.make_opts(reseed=True, **opts), want_stats=stats)
            assert np.array_equal(_bits(bits), exp)
        assert st["rounds"] == want["rounds"]


# m: the edges of a wave, of one edge per thread, of the sampled thresholds and
# of a wave's range; n: the vertices whose maxima fit LDS and more.
@pytest.mark.parametrize("weights", [(1, 1), (0, 3), (1, 1_000_000)])
@pytest.mark.parametrize("n,m", [(1, 1), (40, 64), (64, 65), (500, 1023), (500, 1024),
                                 (600, 1025), (900, 2048), (900, 2049), (5000, 4097),
                                 (9000, 16_385), (40_000, 60_000)])
def test_shapes(hgm, n, m, weights):
    _check(hgm, synth.random_instance(m, n, m, 1, 9, *weights, empty_frac=0.02), seed=m)


@pytest.mark.parametrize("n,m,lo,hi", [(3000, 60, 100, 300), (6000, 700, 9, 40),
                                       (9000, 40, 2040, 2056), (20_000, 3000, 1, 70),
                                       (60_000, 1100, 1, 900)])
def test_long_edges(hgm, n, m, lo, hi):
    """More pins than the last rounds keep in registers, and edges beyond a
    wave's window."""
    _check(hgm, synth.random_instance(m, n, m, lo, hi, 1, 50))


@pytest.mark.parametrize("m", [700, 1500, 4500])
def test_many_rounds(hgm, m):
    """More rounds than the call's record of counts holds go on to the grid."""
    _check(hgm, path_graph(m), reseed=False)


@pytest.mark.parametrize("n", [30, 700, 6000])
def test_pairs(hgm, n):
    rng = np.random.default_rng(n)
    a = rng.integers(0, n, 6 * n)
    pairs = synth.gen._unique_pairs(a, (a + rng.integers(1, n, 6 * n)) % n, n)
    g = synth.from_pairs(n, pairs, rng.integers(1, 9, pairs.shape[0]).astype(np.uint32))
    _check(hgm, g, pairs=True)


def test_hubs(hgm):
    _check(hgm, synth.config_hub_stress(seed=3, n=3000, m=12_000))
    _check(hgm, synth.config_power_law(seed=4, n=9000, m=20_000))


@pytest.mark.parametrize("solo", [0, 2500, 1 << 20])
def test_batch(hgm, solo):
    """Instances on both sides of the vertex counts that fit a workgroup's
    share of LDS, of the bound, and beyond 8 LDS tiles of vertices."""
    lds = hgm.load().hgm_solo_lds_vertices()
    sizes = [(1, 1), (40, 90), (300, 600), (1000, 1024), (3000, 5000), (lds // 4, lds // 2),
             (lds // 2, lds), (lds, 20_000), (lds + 1, 30_000), (3 * lds, 50_000),
             (9 * lds, 4000), (70, 5000)]
    gs = [synth.random_instance(60 + i, n, m, 1, 10, 1, 1 if i % 4 == 0 else 1000, empty_frac=0.01)
          for i, (n, m) in enumerate(sizes)]
    gs += [synth.from_edge_lists(0, [], []), path_graph(300), synth.from_edge_lists(4, [], []),
           synth.random_instance(99, 3000, 30, 1, 1500, 1, 9)]
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    for side in (True, False):
        db = hgm.DeviceBatch.from_host(b, "cuda:0")
        if not side:
            db.v_off = db.v_edges = None
        bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
        for i, g in enumerate(gs):
            exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
            seg = _bits(bits)[int(b.word_base[i]):int(b.word_base[i + 1])]
            assert np.array_equal(seg, exp), f"instance {i}, vertex side {side}"


@pytest.mark.parametrize("solo", [0, 1 << 20])
def test_two_phases(hgm, solo):
    """The first parts of the order, then the edges they leave: instances at the
    least edges that are split, none or nearly all dead at the split, ties at
    its key, weights in the order of the ids, edges beyond a record's pins."""
    import torch
    gs = [synth.random_instance(200 + m, n, m, 1, 9, 1, w, empty_frac=0.02)
          for n in (60, 2500, 30_000) for m in (512, 513, 2048, 2049, 9001) for w in (1, 2, 10**6)]
    gs += [path_graph(5000), disjoint(20_000), disjoint(3000, size=40), star(6000), star(6000, wmax=1),
           synth.random_instance(9, 40_000, 5000, 3, 90, 1, 100)]
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
    got = bits.cpu().numpy().view(np.uint32)
    for i, g in enumerate(gs):
        exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
        assert np.array_equal(got[int(b.word_base[i]):int(b.word_base[i + 1])], exp), (i, g.n, g.m)
