"""GPU parity of the last rounds in one workgroup (the default end of a call
with exact rounds): the bitmap and every per-round count equal the oracle's at
the edges of what that workgroup takes (2048 edges, 8192 pins), for many
rounds, in every variant and layout, with per-round priorities, under a round
limit and with explicit numbers of rounds per check."""
import numpy as np
import pytest

import oracle
import synth
from tests.fixtures import disjoint, path_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _check(hgm, g, seed=1, reseed=False, **kw):
    import torch
    kw.setdefault("solo_max_kappa", -1)
    print(f"n={g.n} m={g.m} kappa={g.kappa} seed={seed} reseed={reseed} {kw}", flush=True)
    exp, ref = oracle.local_max(g.n, g.m, g.e_off, g.e_pins, g.v_off, g.v_edges, g.w, seed,
                                reseed=reseed)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    bits, st = hgm.match(dg, seed, hgm.make_opts(reseed=reseed, **kw))
    got = bits.cpu().numpy().view(np.uint32)
    assert np.array_equal(got, exp)
    assert st["rounds"] == ref["rounds"]
    for k in ("live_edges", "live_pins", "matched_per_round"):
        assert np.array_equal(st[k], ref[k]), k
    sel = oracle.bits_to_bool(got, g.m)
    assert st["matched"] == int(sel.sum())
    assert st["weight"] == int(g.w[sel].astype(np.uint64).sum())


@pytest.mark.parametrize("variant", ["auto", "crcw", "crew"])
@pytest.mark.parametrize("reseed", [False, True])
def test_variants(hgm, variant, reseed):
    for n, m, hi in [(300, 600, 4), (9000, 20_000, 9), (40_000, 120_000, 5)]:
        g = synth.random_instance(m, n, m, 1, hi, 1, 3 if reseed else 1000, empty_frac=0.01)
        _check(hgm, g, m, reseed, variant=variant)


@pytest.mark.parametrize("reseed", [False, True])
@pytest.mark.parametrize("variant", ["auto", "crcw"])
def test_pairs(hgm, variant, reseed):
    rng = np.random.default_rng(8)
    a = rng.integers(0, 9000, 60_000)
    b = (a + rng.integers(1, 9000, 60_000)) % 9000
    pairs = synth.gen._unique_pairs(a, b, 9000)
    g = synth.from_pairs(9000, pairs, rng.integers(1, 9, pairs.shape[0]).astype(np.uint32))
    _check(hgm, g, 5, reseed, variant=variant, pairs=True)


@pytest.mark.parametrize("m", [120, 230, 1500, 2049, 4097])
def test_many_rounds(hgm, m):
    """A path of increasing weights: rounds beyond the rows read back at the
    check, within and beyond the edges that the workgroup takes."""
    _check(hgm, path_graph(m), variant="crcw")
    _check(hgm, path_graph(m), variant="auto", rounds_per_sync=7)


@pytest.mark.parametrize("n,m,size", [(60_000, 2047, 4), (60_000, 2048, 4), (60_000, 2300, 4),
                                      (40_000, 300, 30), (90_000, 40, 600), (30_000, 20, 9000)])
def test_bounds(hgm, n, m, size):
    """Sparse instances whose second round is about as large as the workgroup
    takes, in edges and in pins, and edges longer than all it takes."""
    for variant in ("auto", "crew"):
        _check(hgm, synth.random_instance(m, n, m, size, size, 1, 100), variant=variant)


@pytest.mark.parametrize("per_sync", [1, 2, 33, 99, 100, 200])
def test_rounds_per_sync(hgm, per_sync):
    _check(hgm, path_graph(260), variant="auto", rounds_per_sync=per_sync)
    _check(hgm, synth.random_instance(9, 5000, 15_000, 2, 6, 1, 9), variant="crcw",
           rounds_per_sync=per_sync)
    _check(hgm, disjoint(5000), variant="auto", rounds_per_sync=per_sync)


@pytest.mark.parametrize("variant", ["auto", "crew"])
def test_round_limit(hgm, variant):
    g = path_graph(301)                       # 151 rounds
    _check(hgm, g, 4, variant=variant, max_rounds=151)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    for limit in (1, 3, 60, 150):
        print(f"limit={limit}", flush=True)
        with pytest.raises(hgm.HgmError) as ei:
            hgm.match(dg, 4, hgm.make_opts(variant, max_rounds=limit, solo_max_kappa=-1))
        assert ei.value.code == hgm.HGM_E_ROUND_LIMIT


@pytest.mark.parametrize("reseed", [False, True])
@pytest.mark.parametrize("n,hubs,share", [(100, 0, 0), (400, 0, 0), (2000, 0, 0), (300_000, 0, 0),
                                          (300_000, 1, 0.3), (300_000, 40, 0.5)])
def test_sampled_hubs(hgm, n, hubs, share, reseed):
    """An edge-centric round 0 whose hubs come from a sample of the pins, from
    2^20 pins on: every vertex a hub, more than its table holds, none, one and
    some; the vertex side given and not."""
    import torch
    rng = np.random.default_rng(n + hubs)
    m, size = (1 << 20) // 4 + 3, 4
    pins = rng.integers(hubs, n - size, (m, 1)) + np.arange(size)
    if hubs:
        pick = rng.random(m) < share
        pins[pick, 0] = rng.integers(0, hubs, int(pick.sum()))
    g = synth.from_edge_lists(n, pins, rng.integers(1, 1000, m).astype(np.uint32))
    exp, ref = oracle.local_max(g.n, g.m, g.e_off, g.e_pins, g.v_off, g.v_edges, g.w, 3,
                                reseed=reseed)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    bare = hgm.DeviceHypergraph(g.n, g.m, dg.e_off, dg.e_pins, none, none, dg.w)
    for d, variant in ((dg, "crcw"), (bare, "auto")):
        print(f"n={n} hubs={hubs} reseed={reseed} {variant}", flush=True)
        bits, st = hgm.match(d, 3, hgm.make_opts(variant, reseed=reseed))
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)
        for k in ("live_edges", "live_pins", "matched_per_round"):
            assert np.array_equal(st[k], ref[k]), k
