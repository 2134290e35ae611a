"""Calls that want only the matching on instances whose edges meet few others: a
sample of the edges picks the step of the order that round 1 goes on with, or
the rounds over all live edges.  Both sides of the lines that decide whether the
sample is taken and what it picks, evenly spread and with popular vertices, in
every layout, against the oracle; and the steps are kept where a vertex is
popular."""
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


def _instance(n, m, size, seed):
    """Edges of `size` vertices n / size apart, from a random one on."""
    rng = np.random.default_rng(seed)
    step = n // max(size, 1)
    pins = (rng.integers(0, n, (m, 1)) + step * np.arange(size)) % n
    pins = np.sort(pins, axis=1)
    return synth.from_edge_lists(n, pins, rng.integers(1, 1000, m).astype(np.uint32))


# pins an edge, edges, others met on average: the lines at 2^14, 2^18, 2^19 and
# 2^21 pins, at 1.5, 4, 5, 6 and 14 others up to 2^21 pins, at 3, 4.5 and 5 beyond,
# at 8 pins an edge; fewer edges than are sampled.
@pytest.mark.parametrize("size,m,others", [
    (2, 8191, 1), (2, 8192, 1), (2, 16_384, 1), (2, 30_000, 4.5), (2, 30_000, 5.5),
    (2, 30_000, 13.9), (2, 30_000, 14.1), (4, 1 << 16, 13), (4, (1 << 16) + 1, 13),
    (4, 1 << 19, 11.9), (4, (1 << 19) + 1, 6.1), (4, (1 << 19) + 1, 4.9), (4, 600_000, 2.5),
    (4, 1_700_000, 1.9), (2, 1 << 18, 3), (2, (1 << 18) + 1, 3), (2, 400_000, 5.5),
    (3, 300_000, 3.9), (1, 600_000, 0.3), (0, 600_000, 0), (1, 40_000, 0.5), (0, 40_000, 0), (8, 2050, 0.5), (8, 3000, 9),
    (9, 3000, 9)])
def test_line(hgm, size, m, others):
    import torch
    n = max(int(size * size * m / others), size + 1) if others else 100
    g = _instance(n, m, size, m)
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 3)[0]
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    bare = hgm.DeviceHypergraph(g.n, g.m, dg.e_off, dg.e_pins, none, none, dg.w)
    runs = [(dg, {}), (dg, dict(variant="crcw")), (bare, {})]
    if size == 2:
        runs += [(dg, dict(pairs=True)), (bare, dict(pairs=True))]
    for d, kw in runs:
        print(f"n={n} m={m} size={size} {kw}", flush=True)
        bits, _ = hgm.match(d, 3, hgm.make_opts(**kw), want_stats=False)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)


def _popular(n, m, size, seed):
    """Pins by rank^-1 and their neighbours."""
    rng = np.random.default_rng(seed)
    first = np.minimum(np.exp(rng.random((m, 1)) * np.log(n)).astype(np.int64) - 1, n - 1)
    pins = np.sort((first + rng.integers(1, n // size, (m, 1)) * np.arange(size)) % n, axis=1)
    return synth.from_edge_lists(n, pins, rng.integers(1, 1000, m).astype(np.uint32))


@pytest.mark.parametrize("size,m,others", [(2, 9000, 2), (2, 40_000, 1), (3, 200_000, 4),
                                           (2, 1_200_000, 1)])
def test_popular(hgm, size, m, others):
    g = _popular(int(size * size * m / others), m, size, m)
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 3)[0]
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    forms = [dict(), dict(rounds_per_sync=1), dict(rounds_per_sync=3), dict(edge_grid=40),
             dict(tail_pins=-1)] + ([dict(pairs=True)] if size == 2 else [])
    for kw in forms:
        print(f"n={g.n} m={m} size={size} {kw}", flush=True)
        bits, _ = hgm.match(dg, 3, hgm.make_opts(**kw), want_stats=False)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)


def test_batch(hgm):
    """The sample takes a batch's vertices apart."""
    gs = [_instance(90_000, 20_000, 3, 1), _popular(60_000, 20_000, 2, 2), _instance(50, 60, 2, 3),
          synth.from_edge_lists(4, [], []), _instance(90_000, 20_000, 3, 1)]
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=-1), want_stats=False)
    got = bits.cpu().numpy().view(np.uint32)
    for i, g in enumerate(gs):
        exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
        assert np.array_equal(got[int(b.word_base[i]):int(b.word_base[i + 1])], exp), i


def test_steps_stay_for_a_popular_vertex(hgm):
    """A star, whose edges meet few others by the means and all others in truth:
    admission takes a fraction of the time of the rounds over all live edges."""
    import torch
    m = 300_000
    g = synth.from_edge_lists(m + 1, np.stack([np.zeros(m, np.int64), np.arange(1, m + 1)], 1),
                              np.random.default_rng(1).integers(1, 999, m).astype(np.uint32))
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    dg = hgm.DeviceHypergraph(g.n, g.m, dg.e_off, dg.e_pins, none, none, dg.w)
    ws, best = hgm.alloc_workspace(dg), {}
    for stats in (False, True):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hgm.match(dg, 3, workspace=ws, want_stats=stats)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[stats] = min(t)
    print({k: round(v * 1e6) for k, v in best.items()}, flush=True)
    assert best[False] < 0.8 * best[True]


def test_noalloc(hgm):
    g = _instance(60_000, 20_000, 2, 9)
    import torch
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    bits = torch.empty((g.m + 31) // 32, dtype=torch.int32, device="cuda:0")
    assert hgm.hgm_match_noalloc(dg.csr(), 3, bits.data_ptr()) == 0
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 3)[0]
    assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)
