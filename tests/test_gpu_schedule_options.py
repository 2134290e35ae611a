"""Schedule options that a call must not pass over: results equal the oracle's
at every value, and the values that cost time cost it, which is how a call
shows from outside that it has heeded them."""
import time

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


def _best(hgm, g, want_stats, reps=8, **kw):
    """Least time of a call, its result checked."""
    import torch
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 3)[0]
    _, ref = oracle.local_max(g.n, g.m, g.e_off, g.e_pins, g.v_off, g.v_edges, g.w, 3)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    o = hgm.make_opts(**kw)
    ws = hgm.alloc_workspace(dg, o)
    t = []
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        bits, st = hgm.match(dg, 3, o, workspace=ws, want_stats=want_stats)
        torch.cuda.synchronize()
        t.append(time.perf_counter() - t0)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)
        if want_stats:
            assert st["rounds"] == ref["rounds"]
            assert np.array_equal(st["live_pins"], ref["live_pins"])
    print(kw, want_stats, round(min(t) * 1e6), "us", flush=True)
    return min(t)


@pytest.mark.parametrize("variant", ["auto", "crcw", "crew"])
def test_first_batch(hgm, variant):
    """32 rounds before the first check, where ten are enough; and four."""
    g = synth.random_instance(12, 20_000, 60_000, 2, 8, 1, 1000)
    few = _best(hgm, g, True, variant=variant, first_batch_pct=1)
    many = _best(hgm, g, True, variant=variant, first_batch_pct=400)
    usual = _best(hgm, g, True, variant=variant)
    assert many > 1.3 * usual and many > 1.3 * few


def test_never_a_last_workgroup(hgm):
    """A path of increasing weights: 750 rounds, nearly all of them in the last
    workgroup, or with tail_pins -1 none, whatever the call wants."""
    g = path_graph(1500)
    for want_stats in (False, True):
        usual = _best(hgm, g, want_stats, reps=4, solo_max_kappa=-1)
        never = _best(hgm, g, want_stats, reps=4, solo_max_kappa=-1, tail_pins=-1)
        assert never > 1.5 * usual


@pytest.mark.parametrize("n,m", [(500, 1025), (4000, 12_000), (30_000, 90_000)])
def test_never_a_last_workgroup_parity(hgm, n, m):
    g = synth.random_instance(m, n, m, 1, 7, 1, 9, empty_frac=0.02)
    for kw in (dict(), dict(variant="crcw"), dict(rounds_per_sync=1), dict(rounds_per_sync=7)):
        _best(hgm, g, False, reps=2, solo_max_kappa=-1, tail_pins=-1, **kw)
