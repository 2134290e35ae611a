"""The autotuner starts from what a call without options gets, keeps it where no
candidate is faster, and does not give up for one kind of call what the other
kind gains."""
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


def _median(call, reps=15):
    import torch
    t = []
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        t.append((time.perf_counter() - t0) * 1e3)
    return sorted(t)[reps // 2]


def test_one_instance(hgm, tmp_path):
    """Calls with counts end in one workgroup (tail_pins 0), a quarter of their
    time here, and calls without run by admission, half of it: no candidate
    that gives either up is taken."""
    g = synth.random_instance(71, 10_000, 20_000, 2, 9, 1, 1000)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    best, rep = hgm.tune(dg, 5, hgm.make_opts("auto"), reps=7, cache=str(tmp_path / "c.txt"))
    print(rep, flush=True)
    assert rep["identical"]
    assert best.tail_pins == 0 and best.bin_shift in (-1, 0)
    ws = hgm.alloc_workspace(dg, hgm.make_opts(edge_grid=16384))
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5)[0]
    for stats in (False, True):
        call = lambda o: hgm.match(dg, 5, o, workspace=ws, want_stats=stats)
        assert np.array_equal(call(best)[0].cpu().numpy().view(np.uint32), exp)
        usual, tuned = _median(lambda: call(hgm.make_opts())), _median(lambda: call(best))
        print(f"stats={stats} default {usual:.4f} tuned {tuned:.4f} ms", flush=True)
        assert tuned < 1.2 * usual
    assert open(tmp_path / "c.txt").read().count("version=2") == 1


def test_default_time(hgm):
    """ms_default is the time of a call without options."""
    g = synth.random_instance(72, 200_000, 1_000_000, 2, 9, 1, 1000)
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    _, rep = hgm.tune(dg, 5, reps=5)
    ws = hgm.alloc_workspace(dg)
    usual = _median(lambda: hgm.match(dg, 5, workspace=ws, want_stats=False))
    print(rep, f"default {usual:.4f} ms", flush=True)
    assert abs(rep["ms_default"] - usual) < 0.15 * usual
