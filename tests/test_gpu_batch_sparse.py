"""Batches of instances with few pins a vertex whose vertices share slots in a
workgroup: whichever of the one-workgroup kernels, the rounds by admission and
the rounds over all live edges takes them, every bitmap equals the oracle's;
and the default is not several times slower than the grid's rounds."""
import time

import numpy as np
import pytest

import oracle
import synth
from tests.test_gpu_long_edges import _instance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _sparse(n, m, size, seed):
    rng = np.random.default_rng(seed)
    return _instance(n, rng.integers(max(1, size // 2), size + size // 2 + 1, m),
                     rng.integers(1, 99, m), seed)


@pytest.mark.parametrize("n,m,size", [(18_500, 5000, 2), (40_000, 1000, 7), (40_000, 1000, 9),
                                      (100_000, 1000, 32), (60_000, 20_000, 1),
                                      (60_000, 9000, 4), (17_000, 1000, 32)])
@pytest.mark.parametrize("count", [1, 3, 30])
def test_parity(hgm, n, m, size, count):
    gs = [_sparse(n, m, size, 10 * i + m) for i in range(min(count, 3))]
    gs = [gs[i % len(gs)] for i in range(count)]
    if count == 3:     # one of another kind among them
        gs[1] = synth.random_instance(5, 300, 900, 1, 6, 1, 9)
    b = synth.batch_from_instances(gs, np.arange(5, 5 + count, dtype=np.uint32))
    for side in (True, False):
        db = hgm.DeviceBatch.from_host(b, "cuda:0")
        if not side:
            db.v_off = db.v_edges = None
        for solo in (0, -1):
            print(f"{count} of n={n} m={m} size={size} side={side} solo={solo}", flush=True)
            bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
            got = bits.cpu().numpy().view(np.uint32)
            for i, g in enumerate(gs):
                exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
                seg = got[int(b.word_base[i]):int(b.word_base[i + 1])]
                assert np.array_equal(seg, exp), i


@pytest.mark.parametrize("count", [1, 16])
def test_time(hgm, count):
    import torch
    gs = [_sparse(100_000, 1000, 32, i) for i in range(count)]
    b = synth.batch_from_instances(gs, np.arange(count, dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    best = {}
    for solo in (0, -1):
        o, t = hgm.make_opts(solo_max_kappa=solo), []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hgm.match_batch(db, o, want_stats=False)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[solo] = min(t)
    print({k: round(v * 1e6) for k, v in best.items()}, flush=True)
    assert best[0] < 1.6 * best[-1]
