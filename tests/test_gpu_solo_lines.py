"""hgm_match on instances of at most 1,024 edges, on both sides of the lines up
to which one workgroup takes them by default (in pins, by the vertices): the
bitmap equals the oracle's, and the default is not several times slower than
the grid's rounds where vertices share slots."""
import time

import numpy as np
import pytest

from tests.test_gpu_long_edges import _exact, _instance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _of_pins(n, m, kappa, seed):
    sizes = np.full(m, kappa // m)
    sizes[:kappa - int(sizes.sum())] += 1
    return _instance(n, sizes, np.random.default_rng(seed).integers(1, 40, m), seed)


@pytest.mark.parametrize("n", [400, 17_000, 18_500, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("kappa", [4096, 4097, 8192, 8193, 16_384, 16_385])
def test_lines(hgm, n, kappa):
    for m in (200, 1024):
        g = _of_pins(n, m, kappa, 3)
        dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
        print(f"n={n} m={m} kappa={kappa}", flush=True)
        for stats in (False, True):
            bits, _ = hgm.match(dg, 3, want_stats=stats)
            assert np.array_equal(bits.cpu().numpy().view(np.uint32), _exact(g))


@pytest.mark.parametrize("n,kappa", [(500_009, 64_000), (100_003, 64_000), (500_009, 32_000)])
def test_time(hgm, n, kappa):
    import torch
    dg = hgm.DeviceHypergraph.from_host(_of_pins(n, 1000, kappa, 5), "cuda:0")
    ws = hgm.alloc_workspace(dg)
    best = {}
    for solo in (0, -1):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hgm.match(dg, 3, hgm.make_opts(solo_max_kappa=solo), workspace=ws, want_stats=False)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[solo] = min(t)
    print(f"n={n} kappa={kappa}", {k: round(v * 1e6) for k, v in best.items()}, flush=True)
    assert best[0] < 2 * best[-1]
