"""Calls that want only the matching at the interface's largest sizes: n up to
2^31 - 1 on a workspace full of ones (whatever is not cleared shows), and
kappa near 2^31 and 2^30 by copies of a small instance (test_gpu_maxsize).

A matching does not depend on how the vertices are numbered, so the oracle
gets the edges on their few distinct vertices, numbered from 0."""
import numpy as np
import pytest

import oracle
import synth
from tests import test_gpu_maxsize as tiled

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


def _spread(g, n, seed):
    """The edges of g on ids spread over [0, n), the last ones among them."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = np.unique(rng.integers(0, n - g.n, 4 * g.n))
    ids = np.concatenate([rng.permutation(ids)[:g.n - 40], np.arange(n - 40, n)])
    return rng.permutation(ids).astype(np.int32)[g.e_pins]


@pytest.mark.parametrize("n", [2 ** 31 - 31, 2 ** 31 - 2, 2 ** 31 - 1])
def test_n_near_2_31(hgm, n):
    import torch
    g = synth.random_instance(501, 2000, 5000, 1, 7, 1, 30, empty_frac=0.01)
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 9)[0]
    t = lambda a: torch.from_numpy(a).to("cuda:0")
    none = torch.empty(0, dtype=torch.int32, device="cuda:0")
    dg = hgm.DeviceHypergraph(n, g.m, t(g.e_off), t(_spread(g, n, 502)), none, none,
                              t(g.w.view(np.int32)))
    ws = hgm.alloc_workspace(dg)
    print(f"n={n} workspace {ws.numel() / 2 ** 30:.1f} GiB", flush=True)
    for _ in range(2):
        ws.fill_(255)
        bits, _ = hgm.match(dg, 9, workspace=ws, want_stats=False)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)


def _check_tiled(hgm, K, g0, variant, vertex_side):
    bits0 = tiled._expect_g0(g0, 5)[0]
    dg = tiled._device_tiled(hgm, g0, K, vertex_side)
    print(f"K={K} kappa={dg.kappa} {variant} vertex_side={vertex_side}", flush=True)
    bits, _ = hgm.match(dg, 5, hgm.make_opts(variant), want_stats=False)
    got = bits.cpu().numpy().view(np.uint32).reshape(K, tiled.M0 // 32)
    assert np.array_equal(got, np.broadcast_to(bits0, got.shape))


def test_kappa_near_2_31_edge_form(hgm):
    g0 = tiled._g0()
    _check_tiled(hgm, (2 ** 31 - 1) // g0.kappa, g0, "crcw", False)


def test_kappa_2_30_auto_with_vertex_side(hgm):
    g0 = tiled._g0()
    _check_tiled(hgm, 2 ** 30 // g0.kappa, g0, "auto", True)
