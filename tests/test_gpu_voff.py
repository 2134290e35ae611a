"""A v_off that is not the transpose of the edge side, in calls that want only
the matching: refused where the rounds over all live edges with automatic bins
refuse it, answered as those rounds answer it where they do not, and a correct
one is accepted whatever the alignment and the remainders of the pins."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

N = (1 << 17) + 77      # automatic bins: n >= 2^17, kappa >= 2^20; 33 bins, the last of 77


@pytest.fixture(scope="module")
def hgm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_22976_amd as lib
    lib.load()
    return lib


@pytest.fixture(scope="module")
def skewed():
    """The lower half of the vertices holds three quarters of the pins."""
    g = synth.random_instance(31, N, 250_000, 4, 6, 1, 1000)
    rng = np.random.default_rng(32)
    low = rng.random(g.kappa) < 0.5
    pins = np.where(low, g.e_pins // 2, g.e_pins)
    edges = [sorted(set(pins[a:b].tolist())) for a, b in zip(g.e_off[:-1], g.e_off[1:])]
    g = synth.from_edge_lists(N, edges, g.w)
    assert g.kappa >= 1 << 20
    return g


def _device(hgm, g, v_off=None, shift=0):
    """The instance on the GPU, with another v_off, or with its pins `shift`
    elements behind an aligned address."""
    import torch
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    if v_off is not None:
        dg.v_off = torch.from_numpy(v_off.astype(np.int32)).to("cuda:0")
    if shift:
        room = torch.empty(g.kappa + shift, dtype=torch.int32, device="cuda:0")
        room[shift:] = dg.e_pins
        dg.e_pins = room[shift:]
    return dg


def _match(hgm, dg, ws=None, want_stats=False, **kw):
    import torch
    bits, _ = hgm.match(dg, 7, hgm.make_opts("auto", **kw), workspace=ws, want_stats=want_stats)
    torch.cuda.synchronize()
    return bits.cpu().numpy().view(np.uint32)


def _exact(g):
    return oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 7)[0]


def _offsets(degrees):
    return np.concatenate([[0], np.cumsum(degrees)])


@pytest.mark.parametrize("noalloc", [False, True])
def test_refused(hgm, skewed, noalloc):
    """The degrees in reverse order: the lower bins get too little room."""
    import torch
    g = skewed
    dg = _device(hgm, g, _offsets(np.diff(g.v_off)[::-1]))
    ws = hgm.alloc_workspace(dg)
    print("reversed degrees", flush=True)
    if noalloc:
        assert ws.numel() <= hgm.hgm_noalloc_max_bytes()
        bits = torch.empty((g.m + 31) // 32, dtype=torch.int32, device="cuda:0")
        assert hgm.hgm_match_noalloc(dg.csr(), 7, bits.data_ptr()) == hgm.HGM_E_CSR
    else:
        with pytest.raises(hgm.HgmError) as ei:
            _match(hgm, dg, ws)
        assert ei.value.code == hgm.HGM_E_CSR
    assert np.array_equal(_match(hgm, _device(hgm, g), ws), _exact(g))


def test_bad_offsets(hgm, skewed):
    """Offsets that decrease, or beyond kappa: refused before anything is read
    through them."""
    g = skewed
    for at, value in ((1000, -5), (1000, 0), (N - 3, g.kappa + 9)):
        v_off = g.v_off.copy()
        v_off[at] = value
        print(f"v_off[{at}] = {value}", flush=True)
        with pytest.raises(hgm.HgmError) as ei:
            _match(hgm, _device(hgm, g, v_off))
        assert ei.value.code == hgm.HGM_E_CSR


def test_accepted(hgm, skewed):
    """A few pins moved to another bin leave room enough: answered as the rounds
    over all live edges do.  Nearly all degrees on the last vertex: those rounds
    begin with the edge form and use no bins."""
    g = skewed
    deg = np.diff(g.v_off)
    deg[10] -= 1
    deg[N - 10] += 1
    dg = _device(hgm, g, _offsets(deg))
    print("one pin moved", flush=True)
    assert np.array_equal(_match(hgm, dg), _match(hgm, dg, want_stats=True))
    dg = _device(hgm, g, np.concatenate([np.zeros(N), [g.kappa]]))
    print("all on the last vertex", flush=True)
    assert np.array_equal(_match(hgm, dg), _exact(g))


@pytest.mark.parametrize("cut", [0, 1, 2, 3])
def test_correct(hgm, skewed, cut):
    g = skewed
    if cut:      # kappa less 1, 2 or 3 pins: the remainders of a 16-byte load
        edges = [g.e_pins[a:b].tolist() for a, b in zip(g.e_off[:-1], g.e_off[1:])]
        longest = max(range(g.m), key=lambda e: len(edges[e]))
        edges[longest] = edges[longest][:len(edges[longest]) - cut]
        g = synth.from_edge_lists(N, edges, g.w)
    for shift in range(4):
        print(f"kappa={g.kappa} shift={shift}", flush=True)
        assert np.array_equal(_match(hgm, _device(hgm, g, shift=shift)), _exact(g))
