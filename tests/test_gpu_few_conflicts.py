"""Calls that want only the matching on both sides of the line up to which
instances whose edges meet few others run the rounds over all live edges, in
every layout and variant that the line tells apart, against the oracle."""
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


# pins an edge, edges, others met: 2^15 pins, 2^21 and 6 * 2^20 with the lines
# beside them
@pytest.mark.parametrize("size,m,others", [
    (2, 16_383, 1), (2, 16_384, 1), (2, 30_000, 5.9), (2, 30_000, 6.1), (2, 30_000, 11.9),
    (2, 30_000, 12.1), (4, 1 << 19, 11.9), (4, (1 << 19) + 1, 6.1), (4, (1 << 19) + 1, 5.9),
    (4, 1_700_000, 1.9), (4, 1_700_000, 2.1), (1, 40_000, 0.5), (0, 40_000, 0)])
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


def test_noalloc(hgm):
    g = _instance(60_000, 20_000, 2, 9)
    import torch
    dg = hgm.DeviceHypergraph.from_host(g, "cuda:0")
    bits = torch.empty((g.m + 31) // 32, dtype=torch.int32, device="cuda:0")
    assert hgm.hgm_match_noalloc(dg.csr(), 3, bits.data_ptr()) == 0
    exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 3)[0]
    assert np.array_equal(bits.cpu().numpy().view(np.uint32), exp)
