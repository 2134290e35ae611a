"""Instances of a batch with more edges than pins (most edges empty) on both
sides of the solo part's bound: the one-workgroup kernels and the rounds over
the grid agree on who matches them, and every bitmap equals the oracle's."""
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


def _mostly_empty(m, seed):
    rng = np.random.default_rng(seed)
    edges = [[] for _ in range(m)]
    for e in rng.permutation(m)[:min(m, 60)]:
        edges[e] = sorted(rng.choice(50, 3, replace=False).tolist())
    return synth.from_edge_lists(50, edges, rng.integers(1, 9, m))


@pytest.mark.parametrize("solo", [0, 300, 1 << 16, (1 << 31) - 1])
@pytest.mark.parametrize("sizes", [(299, 300, 301), (100, 299), (5, 90_000, 300, 2000, 65_537)])
def test_edges_beyond_the_pins(hgm, sizes, solo):
    gs = [_mostly_empty(m, 40 + m) for m in sizes]
    gs.append(synth.random_instance(7, 200, 60, 1, 4, 1, 9))
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    print(f"edges {sizes} solo={solo}", flush=True)
    bits, _ = hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), want_stats=False)
    got = bits.cpu().numpy().view(np.uint32)
    for i, g in enumerate(gs):
        exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
        assert np.array_equal(got[int(b.word_base[i]):int(b.word_base[i + 1])], exp), i
