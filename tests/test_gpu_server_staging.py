"""Waves of the request server go through chunks of pinned memory: arrays that
end at, below and beyond a chunk, bitmaps larger than all chunks of a worker,
empty requests among them; every bitmap equals the oracle's."""
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


def _serve(hgm, reqs, **kw):
    srv = hgm.Server(2 << 30, **kw)
    try:
        for _ in range(2):                    # the second burst finds every chunk used
            for i, g in enumerate(reqs):
                srv.submit(g, 50 + i, req_id=i)
            got, t0 = {}, time.time()
            while len(got) < len(reqs):
                got.update((r["id"], r) for r in srv.poll(cap=64, timeout_s=0.5))
                assert time.time() - t0 < 60
            for i, g in enumerate(reqs):
                exp = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 50 + i)[0]
                assert got[i]["status"] == 0
                assert np.array_equal(got[i]["bits"], exp), (i, g.m, g.kappa, kw)
    finally:
        srv.close()


CHUNK = 1 << 19  # pins (or weights) in a chunk of 2 MB


def _pinned(g):
    """The same instance in pinned memory, which large arrays are copied from
    without a chunk."""
    import torch
    for k in ("e_off", "e_pins", "v_off", "v_edges", "w"):
        x = getattr(g, k)
        setattr(g, k, torch.from_numpy(x.view(np.int32)).pin_memory().numpy().view(x.dtype))
    return g


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("edge_side_only", [True, False])
@pytest.mark.parametrize("workers", [1, 5])
def test_chunk_edges(hgm, workers, edge_side_only, pinned):
    reqs = [synth.from_edge_lists(0, [], []), synth.from_edge_lists(3, [[0, 2]], [7])]
    for kappa in (1, 63, 64, 65, CHUNK - 300, CHUNK, CHUNK + 1, 3 * CHUNK + 17):
        m = max(1, kappa // 4)
        sizes = np.full(m, kappa // m)
        sizes[:kappa - int(sizes.sum())] += 1
        rng = np.random.default_rng(kappa)
        n = 8 * max(int(sizes.max()), 2) + m
        edges = [((int(rng.integers(n)) + np.arange(k)) % n).tolist() for k in sizes]
        reqs.append(synth.from_edge_lists(n, edges, rng.integers(1, 99, m)))
        reqs.append(synth.from_edge_lists(5, [], []))
    if pinned:  # every other one: direct copies between chunks
        reqs = [_pinned(g) if i % 4 < 2 else g for i, g in enumerate(reqs)]
    _serve(hgm, reqs, workers=workers, edge_side_only=edge_side_only)


def test_bitmap_beyond_the_chunks(hgm):
    """64 workers have 512 KB of chunks each: 4.2 M bits, here twice as many."""
    m = 8_800_003
    off = np.arange(m + 1, dtype=np.int32)
    pins = (np.arange(m, dtype=np.int64) * 7 % 3_000_000).astype(np.int32)
    big = synth.from_edge_lists(10, [[0, 1], [1, 2]], [3, 4])
    big.n, big.m = 3_000_000, m
    big.e_off, big.e_pins = off, pins
    big.w = (np.arange(m) % 1000 + 1).astype(np.uint32)
    _serve(hgm, [synth.from_edge_lists(3, [[0, 2]], [7]), big], workers=64, max_batch=2,
           edge_side_only=True)
