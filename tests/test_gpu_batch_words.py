"""A batch's bitmap words that no edge needs (word_base may leave room behind an
instance) come back zero, whichever kernels match the instances."""
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


@pytest.mark.parametrize("want_stats", [False, True])
@pytest.mark.parametrize("solo", [0, -1, 300])
def test_words_behind_an_instance(hgm, solo, want_stats):
    import torch
    sizes = [(40, 90), (3, 0), (500, 1500), (1, 1), (0, 0), (70, 64)]
    gs = [synth.random_instance(80 + i, n, m, 1, 6, 1, 9) if m else synth.from_edge_lists(n, [], [])
          for i, (n, m) in enumerate(sizes)]
    b = synth.batch_from_instances(gs, np.arange(5, 5 + len(gs), dtype=np.uint32))
    room = [(g.m + 31) // 32 + 1 + i for i, g in enumerate(gs)]
    b.word_base = np.concatenate([[0], np.cumsum(room)]).astype(np.int64)
    db = hgm.DeviceBatch.from_host(b, "cuda:0")
    bits = torch.full((int(b.word_base[-1]),), -1, dtype=torch.int32, device="cuda:0")
    print(f"solo={solo} stats={want_stats}", flush=True)
    hgm.match_batch(db, hgm.make_opts(solo_max_kappa=solo), bits=bits, want_stats=want_stats)
    got = bits.cpu().numpy().view(np.uint32)
    for i, g in enumerate(gs):
        exp = np.zeros(room[i], np.uint32)
        exp[:(g.m + 31) // 32] = oracle.greedy(g.n, g.m, g.e_off, g.e_pins, g.w, 5 + i)[0]
        assert np.array_equal(got[int(b.word_base[i]):int(b.word_base[i + 1])], exp), i
