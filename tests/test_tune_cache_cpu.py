"""Lines of a tuned-schedule cache, without a GPU (the key's device part reads
"unknown" then).  A line without a version wrote the library's defaults out,
whose meaning has since come to differ by the kind of call: they are read as
defaults.  A line of version 2 is taken as it stands."""
import ctypes

import pytest

import paper_2602_22976_amd as hgm
from tests.test_abi_cpu import _csr


@pytest.fixture(scope="module")
def lib():
    return hgm.load()


def _read(lib, tmp_path, line, **kw):
    path = tmp_path / "cache.txt"
    path.write_text(line + "\n")
    c = _csr(10_000, 20_000, 100_000)      # round(log2 kappa) = 17, mean size 5
    o = hgm.make_opts(**kw)
    assert lib.hgm_tuned_opts(str(path).encode(), ctypes.byref(c), ctypes.byref(o)) == 0
    return hgm.opts_dict(o)


KEY = "unknown match v0 p0 r0 k17 d5 c0 :"


def test_written_out_defaults(lib, tmp_path):
    o = _read(lib, tmp_path, KEY + " grid=1536 bpc=8 hub=8192 hot=64 clear=8 first=40 tail=-1 bins=0"
                                   " ms_default=1 ms_tuned=0.5")
    assert o == {k: 0 for k in o}


def test_tuned_fields_of_an_older_line(lib, tmp_path):
    o = _read(lib, tmp_path, KEY + " grid=2048 bpc=8 hub=1024 hot=64 clear=2 first=40 tail=4096"
                                   " bins=-1 ms_default=1 ms_tuned=0.5")
    assert (o["edge_grid"], o["hub_threshold"], o["clear_ratio"], o["tail_pins"],
            o["bin_shift"]) == (2048, 1024, 2, 4096, -1)
    assert o["blocks_per_cu"] == o["hot_degree"] == o["first_batch_pct"] == 0


def test_version_2(lib, tmp_path):
    o = _read(lib, tmp_path, KEY + " version=2 grid=1536 bpc=0 hub=0 hot=64 clear=0 first=40"
                                   " tail=-1 bins=0 ms_default=1 ms_tuned=0.5")
    assert (o["edge_grid"], o["hot_degree"], o["first_batch_pct"], o["tail_pins"]) == (1536, 64, 40, -1)
    assert o["blocks_per_cu"] == o["hub_threshold"] == 0


def test_graphs(lib, tmp_path):
    key = KEY.replace("p0", "p1")
    o = _read(lib, tmp_path, key + " first=35 tail=-1 grid=1536", pairs=True)
    assert o["first_batch_pct"] == o["tail_pins"] == o["edge_grid"] == 0
    o = _read(lib, tmp_path, key + " first=40", pairs=True)
    assert o["first_batch_pct"] == 40


def test_batches(lib, tmp_path):
    path = tmp_path / "cache.txt"
    path.write_text("unknown batch v0 p0 r0 k17 d5 c3 : solo=65536 grid=4096 bpc=8 hub=8192\n")
    b = hgm.HgmBatch()
    b.count, b.n_total, b.m_total, b.kappa_total, b.words_total = 8, 9000, 20_000, 100_000, 800
    o = hgm.make_opts()
    assert lib.hgm_tuned_batch_opts(str(path).encode(), ctypes.byref(b), ctypes.byref(o)) == 0
    assert (o.solo_max_kappa, o.edge_grid, o.blocks_per_cu, o.hub_threshold) == (65536, 0, 0, 0)
