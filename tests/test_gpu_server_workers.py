"""The server's chunks at numbers of workers that do not divide its pinned
memory: every bitmap equals the oracle's (as in test_gpu_server_staging)."""
import pytest

from tests import test_gpu_server_staging as staging

pytestmark = pytest.mark.gpu
hgm = staging.hgm


@pytest.mark.parametrize("workers", [9, 11, 37])
def test_chunk_edges(hgm, workers):
    for pinned in (False, True):
        staging.test_chunk_edges(hgm, workers, workers == 11, pinned)
