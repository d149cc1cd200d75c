"""The coding kernel's maps from blocks to workers and units, and the dual vectors' cut of the workers into runs: layouts
with whole rounds of eight units and a rest, buckets shared by workgroups with more workers than one XCD may hold, and
pieces with more than one run of more than one worker.  Dual vectors and streams bit for bit."""
import pytest

from test_gpu_game import qgx, test_dual_vectors_formed_in_the_coding_kernel as compare_routes  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,bucket,n_levels,slotted", [
    (8 * 4096, 3, 4096, 16, True), (19 * 4096 + 40, 5, 4096, 16, True), ((1 << 20) + 8, 5, 8192, 16, True),
    (2 * 65536 + 4096, 44, 65536, 32, True), (2 * 65536 + 4096, 57, 65536, 32, False), (65536 + 20000, 33, 65536, 126, True)])
def test_maps(qgx, d, K, bucket, n_levels, slotted):
    compare_routes(qgx, d, K, bucket, n_levels, slotted, None)
