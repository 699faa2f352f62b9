"""The iteration on both sides of the smallest size at which its stores go past the caches (3 MB of two vectors)."""
import pytest

from tests import test_gpu_iteration_stores as stores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [5, 16])
@pytest.mark.parametrize("n", [(3 << 20) // 24, (3 << 20) // 24 + 1])
def test_iteration_matches_graph(n, k):
    stores.test_iteration_matches_graph(n, k)
