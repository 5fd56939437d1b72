"""Final tree of narrow pools around the sizes where a thread of the block looks after one more node, and of the largest pool."""
import pytest

from test_gpu_narrow_tree import test_final_tree_and_accept_walk as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scores", ["falling", "ties", "equal", "special"])
@pytest.mark.parametrize("k,calls,m,n", [(8, 9, 63, 65), (8, 9, 64, 66), (16, 16, 128, 1024), (16, 16, 60, 2048), (16, 16, 60, 3074),
                                         (16, 16, 128, 3856), (16, 16, 1, 3857)])
def test_more_nodes_per_thread(k, calls, m, n, scores):
    check(k, calls, m, n, scores)
