"""Final tree of pools of up to 256 nodes, which one wave selects: two and four scores a lane, pools that are not full, masks on either side
of the size from which a wave writes a row."""
import pytest

from test_gpu_narrow_tree import test_final_tree_and_accept_walk as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scores", ["falling", "ties", "equal", "special"])
@pytest.mark.parametrize("k,calls,m,n", [(4, 3, 16, 36), (16, 1, 16, 17), (8, 2, 60, 64), (8, 2, 51, 65), (8, 2, 52, 66), (4, 8, 25, 117),
                                         (4, 9, 127, 129), (4, 9, 128, 130), (4, 9, 25, 133), (9, 4, 60, 193), (9, 4, 128, 194), (9, 4, 1, 253),
                                         (5, 11, 60, 256), (5, 11, 127, 2)])
def test_one_wave_selects(k, calls, m, n, scores):
    check(k, calls, m, n, scores)
