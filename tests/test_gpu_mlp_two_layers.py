"""The weight gradients of the two lower layers in one launch (k_dw_two) at the edges of their shares: more layers above, whose bias sums lie beside theirs,
a second layer with more tiles than the first and with fewer, workgroups with tiles of one layer only and of both; by the protocol of test_gpu_mlp_tiles."""
import pytest

import test_gpu_mlp_tiles as tiles

pytestmark = pytest.mark.gpu

SHAPES = [          # layer sizes, workers, rows per worker
    ((40, 70, 66, 50, 5), 3, 20),
    ((70, 40, 33, 129, 34, 4), 2, 70),
    ((33, 33, 400, 4), 5, 33),
    ((400, 33, 33, 4), 9, 16),
    ((257, 258, 259, 5), 40, 12),
]


@pytest.mark.parametrize("rule", list(tiles.RULES))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s[0])) + "_M%d_B%d" % s[1:])
def test_gradients_and_left_hand_sides(shape, rule):
    tiles.test_gradients_and_left_hand_sides(shape, rule)
