"""Network gradients on grids with inner bricks (16 x 4 x 4 voxels, whose halo needs no wrap), at the
finest level and one below it, and with more bricks than the weight gradient has partial sums (96), a
remainder among them. Reference and tolerances as in test_gpu_nn_backward.
"""
import pytest

from test_gpu_nn_backward import pytestmark, test_gradient_at_brick_edges as check  # noqa: F401


@pytest.mark.parametrize("n", [(96, 24, 24), (52, 28, 20), (48, 12, 12)])
def test_gradient_with_inner_bricks(n):
    check(n)
