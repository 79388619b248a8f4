"""GPU parity of raw ranks (padded copies of the factors and intermediates, gradients cropped by the sum over
K-slices or by a copy) where their copies can go wrong: ranks below one 16-byte group, one off a multiple of
eight, matrices that end inside a group, and token counts on both sides of the sliced gradients."""
import pytest

from test_gpu_conv import run_tucker
from test_gpu_linear import run_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n_in,n_out,r", [(3, 8, 16, 1), (41, 16, 24, 3), (300, 64, 40, 7), (513, 72, 136, 9), (4099, 64, 64, 15),
                                            (6000, 48, 96, 33), (700, 264, 520, 129)])
def test_raw_rank_linear(T, n_in, n_out, r):
    run_linear(T, n_in, n_out, r, "bf16", 0, seed=T + r)


@pytest.mark.parametrize("N,hw,C,S,r1,r2,stride", [(1, 5, 8, 16, 1, 3, 1), (2, 9, 16, 24, 7, 9, 2), (5, 14, 40, 64, 17, 24, 1),
                                                   (6, 28, 64, 64, 24, 33, 1)])
def test_raw_rank_tucker(N, hw, C, S, r1, r2, stride):
    run_tucker(N, hw, hw, C, S, r1, r2, 3, stride, 1, "bf16", 0, seed=hw + r1)
