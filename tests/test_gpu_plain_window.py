"""GPU parity of windowed attention with a bias in the plain layout: the loads of four columns at the end of
a row, of the last row and of the tensor, runs that change the slice, every remainder of N by 4."""
import numpy as np
import pytest

import oracle
from workloads import EXCLUDED
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 33, 1, 1), (2, 3, 36, 2, 3), (5, 2, 47, 1, 2), (6, 4, 49, 3, 2), (300, 12, 50, 4, 12),
                                   (1200, 3, 63, 8, 3), (3, 2, 64, 3, 1), (2, 2, 144, 1, 2), (2, 2, 145, 2, 1), (40, 12, 146, 4, 12)])
def test_plain_window_bias(gpu, shape):  # noqa: F811
    B, H, N, bB, bH = shape
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 32), 6000 + N)
    p = oracle.derive_params(sQ, sK, 32)
    rng = np.random.default_rng(N)
    bias = rng.integers(-2500, 2500, size=(bB, bH, N, N)).astype(np.int32)
    bias[rng.random(bias.shape) < 0.25] = EXCLUDED
    bias[..., N - 1] = 17
    assert_same(run_gpu(gpu, Q, K, V, p, 64, bias=bias), oracle.qflash_attention(Q, K, V, p, 64, bias=bias), "plain %s" % (shape,))
