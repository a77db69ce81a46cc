"""GPU parity of windowed attention on both sides of the lines where the kernel requests its first pair ahead of the table's barrier or
behind it: at most four runs of pairs to a workgroup and more, one pair to a run and two, with wavefronts that have none."""
import numpy as np
import pytest

import oracle
from workloads import EXCLUDED
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu


# pairs, of which a run takes as few as six or seven runs to a workgroup allow: 1024 four runs of one pair, 1025 five (the last workgroup has
# pairs for some of them only), 1536 six, 2049 two pairs to a run
@pytest.mark.parametrize("kind", ["plain", "packed", "none"])
@pytest.mark.parametrize("shape", [(512, 2, 64, 2, 1), (205, 5, 49, 41, 5), (512, 3, 33, 4, 3), (683, 3, 64, 1, 3)])
def test_first_requests(gpu, shape, kind):  # noqa: F811
    B, H, N, bB, bH = shape
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 32), 7100 + N)
    p = oracle.derive_params(sQ, sK, 32)
    bias = None
    if kind != "none":
        rng = np.random.default_rng(N)
        bias = rng.integers(-2500, 2500, size=(bB, bH, N, N)).astype(np.int32)
        bias[rng.random(bias.shape) < 0.25] = EXCLUDED
        bias[..., 0] = -3
    got = run_gpu(gpu, Q, K, V, p, 64, bias=bias, packed=kind == "packed")
    assert_same(got, oracle.qflash_attention(Q, K, V, p, 64, bias=bias), "%s %s" % (kind, shape))
