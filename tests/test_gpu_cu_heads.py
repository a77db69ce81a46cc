"""GPU parity of the whole-compute-unit kernel with one set of constants per head: heads with and without a
table in one workgroup, pairs of several heads behind one table, workgroups without any, a short last workgroup."""
import pytest

import oracle
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bhn,gains", [
    ((60, 12, 197), [0.2, 1.0, 30.0]),        # tables of different sizes, some heads too fine for one
    ((129, 4, 70), [1.0, 1.2]),               # every head has a table
    ((103, 5, 130), [0.1]),                   # none has
    ((87, 3, 200), [1.0, 0.15, 2.0]),         # last workgroup with fewer pairs
    ((100, 6, 256), [0.9, 0.3]),
    ((600, 1, 65), [1.0])])
def test_whole_compute_unit_per_head(gpu, bhn, gains):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N = bhn
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 64), 7000 + N)
    ps = [oracle.derive_params(sQ * gains[h % len(gains)], sK, 64, out_round=N % 2) for h in range(H)]
    out = run_gpu(gpu, Q, K, V, ps, 64)
    assert ctx.cache_info().last_kernel == 3, bhn
    assert_same(out, oracle.qflash_attention(Q, K, V, ps, 64), "whole CU per head %s" % (bhn,))
