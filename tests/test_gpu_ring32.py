"""GPU parity of the direct-load ring with 32 features per head: edges of tiles and row blocks, every
workgroup size the plan can choose, look-ups mixed with computed weights (full tiles) and ragged tails."""
import pytest

import oracle
from tests.ring_plan import ring_plan, table_bytes
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu

# (B, H, N): more than two workgroups of 32 rows per compute unit, so that the keys are not shared out
SHAPES = [(60, 4, 65), (60, 4, 96), (45, 4, 128), (45, 4, 129), (30, 4, 191), (30, 4, 256), (24, 4, 257),
          (12, 8, 320), (8, 12, 577), (5, 8, 513), (4, 6, 1000)]


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("bhn", SHAPES)
def test_ring32(gpu, bhn, tile):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N = bhn
    plan = qf.qflash_plan_query(ctx.handle, B, H, N, 32, tile)
    assert plan.kernel == 2 and plan.key_waves == 0 and plan.query_blocks * plan.wavefronts_per_pair * 32 >= N, bhn
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 32), 5000 + N, q_gain=1.0 + (N % 3) * 0.4)
    for scale in (1.0, 40.0):                                # 40: coarse scores, x_shift > 0
        p = oracle.derive_params(sQ * scale, sK * scale, 32, out_round=N % 2)
        assert_same(run_gpu(gpu, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s x%g" % (bhn, scale))
        info = ctx.cache_info()
        assert (info.last_kernel, info.last_key_waves) == (2, 0), bhn
    if N in (129, 577):
        ps = [oracle.derive_params(sQ * g, sK, 32) for g in ([0.2, 1.0, 30.0] + [1.3] * H)[:H]]
        assert_same(run_gpu(gpu, Q, K, V, ps, tile), oracle.qflash_attention(Q, K, V, ps, tile), "%s per head" % (bhn,))


# weight tables on either side of the size from which part of the weights is computed, full tiles and a ragged one
@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("gain", [1.0, 2.6, 2.74, 2.85, 3.5])
def test_ring32_mixed_weights(gpu, gain, tile):  # noqa: F811
    torch, qf, ctx = gpu
    Q, K, V, sQ, sK, _ = rand_case((12, 4, 420, 32), 6000, q_gain=1.0)
    p = oracle.derive_params(sQ * gain, sK, 32)
    assert_same(run_gpu(gpu, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "gain %g" % gain)
    info = ctx.cache_info()
    assert (info.last_kernel, info.last_key_waves) == (2, 0)


# one workgroup to a compute unit, where another share of the weights is computed: full tiles only, and a ragged one
@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("bhn", [(9, 4, 512), (9, 4, 642)])
def test_ring32_alone_on_a_compute_unit(gpu, bhn, tile):  # noqa: F811
    torch, qf, ctx = gpu
    shape = bhn + (32,)
    Q, K, V, sQ, sK, _ = rand_case(shape, 6100 + bhn[2])
    p = oracle.derive_params(sQ, sK, 32)
    plan = ring_plan(shape, tile, table_bytes(p))
    assert plan.ring and plan.units <= 256 and table_bytes(p) >= 7 * 1024
    assert_same(run_gpu(gpu, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s" % (shape,))
    info = ctx.cache_info()
    assert (info.last_kernel, info.last_key_waves) == (2, 0)
