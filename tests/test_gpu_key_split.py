"""GPU parity of the kernel that shares out the keys of 32 query rows (launches too small to fill the
chip): bit for bit against the CPU oracle where its indexing can go wrong -- one key block to several
chunks of wavefronts, ragged last blocks, tiles of 64 and 128 across chunk borders, both head sizes,
four and eight wavefronts per workgroup, bias in both layouts, one or several sets of constants."""
import numpy as np
import pytest

import oracle
from workloads import EXCLUDED
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu

# (B, H, N, d)
SHAPES = [(1, 2, 1, 64), (2, 1, 32, 32), (1, 3, 33, 64), (3, 2, 64, 64), (1, 2, 65, 32), (2, 2, 96, 64), (1, 3, 97, 32),
          (2, 2, 128, 64), (1, 2, 129, 64), (1, 2, 255, 32), (1, 3, 256, 64), (1, 2, 257, 64), (1, 1, 512, 64),
          (1, 1, 513, 32), (1, 2, 545, 64), (1, 1, 1030, 64), (1, 1, 1030, 32),
          (9, 6, 160, 64), (7, 7, 289, 64), (12, 8, 150, 32)]      # more workgroups than compute units


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("shape", SHAPES)
def test_key_split(gpu, shape, tile):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N, d = shape
    plan = qf.qflash_plan_query(ctx.handle, B, H, N, d, tile)
    windowed = d == 32 and 32 < N <= 64
    assert (plan.key_waves > 0) != windowed, shape
    Q, K, V, sQ, sK, _ = rand_case(shape, 3000 + N + d, q_gain=1.0 + (N % 3) * 0.4)
    for scale, rnd in ((1.0, N % 2), (40.0, 0)):             # 40: coarse scores, x_shift > 0
        p = oracle.derive_params(sQ * scale, sK * scale, d, out_round=rnd)
        assert_same(run_gpu(gpu, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s x%g" % (shape, scale))
    ps = [oracle.derive_params(sQ * g, sK, d) for g in ([0.2, 1.0, 30.0] + [1.3] * H)[:H]]     # tables for some heads
    assert_same(run_gpu(gpu, Q, K, V, ps, tile), oracle.qflash_attention(Q, K, V, ps, tile), "%s per head" % (shape,))


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[2] <= 545 and s[0] < 9])
def test_key_split_with_bias(gpu, shape):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N, d = shape
    tile = 128 if N % 2 else 64
    Q, K, V, sQ, sK, _ = rand_case(shape, 4000 + N + d)
    p = oracle.derive_params(sQ, sK, d)
    rng = np.random.default_rng(N)
    bias = rng.integers(-3000, 3000, size=(B, 1, N, N)).astype(np.int32)
    bias[rng.random(bias.shape) < 0.2] = EXCLUDED
    bias[0, 0, N // 2, :] = EXCLUDED                 # a row without keys
    bias[0, 0, 0, : N - 1] = EXCLUDED                # a row with the last key only
    bias[0, 0, 0, N - 1] = 5
    ref = oracle.qflash_attention(Q, K, V, p, tile, bias=bias)
    for packed in (False, True):
        assert_same(run_gpu(gpu, Q, K, V, p, tile, bias=bias, packed=packed), ref, "%s packed %s" % (shape, packed))
