"""GPU parity where the float form of ScaleRelease meets its limit, where the last tile of the direct-load ring takes
another variant and where quotients of the normalisation are whole numbers: sums of weights that pass 65000 in the middle of a sequence (the integer form takes over), numerators
beyond 2^23, and sequences with every kind of remainder."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_kernel_families import batch, run
from tests.test_gpu_parity import gpu, rand_case, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu


def heavy_case(shape, seed):
    """Nearly equal scores (weights 120 to 127) whose maximum moves up a little in most tiles; V at its limits, so that
    the numerators of half the features pass 2^23 in magnitude."""
    B, H, N, d = shape
    rng = np.random.default_rng(seed)
    Q = np.zeros(shape, np.int8)
    K = rng.integers(-1, 2, shape).astype(np.int8)
    Q[..., 0] = rng.integers(1, 4, shape[:3])
    K[..., 0] = np.minimum(np.arange(N) * 20 // N, 127)[None, None, :]
    V = rng.choice(np.array([-128, -127, 127], np.int8), shape)
    V[..., : d // 4] = -128
    V[..., d // 4: d // 2] = 127
    return Q, K, V


@pytest.mark.parametrize("N,d,tile", [(700, 64, 64), (704, 64, 64), (713, 64, 128), (1024, 64, 128), (700, 32, 64), (721, 32, 128), (1152, 32, 64)])
def test_sums_beyond_the_float_form(gpu, N, d, tile):  # noqa: F811
    H = 3
    Q, K, V = heavy_case((batch(H, N), H, N, d), N + d)
    p = oracle.derive_params(0.02, 0.02, d)
    ref, state = oracle.qflash_attention(Q, K, V, p, tile, return_state=True)
    assert state["l"].max() > 65000 + 127 * tile                # reached before the last tile
    assert_same(run(gpu, 2, Q, K, V, p, tile), ref, "sums %d %d %d" % (N, d, tile))


REMAINDERS = [1, 7, 8, 9, 16, 17, 25, 32, 33, 63]


@pytest.mark.parametrize("d,tile,full", [(64, 64, 256), (64, 128, 256), (32, 64, 64), (32, 128, 128)])
@pytest.mark.parametrize("rem", REMAINDERS)
def test_last_tile_of_the_ring(gpu, d, tile, full, rem):  # noqa: F811
    H = 3
    for N in [full + rem] + ([full + 64 + rem] if tile == 128 else []):
        shape = (batch(H, N), H, N, d)
        Q, K, V, sQ, sK, _ = rand_case(shape, 30000 + N, q_gain=1.0 + rem % 2)
        for scale in (1.0, 40.0):                                # 40: coarse scores, x_shift > 0
            p = oracle.derive_params(sQ * scale, sK * scale, d, out_round=rem % 2)
            assert_same(run(gpu, 2, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s x%g" % (shape, scale))


# Every value of V in turn for a whole column, so that the quotient is that integer exactly, and columns one weight above
# and below it; equal weights (the largest denominators) and random ones; a batch per kernel.
@pytest.mark.parametrize("kernel,B,H,N,d,tile", [
    (4, 64, 6, 49, 32, 64), (4, 64, 6, 64, 32, 64), (3, 64, 6, 197, 64, 64), (3, 48, 6, 256, 64, 64), (3, 64, 6, 197, 64, 128),
    (1, 200, 6, 256, 64, 64), (2, 12, 6, 257, 64, 64), (2, 12, 6, 259, 64, 128), (2, 4, 6, 700, 64, 64), (2, 30, 6, 200, 32, 64)])
def test_whole_quotients(gpu, kernel, B, H, N, d, tile):  # noqa: F811
    rng = np.random.default_rng(N + d)
    shape = (B, H, N, d)
    level = ((np.arange(B * H * d) * 3) // 2 % 256 - 128).astype(np.int64).reshape(B, H, 1, d)
    V = np.repeat(level, N, axis=2)
    V[:, :, N // 3, 1::3] += 1
    V[:, :, N // 2, 2::3] -= 1
    V = np.clip(V, -128, 127).astype(np.int8)
    K = rng.integers(-127, 128, shape).astype(np.int8)
    for Q in (np.zeros(shape, np.int8), rng.integers(-127, 128, shape).astype(np.int8)):
        for out_round in (0, 1):
            p = oracle.derive_params(0.02, 0.02, d, out_round=out_round)
            assert_same(run(gpu, kernel, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s %d" % (shape, out_round))
