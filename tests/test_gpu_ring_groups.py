"""GPU parity of the direct-load ring for every size of workgroup the planner chooses, three to eight wavefronts, with
wavefronts beyond the sequence in the last workgroup of a pair (which must meet every barrier), with the wave priorities of
launches of one round and of several, and with sums of weights that change the loop.  Each case states what the plan has to be, so
that a change of the planner cannot move them all onto one size."""
import numpy as np
import pytest

import oracle
from tests.ring_plan import ring_plan, table_bytes, table_span
from tests.test_gpu_float_release import heavy_case
from tests.test_gpu_parity import gpu, rand_case, run_gpu, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu

# B, H, N, d, tile, scale of Q and K (which sets the size of the table), wavefronts to a workgroup, wavefronts of a pair without
# rows, wave priorities: none, one round of workgroups, several
NONE, ONE, MORE = "none", "one round", "several"
CASES = [(22, 4, 700, 64, 64, 0.09, 3, 2, ONE), (22, 4, 770, 64, 64, 0.06, 4, 3, ONE), (60, 4, 705, 64, 64, 0.06, 4, 1, MORE),
         (32, 12, 577, 64, 64, 0.0434, 4, 1, MORE), (22, 4, 257, 64, 64, 0.06, 5, 1, NONE), (20, 3, 513, 64, 64, 0.06, 6, 1, NONE),
         (20, 12, 400, 64, 64, 0.2, 7, 1, ONE), (10, 12, 770, 64, 64, 0.06, 7, 3, ONE), (20, 12, 450, 64, 64, 0.033, 8, 1, ONE),
         (43, 3, 700, 64, 64, 0.033, 8, 2, ONE),
         (22, 4, 700, 64, 128, 0.09, 3, 2, ONE), (22, 4, 770, 64, 128, 0.06, 4, 3, ONE), (40, 4, 705, 64, 128, 0.06, 4, 1, ONE),
         (30, 12, 330, 64, 128, 0.033, 6, 1, MORE), (8, 12, 1025, 64, 128, 0.033, 7, 2, ONE), (20, 12, 450, 64, 128, 0.036, 8, 1, ONE), (22, 12, 450, 64, 128, 0.033, 8, 1, MORE), (36, 3, 900, 64, 128, 0.036, 8, 3, ONE),
         (22, 4, 700, 32, 64, 0.06, 3, 2, ONE), (36, 3, 705, 32, 64, 0.2, 4, 1, ONE), (32, 12, 257, 32, 64, 0.0292, 5, 1, ONE),
         (43, 4, 513, 32, 64, 0.028, 6, 1, ONE), (12, 12, 700, 32, 64, 0.028, 6, 2, ONE),
         (22, 4, 700, 32, 128, 0.06, 3, 2, ONE), (8, 12, 1200, 32, 128, 0.0412, 4, 2, ONE), (20, 8, 400, 32, 128, 0.0412, 5, 2, ONE),
         (43, 4, 700, 32, 128, 0.028, 4, 2, MORE)]


def planned(shape, tile, p):
    plan = ring_plan(shape, tile, table_bytes(p))
    assert plan.ring
    rounds = NONE if plan.even_from == plan.grid else MORE if plan.even_from else ONE
    return plan.waves, plan.waves * plan.blocks - -(-shape[2] // 32), rounds


@pytest.mark.parametrize("B,H,N,d,tile,scale,waves,idle,rounds", CASES)
def test_workgroups_of_every_size(gpu, request, B, H, N, d, tile, scale, waves, idle, rounds):  # noqa: F811
    torch, qf, ctx = gpu
    shape = (B, H, N, d)
    p = oracle.derive_params(scale, scale, d, out_round=N % 2)
    table = request.node.callspec.params["gpu"] == "table"           # (without, the planner is asked for no table)
    assert not table or planned(shape, tile, p) == (waves, idle, rounds)
    inputs = [rand_case(shape, 40000 + N + d)[:3]]
    if N - N % tile - tile >= 560:                                   # keys ahead of the last full tile, of weight 120 and more
        inputs.append(heavy_case(shape, N + d))
    for i, (Q, K, V) in enumerate(inputs):
        ref, state = oracle.qflash_attention(Q, K, V, p, tile, return_state=True)
        if i == 1:
            assert state["l"].max() >= 65000 + 127 * (N % tile + tile)   # the last full tile belongs to the second loop
        assert_same(run_gpu(gpu, Q, K, V, p, tile), ref, "%s inputs %d" % (shape, i))
        info = ctx.cache_info()
        assert (info.last_kernel, info.last_key_waves, info.last_weight_mode) == (2, 0, qf.WEIGHTS_TABLE if table else qf.WEIGHTS_ARITHMETIC)


# Scores exactly on the lowest entry of the weight table, one above and one below it, in every 32-key block of a tile: the
# first block's index is a fused multiply-add whose result is then a zero, of either sign ahead of its clamp, the others' a
# saturating subtraction.
@pytest.mark.parametrize("kernel,B,H,N,d,tile", [(2, 60, 3, 300, 64, 64), (2, 60, 3, 300, 64, 128), (2, 60, 3, 200, 32, 64), (2, 60, 3, 200, 32, 128),
                                                 (3, 64, 12, 197, 64, 64), (3, 64, 12, 197, 64, 128), (1, 135, 6, 256, 64, 64)])
def test_scores_on_the_edge_of_the_table(gpu, request, kernel, B, H, N, d, tile):  # noqa: F811
    torch, qf, ctx = gpu
    p = oracle.derive_params(0.1, 0.1, d)
    edge = table_span(p)
    shape = (B, H, N, d)
    rng = np.random.default_rng(N + d)
    # Q.K = 127 a + b with |b| <= 63 per key: column 0 carries a (K) times 127 (Q), column 1 carries b times 1
    score = -edge + rng.integers(-1, 2, size=(B, H, N))
    score[:, :, ::7] = 0
    score[:, :, 1::11] = rng.integers(-edge, 1, size=score[:, :, 1::11].shape)
    a = np.zeros((d, B, H, N), np.int64)
    rest = score.copy()
    for f in range(d - 1):                                           # as many columns of 127 * 127 as it takes, then the rest
        a[f] = np.clip(rest // 127, -127, 127)
        rest = rest - 127 * a[f]
    a[d - 1] = rest
    assert np.abs(rest).max() <= 127 and edge < 127 * 127 * (d - 1)
    K = np.moveaxis(a, 0, -1).astype(np.int8)
    Q = np.full(shape, 127, np.int8)
    Q[..., d - 1] = 1
    V = rng.integers(-128, 128, size=shape).astype(np.int8)
    assert np.array_equal((Q[:, :, :1].astype(np.int64) @ np.swapaxes(K.astype(np.int64), -1, -2))[:, :, 0], score)
    assert_same(run_gpu(gpu, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "edge %s" % (shape,))
    info = ctx.cache_info()
    mode = qf.WEIGHTS_TABLE if request.node.callspec.params["gpu"] == "table" else qf.WEIGHTS_ARITHMETIC
    assert (info.last_kernel, info.last_key_waves, info.last_weight_mode) == (kernel, 0, mode)
