"""GPU parity of the whole-compute-unit kernel with KV tiles of 128: one full tile, one ragged, a second of one and of
many keys, up to 256; one table, tables for some heads, none, the entry point that allocates nothing, float32 tensors."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import gpu, rand_case, run_gpu, run_dynamic, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bhn,gain", [((103, 7, 65), 1.0), ((65, 12, 127), 1.0), ((60, 12, 128), 0.1), ((129, 4, 129), 1.0),
                                      ((43, 6, 200), 30.0), ((80, 6, 256), 1.0)])
def test_whole_compute_unit_tile_128(gpu, bhn, gain):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N = bhn
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 64), 7500 + N)
    p = oracle.derive_params(sQ * gain, sK, 64, out_round=N % 2)
    ref = oracle.qflash_attention(Q, K, V, p, 128)
    assert_same(run_gpu(gpu, Q, K, V, p, 128), ref, "whole CU, tile 128 %s" % (bhn,))
    assert (ctx.cache_info().last_kernel, ctx.cache_info().last_key_waves) == (3, 0), bhn
    ps = [oracle.derive_params(sQ * g, sK, 64, out_round=0) for g in ([0.2, 1.0, 30.0] * H)[:H]]
    assert_same(run_gpu(gpu, Q, K, V, ps, 128), oracle.qflash_attention(Q, K, V, ps, 128), "the same, per head")


@pytest.mark.parametrize("bhn", [(100, 3, 129), (65, 12, 200), (64, 4, 250), (300, 1, 64)])
def test_whole_compute_unit_tile_128_from_floats(gpu, bhn):  # noqa: F811
    rng = np.random.default_rng(8500 + bhn[2])
    Qf, Kf, Vf = (rng.standard_normal(bhn + (64,), dtype=np.float32) for _ in range(3))
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, 128)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, 128)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert np.array_equal(out, ref)
