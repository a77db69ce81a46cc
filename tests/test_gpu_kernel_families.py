"""GPU parity of each kernel family on launches that really run it.  A launch of at most two blocks of 32 query rows per
compute unit shares out its keys instead (qflash_fwd_split), so that a test with a small batch never reaches the kernel
its shape stands for.  Here every launch is large enough, and says so: the plan before it and the context's report after
it.  Sequence lengths are those where a kernel's indexing can go wrong: one row into a block or a tile, whole blocks
and tiles, ragged tails, every way a workgroup is put together."""
import ctypes

import numpy as np
import pytest

import oracle
from workloads import EXCLUDED
from tests.test_gpu_parity import gpu, lib_params, rand_case, run_gpu, run_dynamic, assert_same  # noqa: F401

pytestmark = pytest.mark.gpu

BLOCKS = 513          # query blocks of 32 rows that an MI355X does not share out keys for


def batch(H, N):
    return -(-BLOCKS // (H * -(-N // 32)))


def random_bias(extents, N, seed):
    rng = np.random.default_rng(seed)
    bias = rng.integers(-3000, 3000, size=extents + (N, N)).astype(np.int32)
    bias[rng.random(bias.shape) < 0.2] = EXCLUDED
    bias[0, 0, N // 2, :] = EXCLUDED                # a row without keys
    return bias


def run(gpu, kernel, Q, K, V, p, tile, bias=None, packed=False):  # noqa: F811
    torch, qf, ctx = gpu
    plan = qf.qflash_plan_query(ctx.handle, *Q.shape, tile, *(bias.shape[:2] if bias is not None else (0, 0)))
    assert (plan.kernel, plan.key_waves) == (kernel, 0), Q.shape
    out = run_gpu(gpu, Q, K, V, p, tile, bias=bias, packed=packed)
    info = ctx.cache_info()
    assert (info.last_kernel, info.last_key_waves) == (kernel, 0), Q.shape
    return out


def scale_sets(sQ, sK, d, H, N):
    """A fine or a middling score scale, a coarse one (x_shift > 0), and one set per head of which some have a table."""
    per_head = [oracle.derive_params(sQ * g, sK, d) for g in ([0.2, 1.0, 30.0] + [1.3] * H)[:H]]
    return oracle.derive_params(sQ, sK, d, out_round=N % 2), oracle.derive_params(sQ * 40.0, sK * 40.0, d), per_head


# without a bias: the direct-load ring of 64 features; the resident kernel where the pairs do not fit one round of
# workgroups of the whole-compute-unit kernel, or where a pair is a single short block
NO_BIAS = [(2, 5, 257, 64, 64, 2), (2, 5, 288, 64, 128, 2), (2, 5, 320, 64, 64, 2), (2, 5, 383, 64, 128, 2), (2, 5, 384, 64, 64, 2),
           (2, 3, 449, 64, 64, 2), (2, 3, 512, 64, 128, 2), (2, 3, 513, 64, 128, 2), (2, 3, 640, 64, 64, 2),
           (2, 2, 1030, 64, 128, 2), (2, 2, 2049, 64, 64, 2), (2, 1, 4096, 64, 64, 2),
           (92, 12, 197, 64, 64, 1), (92, 12, 197, 64, 128, 1), (135, 6, 256, 64, 64, 1), (135, 6, 256, 64, 128, 1),
           (160, 12, 100, 64, 64, 1), (160, 12, 100, 64, 128, 1), (560, 6, 50, 64, 64, 1), (280, 6, 129, 64, 64, 1),
           (173, 3, 20, 32, 64, 1), (301, 2, 32, 32, 128, 1), (600, 1, 1, 32, 64, 1)]


@pytest.mark.parametrize("B,H,N,d,tile,kernel", NO_BIAS)
def test_without_a_bias(gpu, B, H, N, d, tile, kernel):  # noqa: F811
    B = max(B, batch(H, N))
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, d), 11000 + N + d, q_gain=1.0 + (N % 3) * 0.4)
    fine, coarse, per_head = scale_sets(sQ, sK, d, H, N)
    for i, p in enumerate((fine, coarse) if N < 300 else (fine,)):
        assert_same(run(gpu, kernel, Q, K, V, p, tile), oracle.qflash_attention(Q, K, V, p, tile), "%s constants %d" % (Q.shape, i))
    assert_same(run(gpu, kernel, Q, K, V, per_head, tile), oracle.qflash_attention(Q, K, V, per_head, tile), "%s per head" % (Q.shape,))


# with a bias: windows share a workgroup (up to four blocks of rows), whole sequences staged at once or tile by tile,
# the staged two-tile ring with workgroups of four to eight wavefronts, the streamed kernel
WITH_BIAS = [(4, 20, 64, 64, 1), (3, 33, 64, 64, 1), (4, 64, 64, 128, 1), (3, 97, 64, 64, 1), (3, 100, 64, 128, 1), (2, 128, 64, 64, 1),
             (3, 129, 64, 64, 1), (2, 160, 64, 128, 1), (3, 197, 64, 64, 1), (3, 197, 64, 128, 1), (2, 256, 64, 64, 1),
             (3, 257, 64, 64, 1), (2, 300, 64, 64, 1), (3, 257, 64, 128, 2), (2, 300, 64, 128, 2), (3, 384, 64, 128, 2),
             (2, 353, 64, 64, 2), (3, 384, 64, 64, 2), (2, 577, 64, 64, 2), (2, 640, 64, 128, 2), (1, 1089, 64, 64, 2),
             (4, 20, 32, 64, 1), (3, 65, 32, 64, 1), (3, 96, 32, 128, 1), (2, 144, 32, 64, 1), (2, 197, 32, 128, 1), (3, 256, 32, 64, 1),
             (2, 300, 32, 64, 1), (2, 449, 32, 128, 1), (1, 900, 32, 64, 1), (1, 1100, 32, 128, 1), (1, 2060, 32, 64, 0), (1, 2050, 32, 128, 0)]


@pytest.mark.parametrize("H,N,d,tile,kernel", WITH_BIAS)
def test_with_a_bias(gpu, H, N, d, tile, kernel):  # noqa: F811
    B = batch(H, N)
    B += B % 2
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, d), 12000 + N + d, q_gain=1.0 + (N % 3) * 0.4)
    fine, coarse, per_head = scale_sets(sQ, sK, d, H, N)
    for extents, p, label in (((2, H), fine, "fine"), ((1, 1), coarse, "coarse"), ((2, 1), per_head, "per head")):
        bias = random_bias(extents, N, N + d + tile)
        ref = oracle.qflash_attention(Q, K, V, p, tile, bias=bias)
        for packed in (False, True):
            assert_same(run(gpu, kernel, Q, K, V, p, tile, bias=bias, packed=packed), ref, "%s %s packed %s" % (Q.shape, label, packed))


# windows whose bias extents do not divide the batch stay on the resident kernel
@pytest.mark.parametrize("B,H,N,bias_B", [(173, 3, 49, 2), (259, 2, 33, 4), (129, 4, 64, 2)])
def test_windows_the_bias_does_not_divide(gpu, B, H, N, bias_B):  # noqa: F811
    Q, K, V, sQ, sK, _ = rand_case((B, H, N, 32), 13000 + N)
    p = oracle.derive_params(sQ, sK, 32)
    bias = random_bias((bias_B, H), N, N)
    ref = oracle.qflash_attention(Q, K, V, p, 64, bias=bias)
    for packed in (False, True):
        assert_same(run(gpu, 1, Q, K, V, p, 64, bias=bias, packed=packed), ref, "windows %s" % (Q.shape,))


# bias slices that repeat every 8 k units of work: workgroups are dealt to the XCDs by that period; whole and partial
# periods, one pair or several per workgroup, several query blocks per pair, one set of constants and one per head
@pytest.mark.parametrize("shape,bias_bh,tile,kernel", [
    ((44, 2, 197, 64), (8, 2), 64, 1), ((60, 1, 300, 64), (8, 1), 128, 2), ((18, 1, 1200, 64), (8, 1), 64, 2), ((48, 1, 353, 64), (8, 1), 64, 2),
    ((173, 3, 49, 32), (32, 3), 64, 1), ((600, 4, 20, 64), (14, 4), 64, 1), ((18, 2, 449, 32), (4, 2), 64, 1), ((10, 2, 2060, 32), (4, 2), 64, 0)])
def test_bias_period(gpu, shape, bias_bh, tile, kernel):  # noqa: F811
    torch, qf, ctx = gpu
    B, H, N, d = shape
    plan = qf.qflash_plan_query(ctx.handle, *shape, tile, *bias_bh)
    assert plan.bias_period_units > 0 and plan.units > plan.bias_period_units, shape
    Q, K, V, sQ, sK, _ = rand_case(shape, 16000 + N)
    fine, _, per_head = scale_sets(sQ, sK, d, H, N)
    bias = random_bias(bias_bh, N, N)
    for p, label in ((fine, "one set"), (per_head, "per head")):
        ref = oracle.qflash_attention(Q, K, V, p, tile, bias=bias)
        for packed in (False, True):
            assert_same(run(gpu, kernel, Q, K, V, p, tile, bias=bias, packed=packed), ref, "%s %s packed %s" % (shape, label, packed))


# The entry point that allocates nothing, where it builds its table: every family, one call after the other on one
# stream, each with another table in the same memory, a launch without a table in between.
def test_static_entry_point_with_its_table(gpu):  # noqa: F811
    torch, qf, ctx = gpu
    lib = qf.load_library()
    stream = ctypes.c_void_p(torch.cuda.current_stream("cuda:0").cuda_stream)
    done = []
    for (B, H, N, d), tile, gain, bias_bh in (((48, 12, 197, 64), 64, 1.5, None), ((2, 3, 70, 64), 64, 2.0, None), ((16, 8, 300, 64), 64, 1.7, None),
                                              ((66, 12, 130, 64), 128, 1.6, None), ((24, 8, 300, 32), 64, 1.5, None),
                                              ((300, 3, 49, 32), 64, 3.0, (4, 3)), ((60, 3, 100, 32), 64, 3.0, (1, 3)),
                                              ((16, 4, 384, 64), 128, 1.8, (1, 1)), ((40, 6, 197, 64), 64, 2.2, (1, 1))):
        Q, K, V, sQ, sK, _ = rand_case((B, H, N, d), 14000 + N, q_gain=gain)
        p = oracle.derive_params(sQ, sK, d)
        assert ((8 * p.s_inv) >> p.x_shift) + 17 <= 32 * 1024
        bias = None if bias_bh is None else random_bias(bias_bh, N, N)
        t = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (Q, K, V)]
        tb = None if bias is None else torch.from_numpy(bias).to("cuda:0")
        o = torch.full(Q.shape, 0x55, dtype=torch.int8, device="cuda:0")
        lp = lib_params(qf, p)
        rc = lib.qflash_attention_static(ctypes.c_void_p(ctx.handle), *(x.data_ptr() for x in t), o.data_ptr(),
                                         tb.data_ptr() if tb is not None else None, *(bias_bh or (0, 0)), B, H, N, d, tile,
                                         ctypes.byref(lp), stream)
        assert rc == 0, qf.qflash_strerror(rc)
        done.append((Q, K, V, p, tile, bias, o, (t, tb)))
    torch.cuda.synchronize()
    for Q, K, V, p, tile, bias, o, _ in done:
        assert_same(o.cpu().numpy(), oracle.qflash_attention(Q, K, V, p, tile, bias=bias), "static %s" % (Q.shape,))


# float32 tensors where the quantising kernels run ahead of the attention kernel, which finds constants and table on the GPU
@pytest.mark.parametrize("B,H,N,d,tile,slices", [(40, 6, 197, 64, 64, (1, 6)), (40, 6, 197, 64, 128, (2, 1)), (90, 6, 50, 64, 64, (2, 6)),
                                                 (20, 4, 384, 64, 64, (1, 1)), (20, 4, 300, 64, 128, (2, 4)), (173, 3, 49, 32, 64, (2, 3)),
                                                 (180, 3, 20, 32, 64, None), (48, 3, 100, 32, 128, (1, 3)), (48, 4, 100, 32, 64, None),
                                                 (16, 1, 1100, 32, 64, (1, 1)), (8, 1, 2060, 32, 64, (2, 1)), (15, 4, 289, 64, 64, None)])
@pytest.mark.parametrize("sigma", [0.8, 2.0])
def test_constants_and_table_made_on_the_gpu(gpu, B, H, N, d, tile, slices, sigma):  # noqa: F811
    assert B * H * -(-N // 32) >= BLOCKS
    rng = np.random.default_rng(15000 + N)
    Qf, Kf, Vf = (rng.standard_normal((B, H, N, d), dtype=np.float32) * np.float32(sigma) for _ in range(3))
    bias = mask = None
    if slices is not None:
        bias = (0.5 * rng.standard_normal(slices + (N, N))).astype(np.float32)
        mask = (rng.random(slices + (N, N)) < 0.2).astype(np.uint8)
        mask[0, 0, 1, :] = 1
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, tile, out_round=N % 2, bias_real=bias, excluded=mask)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, tile, out_round=N % 2, bias_real=bias, excluded=mask)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert_same(out, ref, "dynamic %s" % (Qf.shape,))
