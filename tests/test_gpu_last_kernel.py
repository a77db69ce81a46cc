"""What the library says of a call is what the call did: the kernel family and the sharing out of keys that
qflash_cache_query reports after a launch equal what qflash_plan_query said of the shape before it, for every
family, with the weight table and without."""
import numpy as np
import pytest

from tests.test_gpu_parity import gpu, lib_params, rand_case  # noqa: F401
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tile,bias_bh,kernel", [
    ((64, 6, 100, 64), 64, None, 3), ((64, 6, 100, 64), 128, None, 3), ((70, 9, 50, 64), 128, None, 3),
    ((84, 12, 197, 64), 64, None, 3),              # no room for a table
    ((250, 24, 197, 64), 64, None, 1),             # too many pairs for one round
    ((300, 3, 49, 32), 64, None, 4), ((300, 3, 49, 32), 64, (4, 3), 4), ((301, 3, 49, 32), 64, (2, 3), 1),
    ((24, 8, 300, 32), 64, None, 2), ((24, 8, 300, 32), 128, None, 2), ((24, 8, 300, 32), 64, (1, 8), 1),
    ((16, 8, 300, 64), 64, None, 2), ((16, 8, 300, 64), 128, (1, 1), 2), ((16, 8, 300, 64), 64, (1, 1), 1),
    ((1, 4, 2100, 32), 64, (1, 1), 0),             # launches so small that their keys are shared out
    ((1, 3, 197, 64), 64, None, 3), ((1, 1, 2100, 32), 128, None, 2)])
def test_query_tells_what_the_launch_does(gpu, shape, tile, bias_bh, kernel):  # noqa: F811
    torch, qf, ctx = gpu
    Q, K, V, sQ, sK, _ = rand_case(shape, 100 + shape[2])
    p = lib_params(qf, oracle.derive_params(sQ, sK, shape[3]))
    t = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (Q, K, V)]
    o = torch.empty_like(t[0])
    bias = None if bias_bh is None else torch.zeros(bias_bh + (shape[2], shape[2]), dtype=torch.int32, device="cuda:0")
    plan = qf.qflash_plan_query(ctx.handle, *shape, tile, *(bias_bh or (0, 0)))
    assert plan.kernel == kernel, shape
    calls = [lambda: ctx.attention(*t, o, p, tile, bias=bias)]
    if bias is not None:
        packed = ctx.pack_bias(bias)
        calls.append(lambda: ctx.attention_packed_bias(*t, o, p, tile, packed, *bias_bh))
    for call in calls:
        call()
        info = ctx.cache_info()
        assert (info.last_kernel, info.last_key_waves) == (plan.kernel, plan.key_waves), shape
    torch.cuda.synchronize()
