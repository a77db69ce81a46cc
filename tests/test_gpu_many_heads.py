"""Bias slices of a launch with more heads than 2^24: the kernels divide by the number of heads, as integers, and that
must not depend on the rounding mode they set for their single-precision arithmetic."""
import pytest

from workloads import EXCLUDED

pytestmark = pytest.mark.gpu


# 34359739: a reciprocal that is one unit in the last place too large, of this number rounded down to 24 bits, gives a
# first guess above 2^32 / 34359739, from which integer division does not recover.  The other: a power of two and a bit.
@pytest.mark.parametrize("H,bias_H", [(34359739, 34359739), (2 * 16777219, 16777219)])
def test_one_token_many_heads(H, bias_H):
    import torch
    import paper_2604_25306_amd as qf
    print("heads", H, "slices", bias_H, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    x = torch.randint(-128, 128, (1, H, 1, 32), generator=gen, device=dev, dtype=torch.int8)
    bias = torch.randint(-9, 9, (1, bias_H, 1, 1), generator=gen, device=dev, dtype=torch.int32)
    bias[torch.rand(bias.shape, generator=gen, device=dev) < 0.5] = int(EXCLUDED)
    out = torch.full_like(x, 0x55)
    with qf.Context(0) as ctx:
        p = qf.qflash_params_from_scales(0.02, 0.02, 0.02, 32)
        ctx.attention(x, x, x, out, p, 64, bias=bias)
        torch.cuda.synchronize()
    # one key: its value, or 0 where it is excluded
    x[bias.repeat(1, H // bias_H, 1, 1).expand(x.shape) == int(EXCLUDED)] = 0
    assert torch.equal(out, x)
