"""Constants of the wrong kind or number are refused before anything is launched: an array of several sets where the
entry point takes one, a buffer that only is as long, arrays of something else.  Refused by the compiled half of
the binding ahead of its look at the tensors, so that no GPU is needed to see it."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2604_25306_amd as qf
from paper_2604_25306_amd import binding

H = 3


def sets():
    return [qf.qflash_params_from_scales(0.04 * (h + 1), 0.04, 0.04, 64) for h in range(H)]


def wrong_as_one():
    ps = sets()
    return [qf.params_array(ps), qf.params_array(ps[:1]), ps, ps[0].astuple(), bytes(ps[0]), bytearray(bytes(ps[0]) * H),
            np.frombuffer(bytes(ps[0]), np.int32), (ctypes.c_int32 * 8)(*ps[0].astuple()), None]


def wrong_as_several():
    one = sets()[0]
    return [(ctypes.c_int32 * (8 * H))(), (ctypes.c_int32 * H)(), ((qf.QFlashParams * 1) * H)(), one]


def calls(ctx, t, bias=None):
    """Every public way to hand over one set of constants, and to hand over several."""
    q, k, v, o = t
    c = qf.Context.__new__(qf.Context)
    c.handle = ctx
    one = [lambda p: qf.qflash_attention(ctx, q, k, v, o, p, 64), lambda p: qf.qflash_attention_static(ctx, q, k, v, o, p, 64),
           lambda p: c.attention_static(q, k, v, o, p, 64),
           lambda p: binding._native().attention(0, ctx, q, k, v, o, p, 64, None, None)]
    several = [lambda p: qf.qflash_attention_per_head(ctx, q, k, v, o, p, 64), lambda p: c.attention(q, k, v, o, p, 64)]
    return one, several


@pytest.fixture(scope="module")
def cpu_layer():
    import torch
    return [torch.zeros((1, H, 8, 64), dtype=torch.int8) for _ in range(4)]


@pytest.mark.parametrize("i", range(9))
def test_one_set_of_constants(cpu_layer, i):
    for call in calls(None, cpu_layer)[0]:
        with pytest.raises(TypeError, match="params must be one QFlashParams"):
            call(wrong_as_one()[i])


@pytest.mark.parametrize("i", range(4))
def test_several_sets_of_constants(cpu_layer, i):
    p = wrong_as_several()[i]
    for call in calls(None, cpu_layer)[1][: 1 if isinstance(p, qf.QFlashParams) else 2]:
        with pytest.raises(TypeError, match="QFlashParams"):
            call(p)
    if not isinstance(p, qf.QFlashParams):
        with pytest.raises(TypeError, match="params must be one QFlashParams or an array of them"):
            qf.qflash_attention_packed_bias(None, *cpu_layer, p, 64, cpu_layer[0], 1, 1)


def test_right_constants_pass_on_to_the_tensor_checks(cpu_layer):
    ps = sets()
    one, several = calls(None, cpu_layer)

    class Named(qf.QFlashParams):
        pass

    for call in one:
        for p in (ps[0], Named(*ps[0].astuple())):
            with pytest.raises(ValueError, match="contiguous int8 CUDA tensor"):
                call(p)
    for call in several:
        for p in (ps, tuple(ps), qf.params_array(ps)):
            with pytest.raises(ValueError, match="contiguous int8 CUDA tensor"):
                call(p)
    for p in (ps[0], ps, qf.params_array(ps)):
        with pytest.raises(ValueError, match="contiguous int8 CUDA tensor"):
            qf.qflash_attention_packed_bias(None, *cpu_layer, p, 64, cpu_layer[0], 1, 1)


@pytest.mark.gpu
def test_nothing_is_launched_with_wrong_constants():
    import torch
    rng = np.random.default_rng(3)
    x = [rng.integers(-127, 128, size=(1, H, 70, 64)).astype(np.int8) for _ in range(3)]
    t = [torch.from_numpy(a).to("cuda:0") for a in x] + [torch.full((1, H, 70, 64), 0x55, dtype=torch.int8, device="cuda:0")]
    with qf.Context(0) as ctx:
        one, several = calls(ctx.handle, t)
        for call in one:
            for p in wrong_as_one():
                with pytest.raises(TypeError):
                    call(p)
        for call in several:
            with pytest.raises(ValueError, match="one QFlashParams per head"):
                call(qf.params_array(sets()[:2]))
        torch.cuda.synchronize()
        assert bool((t[3] == 0x55).all())
        for call, ps in [(c, sets()[:1] * H) for c in one] + [(c, sets()) for c in several]:
            call(ps[0] if call in one else ps)
            torch.cuda.synchronize()
            ref = oracle.qflash_attention(*x, [oracle.params.OracleParams(*p.astuple()) for p in ps], 64)
            assert np.array_equal(t[3].cpu().numpy(), ref)
