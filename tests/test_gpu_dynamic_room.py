"""GPU parity of dynamic quantisation where the launch has room for some weight tables only: scales on both sides of
the limit, rings of both head sizes and tiles, whole windows in LDS."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import gpu, run_dynamic  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma", [0.5, 0.9, 1.1, 3.0])
@pytest.mark.parametrize("shape,tile,bias", [((12, 12, 300, 64), 64, False), ((12, 12, 300, 64), 128, False),
                                             ((12, 12, 330, 32), 64, False), ((48, 12, 144, 32), 64, True)])
def test_dynamic_with_room_for_some_tables(gpu, shape, tile, bias, sigma):  # noqa: F811
    rng = np.random.default_rng(int(10 * sigma) + shape[2])
    Qf, Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) * np.float32(sigma) for _ in range(3))
    real = (0.5 * rng.standard_normal((4, 12, shape[2], shape[2]))).astype(np.float32) if bias else None
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, tile, bias_real=real)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, tile, bias_real=real)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert np.array_equal(out, ref)
