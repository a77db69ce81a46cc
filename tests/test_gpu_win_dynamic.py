"""GPU parity of the windowed kernel that quantises float32 tensors on the way in and converts the bias: every kind of
bias, one slice per pair and slices shared by long runs, runs that wrap around their ring, short last runs."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import gpu, run_dynamic  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bhn,slices,kind,gains", [
    ((1, 1, 33), (1, 1), "both", (1.0, 1.0, 1.0)),          # a single pair
    ((6, 3, 49), (6, 3), "both", (1.0, 1.0, 1.0)),          # every pair its own slice
    ((60, 5, 50), None, "none", (1.0, 2.0, 1.0)),
    ((40, 12, 64), (4, 12), "mask", (1.0, 1.0, 0.01)),
    ((300, 6, 35), (3, 1), "bias", (2.0, 1.0, 1.0)),        # slices shared by heads
    ((512, 11, 49), (8, 11), "both", (1.0, 1.0, 1.0)),      # six pairs to a run
    ((850, 9, 60), None, "none", (0.15, 0.15, 1.0)),        # eight pairs to a run, no table
    ((1600, 7, 34), (16, 7), "both", (30.0, 20.0, 1.0))])   # eleven
def test_windows_from_floats(gpu, bhn, slices, kind, gains):  # noqa: F811
    N = bhn[2]
    shape = bhn + (32,)
    rng = np.random.default_rng(9000 + N)
    Qf, Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) * np.float32(g) for g in gains)
    bias = mask = None
    if kind in ("both", "bias"):
        bias = (0.5 * rng.standard_normal(slices + (N, N))).astype(np.float32)
    if kind in ("both", "mask"):
        mask = (rng.random(slices + (N, N)) < 0.2).astype(np.uint8)
        mask[0, 0, 1, :] = 1                                # a row without a key
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, 64, out_round=N % 2, bias_real=bias, excluded=mask)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, 64, out_round=N % 2, bias_real=bias, excluded=mask)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert (inf.sQ, inf.sK, inf.sV) == (rinfo["sQ"], rinfo["sK"], rinfo["sV"])
    assert np.array_equal(out, ref)


def test_windows_from_floats_bias_on_the_edge(gpu):  # noqa: F811
    """Bias values half-way between two integers of the score unit, to one float32 rounding, and far beyond the clip."""
    shape = (16, 3, 49, 32)
    rng = np.random.default_rng(9)
    Qf, Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) for _ in range(3))
    unit = (np.abs(Qf).max() / 127.0) * (np.abs(Kf).max() / 127.0) / np.sqrt(32.0)
    k = rng.integers(-3000, 3000, size=(4, 3, 49, 49)).astype(np.float64)
    bias = ((k + 0.5) * unit).astype(np.float32)
    bias[0, 0, :4] *= np.float32(1e6)
    bias[1, 0, :, 3] = np.float32(3e38)
    ref, _ = oracle.qflash_attention_dynamic(Qf, Kf, Vf, 64, bias_real=bias)
    out, _, _ = run_dynamic(gpu, Qf, Kf, Vf, 64, bias_real=bias)
    assert np.array_equal(out, ref)
