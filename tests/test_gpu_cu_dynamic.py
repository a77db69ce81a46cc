"""GPU parity of the whole-compute-unit kernel that quantises float32 tensors on the way in: ragged last pieces and
tiles, one to several pairs per workgroup, a short last workgroup, several rounds of workgroups, with and without a weight table, degenerate scales."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import gpu, run_dynamic  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bhn,gains", [
    ((257, 1, 1), (1.0, 1.0, 1.0)),            # one row: a workgroup of two pairs, the last with one
    ((301, 1, 33), (1.0, 2.0, 1.0)),
    ((700, 3, 64), (1.0, 1.0, 0.01)),          # nine pairs of one tile each
    ((129, 4, 70), (1.3, 1.0, 1.0)),
    ((103, 5, 130), (0.1, 0.5, 3.0)),          # scales too fine for a table
    ((33, 3, 177), (1.0, 1.0, 1.0)),           # one pair per workgroup
    ((86, 3, 200), (30.0, 20.0, 1.0)),         # coarse scales: x_shift > 0
    ((100, 6, 256), (1.0, 1.0, 1.0)),
    ((60, 12, 197), (1.0, 1.0, 1.0))])
def test_whole_compute_unit_from_floats(gpu, bhn, gains):  # noqa: F811
    shape = bhn + (64,)
    rng = np.random.default_rng(8000 + bhn[2])
    Qf, Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) * np.float32(g) for g in gains)
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, 64, out_round=bhn[2] % 2)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, 64, out_round=bhn[2] % 2)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert (inf.sQ, inf.sK, inf.sV) == (rinfo["sQ"], rinfo["sK"], rinfo["sV"])
    assert np.array_equal(out, ref)


@pytest.mark.parametrize("bhn,kv_tile", [
    ((257, 3, 256), 64),             # more pairs than one round holds, by three
    ((190, 10, 100), 128),
    ((230, 16, 65), 64),
    ((1360, 10, 9), 64)])            # many short pairs
def test_several_rounds_from_floats(gpu, bhn, kv_tile):  # noqa: F811
    shape = bhn + (64,)
    rng = np.random.default_rng(8500 + bhn[2])
    Qf, Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) for _ in range(3))
    ref, rinfo = oracle.qflash_attention_dynamic(Qf, Kf, Vf, kv_tile)
    out, inf, _ = run_dynamic(gpu, Qf, Kf, Vf, kv_tile)
    assert inf.status == 0 and inf.params.astuple() == rinfo["params"].astuple()
    assert np.array_equal(out, ref)


def test_whole_compute_unit_from_floats_degenerate(gpu):  # noqa: F811
    torch, qf, ctx = gpu
    shape = (60, 4, 100, 64)
    rng = np.random.default_rng(8)
    Kf, Vf = (rng.standard_normal(shape, dtype=np.float32) for _ in range(2))
    ref, _ = oracle.qflash_attention_dynamic(np.zeros(shape, np.float32), Kf, Vf, 64)
    out, inf, _ = run_dynamic(gpu, np.zeros(shape, np.float32), Kf, Vf, 64)
    assert inf.status == 0 and inf.sQ == 1.0 and np.array_equal(out, ref)
    out, inf, _ = run_dynamic(gpu, Kf * np.float32(1e-6), Kf * np.float32(1e-6), Vf, 64)
    assert inf.status == qf.ERR["PARAM"] and not out.any()
