"""The span of the weight table (largest score difference that can carry a weight) as qflash_table_span in
csrc/qflash_derive.h computes it, compiled here as host code, enumerated against Algorithm 2 and Eq. 10 in Python
integers: for constants from real scales, where it is exact, and for others the library accepts, where it may
fall back to eight octaves but must never cut off a weight."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import paper_2604_25306_amd as qf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "qflash_derive.h"
extern "C" long long span(int s_inv, int x_shift, int p_mul, int p_shift) { return qflash_table_span(s_inv, x_shift, p_mul, p_shift); }
extern "C" int accepted(const qflash_params* p) { return qflash_params_ok(*p); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("span")
    (d / "span.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2604_25306_amd", "csrc"), str(d / "span.cpp"), "-o", str(d / "span.so")])
    so = ctypes.CDLL(str(d / "span.so"))
    so.span.restype = ctypes.c_longlong
    so.accepted.argtypes = [ctypes.POINTER(qf.QFlashParams)]
    return so


def weight(x, p):
    xs = x << p.x_shift
    q = (xs * p.exp_mul) >> 32
    r = xs + q * p.s_inv
    y = np.where(q > 31, 0, ((r >> 1) + p.s_inv) >> np.minimum(q, 31))
    return np.minimum(127, (y * p.p_mul) >> p.p_shift)


def weights_down(p, octaves):
    return weight(-np.arange(0, octaves * p.s_inv // (1 << p.x_shift) + 2, dtype=np.int64), p)


def eight_octaves(p):
    return -(-8 * p.s_inv >> p.x_shift)


def is_exact(p):
    """The condition under which the exact formula holds (the comment at qflash_table_span)."""
    y1 = -(-(1 << p.p_shift) // p.p_mul)
    return 1274 * y1 >= 10 * p.s_inv and 128 * y1 <= 2 * p.s_inv


@pytest.mark.parametrize("seed", range(6))
def test_span_is_exact(lib, seed):
    rng = np.random.default_rng(seed)
    for _ in range(60):
        s_real = float(10 ** rng.uniform(-2.2, 0.9))
        try:
            p = oracle.derive_params(s_real, float(10 ** rng.uniform(-2.2, 0.9)), 64)
        except ValueError:
            continue
        x_p = lib.span(p.s_inv, p.x_shift, p.p_mul, p.p_shift)
        w = weights_down(p, 21)
        assert is_exact(p) and w[x_p:].max() == 0 and w[x_p - 1] > 0, p
        assert x_p <= eight_octaves(p)


@pytest.mark.parametrize("seed", range(4))
def test_span_of_constants_not_from_real_scales(lib, seed):
    """Requantisation multipliers the library accepts but no scale gives: smaller ones, whose weights end before
    octave 6 (or, with a largest weight of 0, nowhere), and the few larger ones; exp_mul off by up to 0.09 %."""
    rng = np.random.default_rng(100 + seed)
    short = fallen_back = 0
    for _ in range(400):
        s_inv = int(round(2 ** rng.uniform(10, 14.5)))
        x_shift = int(rng.integers(0, 4))
        p_shift = int(rng.integers(8, 25))
        most = min(((128 << p_shift) - 1) // s_inv, ((1 << 23) - 1) >> (24 - p_shift))
        if most < 1:
            continue
        low = max(1, int(most * (0.995 if rng.integers(2) else 2.0 ** -rng.uniform(0, 7))))
        p_mul = int(rng.integers(low, most + 1))
        exp_mul = -int(round((1 << 32) / s_inv * (1.0 + rng.uniform(-0.0009, 0.0009))))
        p = qf.QFlashParams(x_shift, s_inv, exp_mul, 32, p_mul, p_shift, -(-(1 << 30) // s_inv), 0)
        if not lib.accepted(ctypes.byref(p)):
            continue
        x_p = lib.span(s_inv, x_shift, p_mul, p_shift)
        w = weights_down(p, 21)
        assert w[x_p:].max() == 0, p                 # nothing is cut off, whatever the branch
        if is_exact(p):
            short += 1
            assert x_p < eight_octaves(p), p
        else:
            fallen_back += 1
            assert x_p == eight_octaves(p), p
    assert short > 20 and fallen_back > 20
