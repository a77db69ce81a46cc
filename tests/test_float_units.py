"""The kernels' arithmetic on offset integers and on the single-precision units (csrc/qflash_float_units.h), compiled here
as host code and evaluated with real floats under the kernels' rounding (toward minus infinity, denormals kept), against
Python integers.  The constants come from that file too, so that a change of one of them meets its tests."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include <cfenv>
#include <cmath>
#include "qflash_float_units.h"
#define EACH(N) struct Down { Down() { fesetround(FE_DOWNWARD); } ~Down() { fesetround(FE_TONEAREST); } } down; for (int64_t i = 0; i < (N); ++i)
extern "C" {
int64_t constant(int i) {
    const int64_t c[] = {kAccOffset, kAccBias, kFloatReleaseMaxL, kFloatNormaliseMaxL, kScoreOffset0, kMaskedBiased, kMInit, kIndexScale,
                         score_offset_delta(0), score_offset_delta(1), score_offset_delta(2), score_offset_delta(3)};
    return c[i];
}
void release_float(int64_t n, const int* x, const int* a, int* out) { EACH(n) out[i] = release_acc(x[i] + kAccOffset, make_float_release(a[i])) - kAccOffset; }
void release_int(int64_t n, const int* x, const int* a, int* out) { EACH(n) out[i] = release_acc(x[i] + kAccBias, make_release(a[i])) - kAccBias; }
void release_l_float(int64_t n, const int* l, const int* a, int* out) { EACH(n) out[i] = release_l(l[i], make_float_release(a[i])); }
void release_l_int(int64_t n, const int* l, const int* a, int* out) { EACH(n) out[i] = release_l(l[i], make_release(a[i])); }
void pack(int64_t n, const unsigned* p, unsigned* out) { EACH(n) out[i] = pack_weights(p[4 * i], p[4 * i + 1], p[4 * i + 2], p[4 * i + 3]); }
void index0(int64_t n, const int* s /* biased, block 0 */, const int* edge, unsigned* out) {
    EACH(n) out[i] = float_index(s[i], qf_as_float(kIndexScale), index_addend((unsigned)edge[i]));
}
// what v_cvt_pk_u8_f32 leaves: rounded as the mode says, saturated
static int to_byte(float f) { const float r = std::floor(f); return r < 0.0f ? 0 : r > 255.0f ? 255 : (int)r; }
void quotient(int64_t n, int window, const int* x, const float* r, int* out) {
    EACH(n) out[i] = window ? to_byte(FloatQuotient<kScoreOffset0>(r[i])(x[i] + kScoreOffset0, qf_as_float(FloatQuotient<kScoreOffset0>::kScale)))
                            : to_byte(FloatQuotient<kAccOffset>(r[i])(x[i] + kAccOffset, qf_as_float(FloatQuotient<kAccOffset>::kScale)));
}
}
"""
NAMES = ("acc_offset", "acc_bias", "release_max_l", "normalise_max_l", "score_offset0", "masked", "m_init", "index_scale",
         "delta0", "delta1", "delta2", "delta3")
M32 = (1 << 32) - 1
MAX_N, MAX_XP = 4096, 40960


class Units:
    def __init__(self, so):
        so.constant.restype = ctypes.c_int64
        self.so = so
        for i, name in enumerate(NAMES):
            setattr(self, name, so.constant(i))

    def call(self, name, *args, dtype=np.int32):
        arrays = [np.ascontiguousarray(a) for a in args if isinstance(a, np.ndarray)]
        n = len(arrays[-1])
        out = np.empty(n, dtype)
        pointers = [a.ctypes.data_as(ctypes.c_void_p) for a in arrays] + [out.ctypes.data_as(ctypes.c_void_p)]
        getattr(self.so, name)(ctypes.c_int64(n), *[a for a in args if not isinstance(a, np.ndarray)], *pointers)
        return out


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("units")
    (d / "units.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-frounding-math", "-ffp-contract=off", "-fwrapv", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_25306_amd", "csrc"),
                           str(d / "units.cpp"), "-o", str(d / "units.so")])
    return Units(ctypes.CDLL(str(d / "units.so")))


def factors(rng, n):
    a = rng.integers(0, 65537, size=n)
    a[: n // 8] = 65536
    a[n // 8: n // 4] = 65536 - rng.integers(0, 4, size=n // 4 - n // 8)
    a[-6:] = [0, 1, 2, 32767, 32768, 65535]
    return a.astype(np.int32)


def test_scale_release(units):
    """floor(x alpha16 / 2^16): on floats within the offset, on integers for |x| < 2^26; the denominator likewise."""
    rng = np.random.default_rng(6)
    n = 1 << 20
    a = factors(rng, n)
    for name, top in (("release_float", units.acc_offset), ("release_int", 1 << 26)):
        x = rng.integers(-top + (name == "release_int"), top, size=n).astype(np.int32)
        x[:: 4] >>= rng.integers(0, 24, size=len(x[:: 4]))                  # magnitudes of every order
        x[:4] = [0, -1, top - 1, -top + 1]
        x[n // 8: n // 8 + 4] = [0, -1, top - 1, -top + 1]
        assert np.array_equal(units.call(name, x, a), (x.astype(np.int64) * a) >> 16), name
    for name, top in (("release_l_float", 1 << 24), ("release_l_int", 1 << 20)):
        l = rng.integers(0, top, size=n).astype(np.int32)
        l[:3] = [0, 1, top - 1]
        assert np.array_equal(units.call(name, l, a), (l.astype(np.int64) * a) >> 16), name


def test_every_factor_at_the_ends_of_the_offset(units):
    a = np.arange(65537, dtype=np.int32)
    for x in (0, 1, -1, units.acc_offset - 1, -units.acc_offset, 4711, -4711):
        xs = np.full(len(a), x, np.int32)
        assert np.array_equal(units.call("release_float", xs, a), (xs.astype(np.int64) * a) >> 16), x


def test_range_of_the_numerator(units):
    """|x| <= 128 l + 129 per tile, whatever the weights, values and factors: below the limit of l the offset holds it, over
    every tile of the longest sequence, and always where a sequence has 256 keys at most."""
    assert 128 * units.release_max_l + 129 * (MAX_N // 64) < units.acc_offset and 128 * 127 * 256 + 129 * 4 < units.acc_offset
    rng = np.random.default_rng(7)
    for _ in range(300):
        l = x = 0
        for t in range(64):
            a = int(rng.integers(0, 65537)) if rng.random() < 0.5 else 65536 - int(rng.integers(0, 4))
            s = int(rng.integers(0, 127 * 64 + 1))
            v = int(rng.choice([-128, 127, int(rng.integers(-128, 128))]))
            l, x = ((l * a) >> 16) + s, ((x * a) >> 16) + s * v
            assert abs(x) <= 128 * l + 129 * (t + 1)


def test_pack_weights(units):
    """Every three weights below 128 in the bytes that two multiply-adds make, any in the last one."""
    w = np.arange(128, dtype=np.uint32)
    p = np.stack([*np.meshgrid(w, w, w, indexing="ij"), np.zeros((128, 128, 128), np.uint32)], axis=-1).reshape(-1, 4)
    p[:, 3] = np.random.default_rng(8).integers(0, 128, size=len(p))
    want = p[:, 0] | p[:, 1] << 8 | p[:, 2] << 16 | p[:, 3] << 24
    out = np.empty(len(p), np.uint32)
    units.so.pack(ctypes.c_int64(len(p)), p.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p))
    assert np.array_equal(out, want)


def test_score_offsets(units):
    """Each block of 32 keys carries a constant the instruction set has built in.  Taking a block's own offset out of its
    maximum and adding it to the table edge gives the maximum and the index of the common offset; a key beyond the sequence
    is below every score and every edge, and nothing wraps."""
    off, deltas = units.acc_bias, (units.delta0, units.delta1, units.delta2, units.delta3)
    for d, f in zip(deltas, (np.float32(1 / (2 * np.pi)), 2.0, 4.0, 1.0)):
        assert int(np.array(f, np.float32).view(np.uint32)) == off + d
    assert off + units.delta0 == units.score_offset0
    lowest = units.m_init - MAX_XP                          # the lowest edge: the first maximum less the longest table
    assert off + lowest > units.masked and units.m_init == -(1 << 21)
    rng = np.random.default_rng(11)
    for _ in range(20000):
        x_p = int(rng.integers(1, MAX_XP + 1))
        scores = [int(v) for v in rng.integers(-(1 << 21) + 1, 1 << 21, size=4)]
        m = int(rng.integers(max(scores), 1 << 21))
        edge = (m + off - x_p) & M32
        top = []
        for s, d in zip(scores, deltas):
            sb, masked, edge_kb = (s + off + d) & M32, units.masked + d, (edge + d) & M32
            assert 0 <= masked < sb < 1 << 32
            assert max(0, sb - edge_kb) == max(0, s - m + x_p) and max(0, masked - edge_kb) == 0
            top.append((max(sb, masked) - d) & M32)
        assert max(top) == max(scores) + off


def test_float_index(units):
    """max(0, score - edge) of block 0, which lies in one binade, [1/8, 1/4), with every score and edge; at the edge, beside it,
    and for a key beyond the sequence."""
    lo, hi = units.score_offset0 + units.m_init - MAX_XP, units.score_offset0 + (1 << 21)
    assert 0x3E000000 <= units.masked + units.delta0 < lo and hi < 0x3E800000
    assert np.array([units.index_scale], np.uint32).view(np.float32)[0] == np.float32(2.0) ** -123
    rng = np.random.default_rng(12)
    n = 1 << 20
    x_p = rng.integers(1, MAX_XP + 1, size=n)
    x_p[: n // 4] = MAX_XP
    m = rng.integers(units.m_init, 1 << 21, size=n)
    m[:: 64], m[1:: 64] = units.m_init, (1 << 21) - 1
    s = np.maximum(m - rng.integers(0, 2 * MAX_XP, size=n), units.m_init)
    near = slice(n // 2, None)
    s[near] = (m - x_p)[near] + rng.integers(-2, 3, size=n - n // 2)        # the edge itself and beside it
    s = np.clip(s, units.m_init - MAX_XP, (1 << 21) - 1)
    edge = (m + units.acc_bias - x_p).astype(np.int64)
    got = units.call("index0", (s + units.score_offset0).astype(np.int32), edge.astype(np.int32), dtype=np.uint32)
    assert np.array_equal(got, np.maximum(0, s - (m - x_p)))
    beyond = np.full(n, units.masked + units.delta0, np.int32)
    assert not units.call("index0", beyond, edge.astype(np.int32), dtype=np.uint32).any()


def reciprocals(l):
    """The floats at most one unit in the last place from 1 / l."""
    exact = 1.0 / l.astype(np.float64)
    near = exact.astype(np.float32)
    ulp = np.spacing(np.where(near > exact, np.nextafter(near, np.float32(0)), near)).astype(np.float64)
    for r in (near, np.nextafter(near, np.float32(2)), np.nextafter(near, np.float32(0))):
        yield np.where(np.abs(r.astype(np.float64) - exact) <= ulp, r, near)


@pytest.mark.parametrize("window", [0, 1])
def test_normalisation(units, window):
    """floor(x / l) saturated, for every l the float form is used for and every reciprocal within one unit in the last place,
    at every whole quotient and one off it, and at the largest numerators."""
    # a reciprocal off by 2^-23 moves a quotient of 128 by less than its distance from an integer, 1 / (2 l); sequences of
    # 256 keys are never tested for the limit
    assert 127 * 256 <= units.normalise_max_l and 2 * units.normalise_max_l * 128 < 1 << 23
    l = np.arange(1, (64 * 127 if window else units.normalise_max_l) + 1, dtype=np.int64)
    top = (1 << 20) - 1 if window else units.acc_offset - 1
    for k in [-129, -128, -127, -126, -65, -64, -63, -33, -2, -1, 0, 1, 2, 31, 63, 64, 65, 95, 125, 126, 127, 128, 129]:
        for off in (-1, 0, 1):
            x = np.clip(k * l + off, -top, top)
            want = np.clip(x // l, -128, 127) + 128
            for r in reciprocals(l):
                assert np.array_equal(units.call("quotient", window, x.astype(np.int32), r.astype(np.float32)), want), (k, off)
    assert units.call("quotient", window, np.zeros(1, np.int32), np.zeros(1, np.float32))[0] == 128      # no key: output 0
