"""The quotients that kernels make of reciprocals from the host, against Python integers, and the order in which windowed launches
take their pairs with them: every pair once."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_25306_amd", "csrc")
SHIM = """
#include <cstring>
#include "qflash_win_order.h"
extern "C" unsigned divide(unsigned n, unsigned d, unsigned* rest) { return qflash_divide(n, d, qflash_reciprocal(d), rest); }
extern "C" int small(int n, unsigned d) { return qflash_small_quotient(n, qflash_small_reciprocal(d)); }
extern "C" unsigned pieces(int N) { static QflashKernelArgs a; a.N = N; a.B = a.H = 1; qflash_cu_reciprocals(&a); return a.cu_inv_per; }
static QflashKernelArgs launch(int bias, int mask, int bias_B, int bias_H, int B, int H) {
    static QflashKernelArgs a;
    std::memset(&a, 0, sizeof a);
    static const int32_t some_bias = 0;
    static const uint8_t some_mask = 0;
    a.bias = bias ? &some_bias : nullptr; a.dyn_mask = mask ? &some_mask : nullptr;
    a.bias_B = bias_B; a.bias_H = bias_H; a.B = B; a.H = H;
    qflash_win_order(&a);
    return a;
}
// pair, slice and pairs left in the slice of position t, as a run finds them that starts there (from = t) or earlier
extern "C" void walk(int bias, int mask, int bias_B, int bias_H, int B, int H, int from, int n, long long* out) {
    const QflashKernelArgs a = launch(bias, mask, bias_B, bias_H, B, H);
    const WinOrder order(a, bias || mask);
    WinPair p = order.at(from);
    for (int k = 0; k < n; ++k, out += 3) {
        out[0] = order.pair_index(p); out[1] = p.s_idx; out[2] = order.left_in_slice(p);
        if (k + 1 < n) order.advance(p);
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           str(d / "order.cpp"), os.path.join(CSRC, "qflash_plan.cpp"), "-o", str(d / "order.so")])
    so = ctypes.CDLL(str(d / "order.so"))
    so.divide.restype = ctypes.c_uint
    so.divide.argtypes = [ctypes.c_uint, ctypes.c_uint, ctypes.POINTER(ctypes.c_uint)]
    return so


def test_quotients(lib):
    rest = ctypes.c_uint()
    top = 2 ** 32 - 1
    for d in (1, 2, 3, 5, 7, 24, 49, 64, 255, 4096, 65535, 65536, 65537, 3 ** 13, 2 ** 21 - 1, 2 ** 31 - 1, 2 ** 31, top - 1, top):
        near = {m * d + e for m in (0, 1, 2, 3, 1000, top // d - 1, top // d) for e in (-1, 0, 1, d - 1)}
        for n in sorted(x for x in near | {0, 1, 2 ** 16, 2 ** 31, top} if 0 <= x <= top):
            assert (lib.divide(n, d, ctypes.byref(rest)), rest.value) == divmod(n, d), (n, d)


def test_small_quotients(lib):
    for d in range(1, 9):                          # query blocks of at most 256 tokens
        for n in range(65536 // d):
            assert lib.small(n, d) == n // d
    lib.pieces.restype = ctypes.c_uint
    for N in range(1, 257):                        # pieces of sixteen rows of a pair's three tensors: the high word of the product
        per = 3 * ((N + 15) // 16)
        inv = lib.pieces(N)
        assert all(x * inv >> 32 == x // per for x in list(range(64 * per)) + [2 ** 24])


def walk(lib, launch, start, n):
    out = (ctypes.c_longlong * (3 * n))()
    lib.walk(*launch, start, n, out)
    return [tuple(out[3 * k:3 * k + 3]) for k in range(n)]


def expected(bias, mask, bias_B, bias_H, B, H, t):
    """Position t of the order, from what it is meant to be: by slice (window, head of the bias), then batch step, then head step."""
    if not (bias or mask):
        bias_B = bias_H = 1                        # (extents of no bias count for nothing)
    rh, r = H // bias_H, (B // bias_B) * (H // bias_H)
    s, k = divmod(t, r)
    b, h = s // bias_H + k // rh * bias_B, s % bias_H + k % rh * bias_H
    return b * H + h, s, r - k


CASES = [(1, 0, 4, 3, 12, 6), (0, 1, 4, 1, 4, 5), (1, 1, 1, 6, 7, 6), (0, 0, 1, 1, 5, 3), (0, 0, 9, 9, 5, 3), (1, 0, 1, 1, 1, 1), (1, 0, 8, 2, 8, 2),
         (1, 0, 3, 2, 9, 8)]


@pytest.mark.parametrize("launch", CASES)
def test_every_pair_once(lib, launch):
    B, H = launch[4:]
    want = [expected(*launch, t) for t in range(B * H)]
    assert sorted(w[0] for w in want) == list(range(B * H))
    if launch[0] or launch[1]:
        for pair, s, _ in want:                    # the slice is the one the pair's bias lies in
            b, h = divmod(pair, H)
            assert (b % launch[2]) * launch[3] + h % launch[3] == s
    for start in range(B * H):                     # a run may start anywhere, and goes on over the ends of slices
        assert walk(lib, launch, start, B * H - start) == want[start:]


@pytest.mark.parametrize("launch", [(1, 0, 64, 3, 64 * 170000, 24), (1, 0, 65536, 1, 65536 * 16, 30), (0, 0, 0, 0, 2 ** 26 - 5, 31), (1, 0, 1, 7, 3 ** 17, 14)])
def test_positions_of_the_largest_launches(lib, launch):
    T = launch[4] * launch[5]
    assert T < 2 ** 31
    for start in (0, 1, T // 3, T // 2 - 2, T - 9):
        assert walk(lib, launch, start, 9) == [expected(*launch, t) for t in range(start, start + 9)]
