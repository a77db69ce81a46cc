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
#include "qflash_internal.h"
extern "C" unsigned divide(unsigned n, unsigned d, unsigned* rest) { return qflash_divide(n, d, qflash_reciprocal(d), rest); }
extern "C" int small(int n, unsigned d) { return qflash_small_quotient(n, qflash_small_reciprocal(d)); }
extern "C" unsigned pieces(int N) { static QflashKernelArgs a; a.N = N; a.B = a.H = 1; qflash_cu_reciprocals(&a); return a.cu_inv_per; }
extern "C" void order(int bias, int mask, int bias_B, int bias_H, int B, int H, unsigned* out) {
    static QflashKernelArgs a;
    std::memset(&a, 0, sizeof a);
    static const int32_t some_bias = 0;
    static const uint8_t some_mask = 0;
    a.bias = bias ? &some_bias : nullptr; a.dyn_mask = mask ? &some_mask : nullptr;
    a.bias_B = bias_B; a.bias_H = bias_H; a.B = B; a.H = H;
    qflash_win_order(&a);
    const unsigned all[] = {(unsigned)a.win_rb, (unsigned)a.win_rh, a.win_inv_r, a.win_inv_rh, a.win_inv_bh};
    std::memcpy(out, all, sizeof all);
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


@pytest.mark.parametrize("bias,mask,bias_B,bias_H,B,H", [(1, 0, 4, 3, 12, 6), (0, 1, 4, 1, 4, 5), (1, 1, 1, 6, 7, 6), (0, 0, 1, 1, 5, 3), (0, 0, 9, 9, 5, 3)])
def test_every_pair_once(lib, bias, mask, bias_B, bias_H, B, H):
    out = (ctypes.c_uint * 5)()
    lib.order(bias, mask, bias_B, bias_H, B, H, out)
    if not (bias or mask):
        bias_B = bias_H = 1                        # (extents of no bias count for nothing)
    rb, rh = B // bias_B, H // bias_H
    assert list(out) == [rb, rh] + [(2 ** 32 - 1) // d for d in (rb * rh, rh, bias_H)]
    rest, seen = ctypes.c_uint(), []

    def divide(n, d):
        return lib.divide(n, d, ctypes.byref(rest)), rest.value

    for t in range(B * H):
        s, r = divide(t, rb * rh)
        i, j = divide(r, rh)
        wb, hb = divide(s, bias_H)
        b, h = wb + i * bias_B, hb + j * bias_H
        assert (b % bias_B) * bias_H + h % bias_H == s       # pairs of a slice one after the other
        seen.append(b * H + h)
    assert sorted(seen) == list(range(B * H))
