"""The launch that qflash_plan.cpp lays out for a call of the direct-load ring, with the weight table its constants have:
that file compiled for the host.  (qflash_plan_query knows no constants and assumes a table of its own size.)"""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_25306_amd", "csrc")
SHIM = """
#include <cstring>
#include "qflash_derive.h"
#include "qflash_internal.h"
extern "C" int table_span(int s_inv, int x_shift, int p_mul, int p_shift) { return (int)qflash_table_span(s_inv, x_shift, p_mul, p_shift); }
extern "C" int table_bytes(int s_inv, int x_shift, int p_mul, int p_shift) {
    const long long x_p = qflash_table_span(s_inv, x_shift, p_mul, p_shift);
    return x_p + 16 <= kTableMaxBytes ? qflash_table_bytes((int)x_p) : 0;
}
extern "C" void plan(int B, int H, int N, int d, int tile, int table, int per_head, int qmax, int* out) {
    static QflashKernelArgs a;
    std::memset(&a, 0, sizeof a);
    a.B = B; a.H = H; a.N = N; a.n_cu = 256; a.bias_B = a.bias_H = 1; a.per_head = per_head; a.qmax = qmax;
    const int lds = 160 * 1024;
    const int rc = qflash_plan_family(d, tile, lds, QflashCallKind{}, &table, &a);
    qflash_plan_split(d, lds, table, &a);
    const int all[] = {rc == 0 && a.ring_dma && !a.split_waves, a.waves_per_head, a.n_qtiles, a.n_units, 8 * a.units_per_xcd, a.ring_even_from,
                       (int)qflash_ring_lds_bytes(a.waves_per_head, tile, table, d)};
    std::memcpy(out, all, sizeof all);
}
"""
# ring: the launch runs that kernel; waves: to a workgroup; blocks: workgroups of a pair; even_from: the first one whose wavefronts
# give way to those further behind (grid: none does); lds: bytes of a workgroup
RingPlan = collections.namedtuple("RingPlan", "ring waves blocks units grid even_from lds")


@functools.lru_cache(None)
def _library():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC, src,
                               os.path.join(CSRC, "qflash_plan.cpp"), "-o", out])
        return ctypes.CDLL(out)


def table_span(params):
    """Score difference to the running maximum at which the table begins: its entry 0, of weight 0."""
    return _library().table_span(params.s_inv, params.x_shift, params.p_mul, params.p_shift)


def table_bytes(params):
    """Size of the weight table, 0 where there is none; of several sets of constants the largest."""
    if isinstance(params, (list, tuple)):
        return max(table_bytes(p) for p in params)
    return _library().table_bytes(params.s_inv, params.x_shift, params.p_mul, params.p_shift)


def ring_plan(shape, tile, table, per_head=False, qmax=False):
    out = (ctypes.c_int * 7)()
    _library().plan(*shape, tile, table, int(per_head), int(qmax), out)
    return RingPlan(*out)
