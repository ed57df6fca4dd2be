"""The library's launch rules (csrc/launch_rules.hpp: host code without HIP), compiled with the
host compiler, so that a test can say which kernel and layout its sizes reach."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2502_17728_amd import build as B

SHIM = r"""
#include "launch_rules.hpp"
using namespace dn;
static int64_t packed(int64_t N, int gated) { return gated ? 2 * ((N + 15) / 16) * 16 : N; }
extern "C" {
int product(int64_t M, int64_t K, int64_t N, int dtype, int gated, int plain) {
    return (int)product_kernel(M, packed(N, gated), K, dtype, gated, plain);
}
int narrow(int64_t M, int64_t N, int gated, int plain) {
    bool narrow;
    plan_256_tiles(M, packed(N, gated), !plain, &narrow);
    return narrow;
}
void streamed(int64_t M, int64_t K, int64_t N, int dtype, int gated, int* rf_nc) {
    const int64_t nblocks = (packed(N, gated) + 15) / 16;
    if (dtype == 0) return plan_f32(M, K, nblocks, gated, rf_nc, rf_nc + 1);
    const SkinnyPlan p = plan_skinny(M, K, nblocks, gated);
    rf_nc[0] = p.rf;
    rf_nc[1] = p.nc;
}
int softmax(int64_t BH, int64_t Lq, int64_t Lk, int64_t d, int causal) { return (int)softmax_layout(BH, Lq, Lk, d, causal); }
int prefill(int64_t BH, int64_t Lq, int64_t Lk, int64_t d, int causal) {
    return kPrefillBQ[prefill_layout(BH, Lq, Lk, d, causal)];
}
int phased(int64_t Lk) { return prefill_phased(Lk); }
void decode(int64_t BH, int64_t Lk, int64_t d, int64_t* units_per_wgs_slots) {
    const DecodePlan p = decode_plan(BH, Lk, d);
    units_per_wgs_slots[0] = p.units;
    units_per_wgs_slots[1] = p.per;
    units_per_wgs_slots[2] = p.wgs;
    units_per_wgs_slots[3] = p.slots;
}
size_t noalloc_partials(int64_t BH, int64_t Lq, int64_t Lk, int64_t d) {
    return attention_decode_partials_bytes(BH, Lq, Lk, d);
}
}
"""
PRODUCT = ("decode", "streamed", "tiles128", "tiles256", "two_stage")
SOFTMAX = ("256", "128", "64", "32", "split")
F32, BF16 = 0, 1


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        open(src, "w").write(SHIM)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-fPIC", "-shared", "-I", B.CSRC, src, "-o", lib])
        lib = ctypes.CDLL(lib)
    i64, i32 = ctypes.c_int64, ctypes.c_int
    lib.product.argtypes = [i64] * 3 + [i32] * 3
    lib.narrow.argtypes = [i64] * 2 + [i32] * 2
    lib.streamed.argtypes = [i64] * 3 + [i32] * 2 + [ctypes.POINTER(i32)]
    lib.softmax.argtypes = lib.prefill.argtypes = [i64] * 4 + [i32]
    lib.phased.argtypes = [i64]
    lib.decode.argtypes = [i64] * 3 + [ctypes.POINTER(i64)]
    lib.noalloc_partials.argtypes, lib.noalloc_partials.restype = [i64] * 4, ctypes.c_size_t
    return lib


def product(M, K, N, dtype=BF16, gated=False, plain=False):
    """The kernel that takes x[M, K] . W[K, N] on packed weights; tiles256 may be 192 wide (tiles256x192)."""
    name = PRODUCT[_lib().product(M, K, N, dtype, gated, plain)]
    return "tiles256x192" if name == "tiles256" and _lib().narrow(M, N, gated, plain) else name


def streamed_plan(M, K, N, dtype=BF16, gated=False):
    """(row fragments, column blocks) of the streamed kernel."""
    out = (ctypes.c_int * 2)()
    _lib().streamed(M, K, N, dtype, gated, out)
    return tuple(out)


def softmax(BH, Lq, Lk, d, causal):
    return SOFTMAX[_lib().softmax(BH, Lq, Lk, d, causal)]


def prefill(BH, Lq, Lk, d, causal):
    """Query rows per workgroup."""
    return _lib().prefill(BH, Lq, Lk, d, causal)


def phased(Lk):
    """256 query rows per workgroup: its halves run one phase apart."""
    return bool(_lib().phased(Lk))


def decode(BH, Lk, d):
    """(units per head, units per workgroup, workgroups, partial slots) of the deal across heads."""
    out = (ctypes.c_int64 * 4)()
    _lib().decode(BH, Lk, d, out)
    return tuple(out)


def noalloc_partials(BH, Lq, Lk, d):
    """Bytes of partials a decode call without a workspace leaves in the library's array."""
    return _lib().noalloc_partials(BH, Lq, Lk, d)
