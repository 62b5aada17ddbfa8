"""CPU replay of the GEMM kernels and their launcher (gemm.hip, from the source
as it is): the pipelined FP64 kernel in its three tile shapes and gemm_kernel in
both precisions.

The operands lie against a page that cannot be touched, once at their end and
once at their beginning, so that a load outside an operand ends the run.  What
is no part of an operand (the words between columns, the other triangle of a
triangular operand) holds NaN, which must not reach the result: consumers of
factors whose other triangle is left undefined rely on that.  The entries are
small whole numbers, so the result has to be exact."""

import itertools
import os
import subprocess

import pytest

import host_lanes
from host_lanes import CLANG, CSRC, between

STUBS = r"""
#include <atomic>
#include <mutex>
#include <type_traits>
#include <unordered_map>
#include <cstddef>
#include <cstring>
#include <limits>
#include <sys/mman.h>
enum { hipErrorInvalidValue = 1 };
typedef int hipEvent_t;
static hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
static hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
static hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
static hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
static hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
static hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_s_waitcnt(x)
#define __builtin_amdgcn_s_barrier() __syncthreads()
namespace zolo {
static bool stats_on() { return false; }
struct StatScope {
    StatScope(const char*, hipStream_t, double, double = 0.0) {}
    void end() {}
};
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
template <class T> struct Mfma;
// D = A B + C of a wave: A[l % 16][l / 16] and B[l / 16][l % 16] in lane l.
template <class T, class V>
static V mfma_host(T a, T b, V c) {
    const double* s = meet(a, b);
    const int lane = g_tid & 63;
    for (int e = 0; e < 4; ++e)
        for (int k = 0; k < 4; ++k)
            c[e] += (T)s[Mfma<T>::row(lane, e) + 16 * k] * (T)s[kMaxThreads + (lane & 15) + 16 * k];
    return c;
}
template <> struct Mfma<double> {
    typedef d4 acc;
    static int row(int lane, int e) { return (lane >> 4) + 4 * e; }
    static acc run(double a, double b, acc c) { return mfma_host(a, b, c); }
};
template <> struct Mfma<float> {
    typedef f4 acc;
    static int row(int lane, int e) { return 4 * (lane >> 4) + e; }
    static acc run(float a, float b, acc c) { return mfma_host(a, b, c); }
};
static d4 mfma_f64_16x16x4(double a, double b, d4 c) { return mfma_host(a, b, c); }
"""

DRIVER = r"""
using namespace zolo;
// `count` words that end (at_end) or begin at a page that cannot be touched.
template <class T>
struct Guarded {
    char* base;
    size_t bytes;
    T* p;
    Guarded(long long count, bool at_end) {
        const size_t page = 4096, body = (count * sizeof(T) + page - 1) / page * page;
        bytes = body + 2 * page;
        base = (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        mprotect(base, page, PROT_NONE);
        mprotect(base + page + body, page, PROT_NONE);
        p = (T*)(at_end ? base + page + body - count * sizeof(T) : base + page);
        for (long long i = 0; i < count; ++i) p[i] = std::numeric_limits<T>::quiet_NaN();
    }
    ~Guarded() { munmap(base, bytes); }
};
static unsigned g_seed;
static int entry() { g_seed = g_seed * 1664525u + 1013904223u; return (int)(g_seed >> 20) % 9 - 4; }

// how: 0 the dispatcher, 1 gemm_split, 2 gemm_few, 3..5 the pipelined kernel's tile shapes.
template <class T>
static int run_case(int how, int ta, int tb, int m, int n, int k, int pad, unsigned flags, int batch, int reduce,
                    int batch2, int nalpha, int with_c, bool at_end) {
    g_seed = 1u + m * 131 + n * 17 + k;
    const int ar = ta ? k : m, ac = ta ? m : k, br = tb ? n : k, bc = tb ? k : n, nb = batch * batch2;
    const int nout = (reduce ? 1 : batch) * batch2;
    const long long lda = ar + pad, ldb = br + pad, ldc = m + 1;
    const long long sa = lda * (ac - 1) + ar + pad, sb = ldb * (bc - 1) + br + pad, sc = ldc * n;
    Guarded<T> A(sa * (nb - 1) + lda * (ac - 1) + ar, at_end), B(sb * (nb - 1) + ldb * (bc - 1) + br, at_end);
    Guarded<T> C(sc * (nout - 1) + ldc * (n - 1) + m, at_end);
    const long long room = (long long)32 * nout * m * n;
    Guarded<T> work(room, at_end);
    auto a_at = [&](int b, int i, int q) -> T& { return A.p[b * sa + (ta ? q + i * lda : i + q * lda)]; };
    auto b_at = [&](int b, int q, int j) -> T& { return B.p[b * sb + (tb ? j + q * ldb : q + j * ldb)]; };
    auto a_in = [&](int i, int q) { return !(flags & kAUpper && q < i) && !(flags & kALower && q > i); };
    auto b_in = [&](int q, int j) { return !(flags & kBUpper && q > j) && !(flags & kBLower && q < j); };
    for (int b = 0; b < nb; ++b) {
        for (int i = 0; i < m; ++i) for (int q = 0; q < k; ++q) if (a_in(i, q)) a_at(b, i, q) = (T)entry();
        for (int j = 0; j < n; ++j) for (int q = 0; q < k; ++q) if (b_in(q, j)) b_at(b, q, j) = (T)entry();
    }
    auto stored = [&](int i, int j) { return !(flags & kCStoreUpper && i > j) && !(flags & kCStoreLower && i < j); };
    std::vector<double> want((size_t)nout * m * n);
    for (int o = 0; o < nout; ++o)
        for (int j = 0; j < n; ++j)
            for (int i = 0; i < m; ++i) {
                T& c = C.p[o * sc + i + j * ldc];
                if (with_c && stored(i, j)) c = (T)entry();
                double s = 0.0;
                for (int z = 0; z < (reduce ? batch : 1); ++z) {
                    const int b = reduce ? o * batch + z : o, inner = reduce ? z : o % batch;
                    double t = 0.0;
                    for (int q = 0; q < k; ++q) if (a_in(i, q) && b_in(q, j)) t += (double)a_at(b, i, q) * (double)b_at(b, q, j);
                    s += (nalpha ? inner + 1 : 1) * t;
                }
                want[((size_t)o * n + j) * m + i] = 2.0 * s - (with_c ? 3.0 * (double)c : 0.0);
            }
    GemmDescT<T> d;
    d.m = m; d.n = n; d.k = k; d.transa = ta; d.transb = tb;
    d.A = A.p; d.lda = lda; d.strideA = sa; d.strideA2 = sa * batch;
    d.B = B.p; d.ldb = ldb; d.strideB = sb; d.strideB2 = sb * batch;
    d.C = C.p; d.ldc = ldc; d.strideC = sc; d.strideC2 = sc * (reduce ? 1 : batch);
    if (with_c) {
        d.Cin = C.p; d.ldcin = ldc; d.strideCin = sc; d.strideCin2 = d.strideC2; d.beta = -3.0;
    }
    d.alpha = 2.0; d.batch = batch; d.reduce = reduce; d.batch2 = batch2; d.flags = flags;
    d.nalpha = nalpha ? batch : 0;
    for (int b = 0; b < d.nalpha; ++b) d.alphas[b] = b + 1;
    hipError_t e = hipErrorInvalidValue;
    if (how == 0) e = gemm(d, 0);
    if constexpr (sizeof(T) == 8) {
        if (how == 1) e = gemm_split(d, work.p, room, 0);
        if (how == 2) e = gemm_few(d, work.p, room, 0);
        if (how == 3) e = launch_pipe<64, 128>(d, 0);
        if (how == 4) e = launch_pipe<64, 64>(d, 0);
        if (how == 5) e = launch_pipe<128, 64>(d, 0);
    }
    if (e != hipSuccess) return 2;
    for (int o = 0; o < nout; ++o)
        for (int j = 0; j < n; ++j)
            for (int i = 0; i < m; ++i) {
                const double c = (double)C.p[o * sc + i + j * ldc];
                if (stored(i, j) ? c != want[((size_t)o * n + j) * m + i] : c == c) return 1;
            }
    return 0;
}
int main(int argc, char** argv) {
    int f32, how, ta, tb, m, n, k, pad, batch, reduce, batch2, nalpha, with_c, at_end, bad = 0;
    unsigned flags;
    while (std::scanf("%d %d %d %d %d %d %d %d %u %d %d %d %d %d %d", &f32, &how, &ta, &tb, &m, &n, &k, &pad, &flags, &batch,
                      &reduce, &batch2, &nalpha, &with_c, &at_end) == 15) {
        std::printf("f32=%d how=%d ta=%d tb=%d m=%d n=%d k=%d pad=%d flags=%u batch=%d reduce=%d batch2=%d nalpha=%d c=%d end=%d: ",
                    f32, how, ta, tb, m, n, k, pad, flags, batch, reduce, batch2, nalpha, with_c, at_end);
        std::fflush(stdout);
        const int rc = f32 ? run_case<float>(how, ta, tb, m, n, k, pad, flags, batch, reduce, batch2, nalpha, with_c, at_end)
                           : run_case<double>(how, ta, tb, m, n, k, pad, flags, batch, reduce, batch2, nalpha, with_c, at_end);
        std::printf(rc == 0 ? "ok\n" : rc == 1 ? "WRONG\n" : "REFUSED\n");
        bad += rc != 0;
    }
    std::printf("%d bad\n", bad);
    return bad != 0;
}
"""

A_UPPER, A_LOWER, B_UPPER, B_LOWER, C_TILES, C_UPPER, C_LOWER = 1, 2, 4, 8, 16, 32, 64


def source():
    common = open(os.path.join(CSRC, "common.hpp")).read()
    gemm = open(os.path.join(CSRC, "gemm.hip")).read()
    desc = between(common, "enum GemmFlags", "// ---------------------------------------------------------------------------\n// Small device helpers")
    remap = between(common, "constexpr int kNumXcd", "}  // namespace zolo")
    body = host_lanes.launches(gemm[gemm.index("namespace zolo {") + len("namespace zolo {"):], stream="s")
    return "\n".join([host_lanes.SHIM, STUBS, desc, remap, body, DRIVER])


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    d = tmp_path_factory.mktemp("gemm")
    (d / "gemm.cpp").write_text(source())
    r = subprocess.run([CLANG, "-O0", "-std=c++17", "-w", "-o", str(d / "gemm"), str(d / "gemm.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return str(d / "gemm")


def run(exe, cases):
    """cases: dicts over the defaults below, each with its operands at either end of a page."""
    base = dict(f32=0, how=0, ta=0, tb=0, m=64, n=64, k=64, pad=0, flags=0, batch=1, reduce=0, batch2=1, nalpha=0, c=0)
    lines = [" ".join(str(v) for v in ({**base, **x, "end": end}).values()) for x in cases for end in (0, 1)]
    r = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-600:] + r.stderr[-300:]
    assert r.stdout.count(": ok") == len(lines)


ORIENTATIONS = list(itertools.product((0, 1), (0, 1)))


@pytest.mark.parametrize("how", [3, 4, 5])
def test_pipelined_tiles_at_ragged_sizes(exe, how):
    run(exe, [dict(how=how, ta=ta, tb=tb, m=m, n=n, k=k, pad=pad, c=c) for ta, tb in ORIENTATIONS
              for m, n, k, pad, c in ((2, 2, 16, 0, 0), (3, 65, 17, 1, 1), (65, 3, 31, 0, 1), (129, 131, 33, 0, 0))])


@pytest.mark.parametrize("how", [1, 2])
def test_split_products(exe, how):
    # Along k, over a summed batch (pieces that begin and end inside a matrix of
    # it, odd depths), with triangular operands and upper-tile outputs.
    run(exe, [dict(how=how, ta=ta, tb=tb, m=m, n=n, k=k, batch=b, reduce=red, nalpha=red, c=c)
              for ta, tb in ORIENTATIONS for m, n, k, b, red, c in
              ((65, 3, 401, 1, 0, 1), (33, 66, 131, 3, 1, 0), (2, 17, 513, 2, 0, 1))])
    run(exe, [dict(how=how, ta=1, m=130, n=130, k=389, flags=C_TILES | C_UPPER),
              dict(how=how, tb=1, m=67, n=67, k=150, batch=3, reduce=1, nalpha=1, flags=A_UPPER | B_LOWER | C_TILES | C_UPPER),
              dict(how=how, ta=1, m=64, n=70, k=450, flags=A_UPPER)])


@pytest.mark.parametrize("ta,tb", ORIENTATIONS)
def test_triangular_operands_hold_nan_outside(exe, ta, tb):
    cases = []
    for fa, fb in itertools.product((0, A_UPPER, A_LOWER), (0, B_UPPER, B_LOWER)):
        if fa or fb:
            cases += [dict(ta=ta, tb=tb, m=m, n=n, k=k, flags=fa | fb, c=1)
                      for m, n, k in ((70, 65, 67), (130, 35, 100), (20, 90, 15))]
    run(exe, cases)


def test_gemm_kernel(exe):
    # FP32, k below a slice, single rows and columns, both kinds of triangle.
    run(exe, [dict(f32=1, ta=ta, tb=tb, m=m, n=n, k=k, c=1, flags=f) for ta, tb in ORIENTATIONS
              for m, n, k in ((1, 70, 5), (66, 65, 35)) for f in (0, A_UPPER | B_LOWER, A_LOWER | B_UPPER)])
    run(exe, [dict(ta=ta, tb=tb, m=m, n=n, k=k, c=1, batch=2) for ta, tb in ORIENTATIONS
              for m, n, k in ((1, 9, 40), (9, 1, 40), (65, 3, 15), (1, 1, 1))])


def test_tile_ranges_and_outer_batches(exe):
    # Enough tiles for the balanced ranges of the XCDs and for their remap; a
    # second batch dimension.
    run(exe, [dict(how=0, ta=1, m=385, n=390, k=20, flags=C_TILES | C_UPPER, c=1), dict(m=390, n=390, k=40, flags=A_UPPER),
              dict(m=259, n=330, k=17, tb=1), dict(ta=1, m=66, n=30, k=33, batch=2, batch2=3, pad=1),
              dict(m=40, n=66, k=18, batch=3, reduce=1, batch2=2, nalpha=1, c=1)])
