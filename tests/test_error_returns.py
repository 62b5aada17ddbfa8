"""CPU test of zolo_pd's error returns: the solver's host code (zolo_pd.cpp and
coeffs.cpp, as they are) on a HIP runtime and kernels made of stubs.  Work is
queued per stream and done when the stream is waited for, as on a GPU, and the
stubs report a launch error where the test asks for one."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_06204_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

STUBS = r"""
#include "CSRC/learn.hpp"
#include "CSRC/misc.hpp"
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <vector>

static std::map<hipStream_t, std::vector<std::function<void()>>> g_queue;
static int g_fail_orgqr = 0, g_raise_panel = 0;
static long g_streams = 0;
static std::mutex g_mu;
static void push(hipStream_t s, std::function<void()> f) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_queue[s].push_back(std::move(f));
}
static void drain(hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_mu);
    for (auto& f : g_queue[s]) f();
    g_queue[s].clear();
}
extern "C" void stub_set(int fail_orgqr, int raise_panel) {
    g_fail_orgqr = fail_orgqr;
    g_raise_panel = raise_panel;
}
extern "C" int stub_pending() {
    int n = 0;
    for (auto& q : g_queue) n += (int)q.second.size();
    return n;
}
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(++g_streams * 16); return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t* s) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { drain(s); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)16; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    push(st, [=] { std::memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
    return hipSuccess;
}
}
namespace zolo {
int panel_max_coresident() { return 256; }
hipError_t open_cooperative_queue(int, hipStream_t) { return hipSuccess; }
hipError_t scratch_address(int, char** p) { *p = nullptr; return hipSuccess; }
hipError_t scale_copy(int, int, const double*, long long, double*, long long, double, int*, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t shift_copy(int, const T*, long long, T*, long long, long long, const ShiftArgs&, hipStream_t) { return hipSuccess; }
template hipError_t shift_copy<double>(int, const double*, long long, double*, long long, long long, const ShiftArgs&, hipStream_t);
template hipError_t shift_copy<float>(int, const float*, long long, float*, long long, long long, const ShiftArgs&, hipStream_t);
hipError_t stack_init(int, int, const double*, long long, double*, long long, long long, const double*, int, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t symmetrize(int, const T*, long long, T*, long long, int, double, hipStream_t) { return hipSuccess; }
template hipError_t symmetrize<double>(int, const double*, long long, double*, long long, int, double, hipStream_t);
template hipError_t symmetrize<float>(int, const float*, long long, float*, long long, int, double, hipStream_t);
hipError_t fill_vector(int, double*, double, hipStream_t) { return hipSuccess; }
hipError_t mlp_forward(int, const float*, const double*, const int*, const MlpBufs&, hipStream_t) { return hipSuccess; }
hipError_t norm1_upper(int, const double*, long long, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t power_steps(int, int, const double*, long long, int, double*, double*, double*, double*, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t trtri_batched(int, const T*, long long, long long, T*, long long, long long, int, T*, long long, hipStream_t) { return hipSuccess; }
template hipError_t trtri_batched<double>(int, const double*, long long, long long, double*, long long, long long, int, double*, long long, hipStream_t);
hipError_t sketch_features(int, int, const double*, long long, unsigned long long, double*, double*, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t potrf_inverse_batched(int, T*, long long, long long, T*, long long, long long, int, int*, T*, long long, hipStream_t) { return hipSuccess; }
template hipError_t potrf_inverse_batched<double>(int, double*, long long, long long, double*, long long, long long, int, int*, double*, long long, hipStream_t);
template hipError_t potrf_inverse_batched<float>(int, float*, long long, long long, float*, long long, long long, int, int*, float*, long long, hipStream_t);
hipError_t gemm(const GemmDesc&, hipStream_t) { return hipSuccess; }
hipError_t gemm(const SGemmDesc&, hipStream_t) { return hipSuccess; }
hipError_t gemm_few(const GemmDesc&, double*, size_t, hipStream_t) { return hipSuccess; }
hipError_t frob2(int, int, const double*, long long, const double*, long long, double*, double* out, hipStream_t st) {
    push(st, [=] { out[0] = 0.0; out[1] = 1.0; });
    return hipSuccess;
}
hipError_t orth2(int, const double*, long long, double*, double* out, hipStream_t st) {
    push(st, [=] { *out = 0.0; });
    return hipSuccess;
}
template <class S, class D>
hipError_t convert(int, int, const S*, long long, D*, long long, double, hipStream_t) { return hipSuccess; }
template hipError_t convert<double, float>(int, int, const double*, long long, float*, long long, double, hipStream_t);
template hipError_t convert<float, double>(int, int, const float*, long long, double*, long long, double, hipStream_t);
hipError_t assemble_r(int, const double*, long long, long long, int, const QrWork&, double*, long long, long long, hipStream_t) { return hipSuccess; }
// A panel whose bounded wait gives up raises the solve's flag when it runs.
hipError_t structured_geqrf(int, int, int, double*, long long, long long, int, const QrWork& w, hipStream_t st) {
    int* flag = w.error_flag;
    const int raise = g_raise_panel;
    auto panel = [=] { if (raise) *flag = 1; };
    push(st, panel);
    if (w.side_stream) push(w.side_stream, [] {});
    if (w.panel_stream) push(w.panel_stream, panel);
    return hipSuccess;
}
hipError_t structured_orgqr(int, int, int, double*, long long, long long, int, const QrWork&, hipStream_t) {
    return g_fail_orgqr ? hipErrorLaunchFailure : hipSuccess;
}
}
"""

DRIVER = r"""
#include "INCLUDE/zolo.h"
#include <vector>
extern "C" int run(zolo_handle h, int n, int batched) {
    std::vector<double> A((size_t)n * n), Q((size_t)n * n), H((size_t)n * n);
    const double* a[2] = {A.data(), A.data()};
    double* q[2] = {Q.data(), Q.data()};
    double* hh[2] = {H.data(), H.data()};
    const int nn[2] = {n, n}, r[2] = {1, 1};
    const double alpha[2] = {1.0, 1.0}, l[2] = {1e-8, 1e-8};
    zolo_opts o;
    zolo_default_opts(&o);
    o.batch_streams = 2;
    if (batched) return zolo_pd_batched(h, 2, nn, nn, a, nn, alpha, l, r, q, nn, hh, nn, &o, nullptr);
    return zolo_pd(h, n, n, a[0], n, 1.0, 1e-8, 1, q[0], n, hh[0], n, nullptr, nullptr);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("err")
    (d / "stubs.cpp").write_text(STUBS.replace("CSRC", CSRC))
    (d / "driver.cpp").write_text(DRIVER.replace("INCLUDE", os.path.join(ROOT, "include")))
    objs = []
    for src in (os.path.join(CSRC, "zolo_pd.cpp"), os.path.join(CSRC, "coeffs.cpp"), str(d / "stubs.cpp"), str(d / "driver.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        r = subprocess.run([HIPCC, "-xhip", "--cuda-host-only", "-O1", "-std=c++17", "-w", "-fPIC", "-c", src, "-o", objs[-1]],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    r = subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", str(d / "err.so"), *objs, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(str(d / "err.so"))


HIP, CONVERGED = 4, 0


@pytest.mark.parametrize("n", [8, 520])           # without and with the look-ahead's stream
def test_launch_error_leaves_nothing_queued(lib, n):
    h = ctypes.c_void_p()
    assert lib.zolo_create(ctypes.byref(h), None) == 0
    lib.stub_set(0, 0)
    assert lib.run(h, n, 0) == CONVERGED
    # A panel that will raise the flag is queued when a later launch fails.
    lib.stub_set(1, 1)
    assert lib.run(h, n, 0) == HIP
    assert lib.stub_pending() == 0
    # The next call does not see that flag.
    lib.stub_set(0, 0)
    assert lib.run(h, n, 0) == CONVERGED
    assert lib.zolo_destroy(h) == 0


def test_launch_error_of_many_matrices(lib):
    h = ctypes.c_void_p()
    assert lib.zolo_create(ctypes.byref(h), None) == 0
    lib.stub_set(1, 1)
    assert lib.run(h, 8, 1) == HIP
    assert lib.stub_pending() == 0
    lib.stub_set(0, 0)
    assert lib.run(h, 8, 1) == CONVERGED
    assert lib.zolo_destroy(h) == 0
