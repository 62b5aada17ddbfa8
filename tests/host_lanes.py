"""Runs the library's kernels on the CPU, from their source as it is.

SHIM is a small host stand-in for the device language: the threads of a
workgroup are fibers that meet at the workgroup's barriers and at the wave's
exchanges, and launch() runs the workgroups of a grid one after another, in
ascending or descending order (g_descending).  launches() turns kernel launches
in a piece of source into calls of launch()."""

import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_06204_amd", "csrc")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")

SHIM = r"""
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <ucontext.h>
#include <vector>
#define __global__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __restrict__
typedef int hipError_t;
typedef int hipStream_t;
enum { hipSuccess = 0 };
static int hipGetLastError() { return hipSuccess; }
using std::isfinite;
using std::max;
using std::min;
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
#define __align__(n) __attribute__((aligned(n)))
static dim3 blockIdx, blockDim, gridDim, threadIdx;

// Fibers: RUN, at a barrier of the wave, at one of the workgroup, DONE.
enum { RUN, WAVE, GROUP, DONE };
static const int kMaxThreads = 1024;
static ucontext_t g_main, g_ctx[kMaxThreads];
static std::vector<char> g_stack[kMaxThreads];
static int g_state[kMaxThreads], g_tid, g_descending;
static unsigned g_ops[kMaxThreads];
static double g_slot[2][2][kMaxThreads];
static std::function<void()> g_body;
static void block_on(int s) { g_state[g_tid] = s; swapcontext(&g_ctx[g_tid], &g_main); }
static void fiber() { g_body(); g_state[g_tid] = DONE; }
static void __syncthreads() { block_on(GROUP); }
// The values of all 64 lanes of the wave: v, and kMaxThreads words further on v2.
static double* meet(double v, double v2 = 0.0) {
    double* slots = g_slot[g_ops[g_tid]++ & 1][0];
    slots[g_tid] = v;
    slots[kMaxThreads + g_tid] = v2;
    block_on(WAVE);
    return slots + (g_tid & ~63);
}
static double wave_sum(double v) {
    const double* s = meet(v);
    double t = 0.0;
    for (int l = 0; l < 64; ++l) t += s[l];
    return t;
}
static double __shfl_xor(double v, int off, int) { const int l = g_tid & 63; return meet(v)[l ^ off]; }
static double keep_if(double x, int mask) { return mask ? x : 0.0; }
static int opaque(int x) { return x; }
static double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x); }
static double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }

static void run_group(int threads) {
    for (int t = 0; t < threads; ++t) {
        if (g_stack[t].empty()) g_stack[t].resize(32768);
        getcontext(&g_ctx[t]);
        g_ctx[t].uc_stack.ss_sp = g_stack[t].data();
        g_ctx[t].uc_stack.ss_size = g_stack[t].size();
        g_ctx[t].uc_link = &g_main;
        makecontext(&g_ctx[t], fiber, 0);
        g_state[t] = RUN;
        g_ops[t] = 0;
    }
    for (;;) {
        int live = 0;
        for (int w = 0; w < threads; w += 64) {
            for (bool again = true; again;) {
                int at_wave = 0, at_group = 0;
                for (int t = w; t < w + 64; ++t) {
                    if (g_state[t] == RUN) {
                        g_tid = t;
                        threadIdx.x = t;
                        swapcontext(&g_main, &g_ctx[t]);
                    }
                    at_wave += g_state[t] == WAVE;
                    at_group += g_state[t] == GROUP;
                }
                if (at_wave && at_wave != 64) { std::fprintf(stderr, "a wave reduction that not all lanes reach\n"); std::abort(); }
                again = at_wave == 64;
                if (again) for (int t = w; t < w + 64; ++t) g_state[t] = RUN;
                live += again ? 0 : at_group;
            }
        }
        if (live == 0) return;
        for (int t = 0; t < threads; ++t) if (g_state[t] == GROUP) g_state[t] = RUN;
    }
}
template <class F>
static void launch(dim3 grid, int threads, F body) {
    g_body = body;
    gridDim = grid;
    blockDim = dim3(threads);
    const unsigned total = grid.x * grid.y * grid.z;
    for (unsigned i = 0; i < total; ++i) {
        const unsigned b = g_descending ? total - 1 - i : i;
        blockIdx = dim3(b % grid.x, b / grid.x % grid.y, b / grid.x / grid.y);
        run_group(threads);
    }
}
"""


def between(text, first, last):
    i = text.index(first)
    return text[i:text.index(last, i)]


def launches(text, stream="st"):
    text = re.sub(r"\b(\w+(?:<[^<>;]*>)?)<<<(.*?), (\w+), 0, " + stream + r">>>\((.*?)\);",
                  r"launch(\2, \3, [=] { \1(\4); });", text)
    assert "<<<" not in text
    return text
