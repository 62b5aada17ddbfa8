// Structured Householder QR of the stacked matrices M_b = [Y_b; p_b I]
// ((m + n) x n, the [X; sqrt(c_{2j-1}) I] of eq. (12)) for all b at once, and
// the plain Householder QR of an m x n matrix (no identity block), on gfx950.
//
// Structure (Section 3.1 of the paper).  Reflector k pivots on row k of the
// dense block; below the pivot it touches the dense rows k+1..m-1 and the
// identity-block rows m..m+k (the identity block fills in upper triangular as
// the factorisation proceeds).  With M stored as one column-major array, a
// block of NB = 64 reflectors starting at column p0 therefore lives on the
// contiguous rows [p0, m + p0 + NB): m + NB live rows instead of the m + n - p0
// of a dense QR.  The identity rows stay below the dense rows on purpose:
// pivoting on the small rows p I first (identity block on top) loses row-wise
// backward stability when p is tiny, e.g. 1e-10 backward error at kappa = 1e8.
//
// Panel: one launch per panel factors all b together (a cooperative launch
// when a matrix takes more than one workgroup).  Each matrix gets G
// workgroups, each owning a slab of the panel's live rows.  The panel's 64
// columns are factored in leaves of 16, held in registers.  Per column one
// reduction over the rows gives the norm, the update coefficients of the
// leaf's remaining columns and the products with the leaf's earlier
// reflectors (compact WY, Q = I - V T V^T).  At the end of a leaf one MFMA
// reduction and one exchange give V_leaf^T times the other panel columns,
// from which the panel's T is formed and the rest of the panel takes the
// leaf's block reflector.  Every reduction sums partials in a fixed order; its barrier
// waits a bounded time.  On exit the panel's top block holds V explicitly
// (unit diagonal, zeros above) and the R diagonal block is saved apart.
//
// Trailing update and Q formation are GEMMs on the MFMA kernel over the live
// rows:  W = V^T C,  W2 = T^T W,  C -= V W2  (ORGQR: T instead of T^T, last
// to first, then a panel's own columns = [I; 0] - V (T V_top^T)).  Panels
// come in pairs (blocks) and pairs of blocks (superblocks): the second panel
// is updated by the first, the second block by the first, and the rest of
// the matrix by all four panels at once with the compact-WY factor of the
// product, merged pairwise as T = [T1, -T1 V1^T V2 T2; 0, T2], so each
// trailing element is read and written once per 256 columns (stored R
// entries that sit above a later panel's diagonal are masked out of V by the
// GEMM's triangular flags).
#include "misc.hpp"
#include "stats.hpp"

#include <type_traits>
#include <algorithm>
#include <mutex>

namespace zolo {
namespace {

constexpr int kNB = kPanelNB;
constexpr int kLW = 16;                  // leaf width: columns factored one exchange at a time
constexpr int kNL = kNB / kLW;           // leaves per panel
constexpr int kOther = kNB - kLW;        // panel columns outside one leaf
constexpr int kPT = 512;                 // threads per panel workgroup
constexpr int kRG = kPT / 64;            // row groups: every wave owns the leaf's columns over its rows
// Exchanges of one panel: one per column and one at the end of each leaf.
constexpr int kPanelExchanges = kNB + kNL;
static_assert(kLW * kOther == kPanelSlot, "exchange slot sized for the leaf-end sums");
// panel_kernel: slab rows per lane loaded together in the column sweep
// (latency of L2), and rows per lane step of its leaf-end MFMA reduction.
constexpr int kRowUnroll = 2;
constexpr int kQuadUnroll = 16;
// Cache-policy operand of a buffer load that makes it coherent at agent
// scope (sc1 on gfx950), and the fourth word of a raw buffer resource.
constexpr int kCoherentLoad = 16;
constexpr int kBufferRsrcWord3 = 0x00020000;
// s_waitcnt immediate (gfx9 encoding) that waits for vmcnt == 0 only:
// vmcnt bits [3:0],[15:14] = 0, expcnt [6:4] = 7, lgkmcnt [11:8] = 15.
constexpr int kWaitVmcnt0 = 0x0F70;

struct PanelArgs {
    int L, nb, G, rows_per_wg;
    int batch, local;                    // local: each matrix's workgroups on one XCD (register-leaf kernel)
    double* P; long long ld, sp;         // panel top-left (row p0, column p0) of matrix 0
    double* T; long long st;             // T_b, kNB x kNB column-major
    double* Rd; long long srd;           // R diagonal block out, kNB x kNB
    double* partials;                    // [batch][2][G][kPanelSlot]: leaf-end sums
    unsigned* flags;                     // [batch][G]: last exchange each workgroup published
    unsigned long long* colslots;        // [batch][2][G][4 kLW]: tagged column sums (register-leaf kernel)
    unsigned seq;                        // exchange x of this panel is published as seq + x + 1 (columns 0..63, then leaf ends)
    int* error_flag;
    unsigned spin_limit;
};

// A wave-uniform double moved to scalar registers.
__device__ inline double uniform(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// One level of the transposing butterfly: lanes with bit OFF set keep the
// upper HALF of their values, the others the lower, each adding its
// partner's copy of the kept half (compile-time indices keep h in registers).
template <int HALF, int OFF>
__device__ inline void butterfly_step(double (&h)[16], int lane) {
    const bool upper = (lane & OFF) != 0;
#pragma unroll
    for (int j = 0; j < HALF; ++j) {
        const double keep = upper ? h[j + HALF] : h[j];
        const double send = upper ? h[j] : h[j + HALF];
        h[j] = keep + __shfl_xor(send, OFF, 64);
    }
}

// Blocked panel for matrices too tall for the register-leaf kernel below: any
// number of rows per workgroup, the slab in global memory.  The panel's columns
// are factored in leaves of kLW = 16.  Inside a leaf, column k takes one sweep over the slab's rows that applies
// reflector k-1 to the leaf's later columns and accumulates the dot products
// of column k below its pivot with the leaf's 16 columns, then one exchange
// of those 16 sums and of the pivot row's 16 entries, which give the norm,
// the update coefficients of the leaf's later columns and the next column of
// the leaf's own compact-WY factor T_s.  At the end of a leaf, one MFMA
// reduction over the rows forms W = V_s^T [V_prev, C] (V_s: the leaf's
// reflectors; V_prev: the earlier leaves'; C: the later columns of the
// panel), one exchange sums it over the workgroups, the first workgroup
// merges T = [T1, -T1 (V_prev^T V_s) T_s; 0, T_s], and every workgroup
// applies the leaf's block reflector to C:  C -= V_s (T_s^T (V_s^T C)).
// Against one sweep of all 64 columns per column, this sweeps 16 columns per
// column and the whole panel twice per leaf.
__global__ __launch_bounds__(kPT) void panel_kernel(PanelArgs a) {
    __shared__ double s_T[kNB * (kNB + 1) / 2];  // upper T packed by columns: T[i][l] at l (l + 1) / 2 + i
    // Leaf-end sums W[i][q] at i * kOther + q (i: leaf column, q: other
    // column, the earlier leaves' columns first).  While a leaf's columns
    // are factored, its first kRG * kLW entries hold each wave's column sums.
    __shared__ double s_W[kLW * kOther];
    __shared__ double s_coef[kLW], s_z[kLW];
    __shared__ double s_rfl[4];          // beta, tau, scale of the latest reflector
    double* const s_wp = s_W;
    const int g = blockIdx.x % a.G, b = blockIdx.x / a.G;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const long long ld = a.ld;
    double* __restrict__ P = a.P + b * a.sp;
    const int r0 = g * a.rows_per_wg;
    const int r1 = min(a.L, r0 + a.rows_per_wg);
    const int nb = a.nb;
    const long long xld = ld;
    double* __restrict__ X = P + r0;
    constexpr int S = 64 * kRG;          // row stride of a lane
    const int first = r0 + 64 * wv + lane;  // this thread's rows: first + S j
    unsigned* flg = a.flags + (long long)b * a.G;
    unsigned ex = 0;  // exchanges done in this panel

    // Sums cnt values of src over the matrix's workgroups into dst (LDS;
    // src may be dst).  Thread t publishes src[t], which it wrote itself or
    // which a barrier made visible.  Partials, flags and polls are
    // device-coherent (agent-scope) relaxed atomics.  A workgroup barrier
    // does not wait for outstanding global stores, so every storing wave
    // waits for its partial stores to be acknowledged (vmcnt 0) before the
    // barrier after which thread 0 raises the workgroup's flag; without that
    // wait another workgroup can see the flag and read a stale partial.  No
    // release/acquire fences: those would write back or invalidate the whole
    // L2 on every exchange.  Each workgroup has a flag of its own, set to the
    // exchange's sequence number, and thread t polls the flag of workgroup t.
    // Slots alternate between two parities: a workgroup can only rewrite a
    // slot after every other workgroup has published the exchange after the
    // one that read it.  The sums are taken in workgroup order.
    auto exchange = [&](const double* src, double* dst, int cnt) __attribute__((always_inline)) {
        if (a.G == 1) {
            if (src != dst)
                for (int t = tid; t < cnt; t += kPT) dst[t] = src[t];
            __syncthreads();
            ++ex;
            return;
        }
        double* part = a.partials + (((long long)b * 2 + (ex & 1)) * a.G + g) * kPanelSlot;
        for (int t = tid; t < cnt; t += kPT)
            __hip_atomic_store(&part[t], src[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        const unsigned target = a.seq + ex + 1u;
        if (tid == 0) __hip_atomic_store(&flg[g], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int t = tid; t < a.G; t += kPT) {
            if (t == g) continue;
            unsigned spins = 0;
            while (__hip_atomic_load(&flg[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++spins > a.spin_limit) {
                    raise_flag(a.error_flag);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        __syncthreads();
        // The partials are read with plain buffer loads that carry the
        // agent-coherence cache policy (sc1, what an agent-scope relaxed
        // atomic load uses): the compiler keeps atomic loads in order and
        // interleaved their uses with them, one memory round trip per load;
        // plain loads of 32 partials are all issued before the first wait.
        // The barrier after the polls orders them after the flags were seen.
        const double* pb = a.partials + ((long long)b * 2 + (ex & 1)) * a.G * kPanelSlot;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)pb, (short)0, 0x7fffffff, kBufferRsrcWord3);
        for (int t = tid; t < cnt; t += kPT) {
            // Thirty-two loads in flight per round (clamped index, padded
            // with +0.0, which leaves the in-order sum unchanged).
            double sum = 0.0;
            for (int gg = 0; gg < a.G; gg += 32) {
                double v[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) {
                    const int gi = min(gg + u, a.G - 1);
                    v[u] = __builtin_bit_cast(
                        double, __builtin_amdgcn_raw_buffer_load_b64(rs, (gi * kPanelSlot + t) * 8, 0, kCoherentLoad));
                }
#pragma unroll
                for (int u = 0; u < 32; ++u) sum += gg + u < a.G ? v[u] : 0.0;
            }
            dst[t] = sum;
        }
        __syncthreads();
        ++ex;
    };

    // The same exchange done by wave 0 alone, for at most 64 values held one
    // per lane (no workgroup barrier: the wave's own stores are acknowledged
    // before its lane 0 raises the flag).  Returns lane l's sum over the
    // matrix's workgroups (lanes >= cnt: 0).
    auto exchange_wave = [&](double val, int cnt) __attribute__((always_inline)) -> double {
        double* part = a.partials + (((long long)b * 2 + (ex & 1)) * a.G + g) * kPanelSlot;
        if (lane < cnt) __hip_atomic_store(&part[lane], val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        const unsigned target = a.seq + ex + 1u;
        if (lane == 0) __hip_atomic_store(&flg[g], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int t = lane; t < a.G; t += 64) {
            if (t == g) continue;
            unsigned spins = 0;
            while (__hip_atomic_load(&flg[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++spins > a.spin_limit) {
                    raise_flag(a.error_flag);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        asm volatile("" ::: "memory");  // the partials are read after the polls
        const double* pb = a.partials + ((long long)b * 2 + (ex & 1)) * a.G * kPanelSlot;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)pb, (short)0, 0x7fffffff, kBufferRsrcWord3);
        double sum = 0.0;
        if (lane < cnt) {
            for (int gg = 0; gg < a.G; gg += 32) {
                double v[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) {
                    const int gi = min(gg + u, a.G - 1);
                    v[u] = __builtin_bit_cast(
                        double, __builtin_amdgcn_raw_buffer_load_b64(rs, (gi * kPanelSlot + lane) * 8, 0, kCoherentLoad));
                }
#pragma unroll
                for (int u = 0; u < 32; ++u) sum += gg + u < a.G ? v[u] : 0.0;
            }
        }
        return sum;
    };

    for (int c0 = 0; c0 < nb; c0 += kLW) {
        const int lw = min(kLW, nb - c0);
        for (int kk = 0; kk < lw; ++kk) {
            const int k = c0 + kk;
            // Sweep: reflector k-1 (inside this leaf) on the leaf's columns
            // > k-1 (rows >= k-1) and the dot products of column k below the
            // pivot with the leaf's columns.  Each thread owns the same rows
            // in every column (r0 + 64 w + lane + 64 kRG j for wave w), so
            // that it can write column k on its rows after the exchange
            // without a barrier; per-column conditions are uniform.
            double acc[kLW], cq[kLW];
#pragma unroll
            for (int q = 0; q < kLW; ++q) {
                const double c = s_coef[q];
                acc[q] = 0.0;
                cq[q] = (kk > 0 && q > kk && q < lw) ? c : 0.0;
            }
            const double ck = kk > 0 ? s_coef[kk] : 0.0;
            const int lo = max(r0, kk > 0 ? k - 1 : k);
            constexpr int U = kRowUnroll;
            // Rows are taken U at a time, all their loads first, then the
            // arithmetic and the stores row by row in increasing order, so
            // each lane accumulates its rows in the same order as one at a time.
            auto load_row = [&](int row, double (&val)[kLW], double& vraw, double& xraw)
                                __attribute__((always_inline)) {
                const int rl = row >= lo && row < r1 ? row - r0 : lo - r0;
#pragma unroll
                for (int q = 0; q < kLW; ++q) val[q] = X[rl + (c0 + min(q, lw - 1)) * xld];
                vraw = kk > 0 ? X[rl + (k - 1) * xld] : 0.0;
                xraw = X[rl + k * xld];
            };
            auto finish_row = [&](int row, double (&val)[kLW], double vraw, double xraw)
                                  __attribute__((always_inline)) {
                if (row < lo || row >= r1) return;
                const int rl = row - r0;
                const double vprev = kk > 0 ? (row == k - 1 ? 1.0 : vraw) : 0.0;
                const double xk = xraw - ck * vprev;
                const double xa = row > k ? xk : 0.0;  // column k below the pivot
#pragma unroll
                for (int q = 0; q < kLW; ++q) {
                    double v = val[q] - cq[q] * vprev;  // cq = 0 leaves columns <= k as they are
                    if (q == kk) v = xk;
                    val[q] = v;
                    acc[q] += xa * v;
                }
                if (kk > 0) {
#pragma unroll
                    for (int q = 0; q < kLW; ++q)
                        if (q > kk && q < lw) X[rl + (c0 + q) * xld] = val[q];
                }
            };
            for (int row = first; row < r1; row += S * U) {
                double val[U][kLW], vraw[U], xraw[U];
#pragma unroll
                for (int u = 0; u < U; ++u) load_row(row + S * u, val[u], vraw[u], xraw[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) finish_row(row + S * u, val[u], vraw[u], xraw[u]);
            }
            {
                // The 16 column sums of the wave in one transposing butterfly:
                // at offsets 32, 16, 8, 4 each lane keeps half of its values and
                // adds the partner's copy of that half (17 shuffles instead of
                // 16 x 6); then lane l holds value (l >> 2) & 15 summed over the
                // 16 lanes that differ in bits 2-5, and offsets 2, 1 finish it.
                static_assert(kLW == 16, "butterfly written for 16 columns per wave");
                double h[kLW];
#pragma unroll
                for (int q = 0; q < kLW; ++q) h[q] = acc[q];
                butterfly_step<8, 32>(h, lane);
                butterfly_step<4, 16>(h, lane);
                butterfly_step<2, 8>(h, lane);
                butterfly_step<1, 4>(h, lane);
                double t = h[0];
                t += __shfl_xor(t, 2, 64);
                t += __shfl_xor(t, 1, 64);
                if ((lane & 3) == 0) s_wp[wv * kLW + ((lane >> 2) & 15)] = t;
            }
            __syncthreads();
            if (wv == 0) {
                // Wave 0 alone does the column's exchange: lanes 0..15 add
                // the waves' sums in a fixed order, lanes 16..31 read back the
                // pivot row after the update if this slab holds it (zero
                // elsewhere: columns > k were stored above, columns < k are
                // unchanged and column k is recomputed).
                double val = 0.0;
                if (lane < kLW) {
                    val = s_wp[lane];
#pragma unroll
                    for (int q = 1; q < kRG; ++q) val += s_wp[q * kLW + lane];
                } else if (lane < 2 * kLW && k >= r0 && k < r1) {
                    const int q = lane - kLW, rl = k - r0;
                    double v;
                    v = X[rl + (c0 + min(q, lw - 1)) * xld];
                    if (q == kk) v -= ck * (kk > 0 ? X[rl + (k - 1) * xld] : 0.0);
                    val = q < lw ? v : 0.0;
                }
                double sum = val;
                if (a.G > 1) sum = exchange_wave(val, 2 * kLW);
                // Reflector k on x = [alpha; below], beta = -sign(alpha) |x|,
                // v = [1; below / (alpha - beta)]  (no cancellation in alpha - beta).
                const double s2 = __shfl(sum, kk, 64), alpha = __shfl(sum, kLW + kk, 64);
                double beta, tau, scale;
                if (s2 == 0.0) {
                    beta = alpha;
                    tau = 0.0;
                    scale = 0.0;
                } else {
                    const double nrm = sqrt(alpha * alpha + s2);
                    beta = alpha >= 0.0 ? -nrm : nrm;
                    tau = (beta - alpha) / beta;
                    scale = 1.0 / (alpha - beta);
                }
                // v_k^T col (lane > kk) or v_lane^T v_k (lane < kk)
                const double w = __shfl(sum, kLW + (lane & (kLW - 1)), 64) + scale * sum;
                if (lane < lw && lane > kk) s_coef[lane] = tau * w;
                if (lane < kk) s_z[lane] = w;
                if (lane == 0) {
                    s_rfl[0] = beta;
                    s_rfl[1] = tau;
                    s_rfl[2] = scale;
                }
            }
            ++ex;
            __syncthreads();
            const double beta = s_rfl[0], tau = s_rfl[1], scale = s_rfl[2];
            // Column k on this thread's rows: R entry on row k-1, beta on the
            // pivot, v below (column k was not stored by the sweep; column
            // k-1 on these rows was written by this thread).
            for (int row = first; row < r1; row += S) {
                if (row < lo) continue;
                const int rl = row - r0;
                const double vprev = kk > 0 ? (row == k - 1 ? 1.0 : X[rl + (k - 1) * xld]) : 0.0;
                const double x = X[rl + k * xld] - ck * vprev;
                X[rl + k * xld] = row == k ? beta : (row > k ? scale * x : x);
            }
            // Column kk of the leaf's T_s (every workgroup keeps T_s):
            // T[c0+j][k] = -tau sum_l T[c0+j][c0+l] z_l, T[k][k] = tau.
            // Thread 64 + j forms row j of T_s in every column, so it only
            // reads entries it wrote itself.
            if (tid >= 64 && tid <= 64 + kk) {
                const int j = tid - 64;
                const int base = k * (k + 1) / 2 + c0;
                if (j < kk) {
                    double s0 = 0.0, s1 = 0.0;
                    int l = j;
                    for (; l + 1 < kk; l += 2) {
                        s0 += s_T[(c0 + l) * (c0 + l + 1) / 2 + c0 + j] * s_z[l];
                        s1 += s_T[(c0 + l + 1) * (c0 + l + 2) / 2 + c0 + j] * s_z[l + 1];
                    }
                    for (; l < kk; ++l) s0 += s_T[(c0 + l) * (c0 + l + 1) / 2 + c0 + j] * s_z[l];
                    s_T[base + j] = -tau * (s0 + s1);
                } else {
                    s_T[base + kk] = tau;
                }
            }
        }
        __syncthreads();  // the leaf's columns and T_s are complete

        // Leaf end: W = V_s^T [V_prev, C] over rows >= c0 (V_s is zero above
        // row c0, 1 on its diagonal).  Wave w forms the 16 x 16 block of
        // other columns 16 w .. 16 w + 15 with 16 x 16 x 4 MFMAs: lane l
        // holds V_s[row][c0 + l % 16] and Y[row][l % 16] for row = base + l / 16.
        const int nother = nb - lw;
        if (nother == 0) break;
        const int nblk = (nother + 15) / 16;
        const int rs = max(r0, c0);
        // Wave w takes block w % nblk over every nparts-th group of rows
        // (part w / nblk); the parts' blocks are added in part order.
        const int nparts = kRG / nblk;
        const int part = wv / nblk;
        d4 w4 = d4{0, 0, 0, 0};
        const int q0 = (wv % nblk) * 16;
        const int i = lane & 15;
        if (part < nparts) {
            const int cb = q0 < c0 ? q0 : q0 + lw;  // first column of the block (blocks do not straddle the leaf)
            const int ci = c0 + i, cj = cb + i;
            const bool iok = i < lw, jok = cj < nb && (q0 + i) < nother;
            constexpr int UQ = kQuadUnroll;
            for (int base = rs + 4 * UQ * part; base < r1; base += 4 * UQ * nparts) {
                double av[UQ], bv[UQ];
#pragma unroll
                for (int u = 0; u < UQ; ++u) {
                    const int r = base + 4 * u + (lane >> 4);
                    const bool rok = r < r1;
                    const int rl = rok ? r - r0 : 0;
                    const double xa = X[rl + (iok ? ci : c0) * xld];
                    const double xb = X[rl + (jok ? cj : c0) * xld];
                    av[u] = (rok && iok && r >= ci) ? (r == ci ? 1.0 : xa) : 0.0;
                    bv[u] = (rok && jok) ? xb : 0.0;
                }
#pragma unroll
                for (int u = 0; u < UQ; ++u) w4 = mfma_f64_16x16x4(av[u], bv[u], w4);
            }
        }
        for (int pp = 0; pp < nparts; ++pp) {
            if (part == pp) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int ii = Mfma<double>::row(lane, e);
                    double& d = s_W[ii * kOther + q0 + i];
                    d = pp == 0 ? w4[e] : d + w4[e];
                }
            }
            __syncthreads();
        }
        exchange(s_W, s_W, lw * kOther);

        if (g == 0 && c0 > 0) {
            // T[0:c0, c0:c0+lw] = -T1 (V_prev^T V_s) T_s, first M = (V_prev^T V_s) T_s.
            double m[2] = {0.0, 0.0};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = tid + h * kPT;
                if (t < c0 * lw) {
                    const int j = t / lw, i = t % lw;
                    double s = 0.0;
                    for (int l = 0; l <= i; ++l)
                        s += s_W[l * kOther + j] * s_T[(c0 + i) * (c0 + i + 1) / 2 + c0 + l];
                    m[h] = s;
                }
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = tid + h * kPT;
                if (t < c0 * lw) s_W[(t % lw) * kOther + t / lw] = m[h];
            }
            __syncthreads();
            for (int t = tid; t < c0 * lw; t += kPT) {
                const int jj = t / lw, i = t % lw;
                double s = 0.0;
                for (int j = jj; j < c0; ++j) s += s_T[j * (j + 1) / 2 + jj] * s_W[i * kOther + j];
                s_T[(c0 + i) * (c0 + i + 1) / 2 + jj] = -s;
            }
        }
        const int nc = nb - c0 - lw;  // later columns of the panel
        if (nc > 0) {
            // W2 = T_s^T (V_s^T C) in place of V_s^T C, then C -= V_s W2.
            double m[2] = {0.0, 0.0};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = tid + h * kPT;
                if (t < lw * nc) {
                    const int i = t / nc, q = c0 + t % nc;
                    double s = 0.0;
                    for (int l = 0; l <= i; ++l)
                        s += s_T[(c0 + i) * (c0 + i + 1) / 2 + c0 + l] * s_W[l * kOther + q];
                    m[h] = s;
                }
            }
            __syncthreads();
            // W2 goes back transposed, W2[i][q] at q * kLW + i (q: column of
            // C), so that a column's 16 entries are contiguous.
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = tid + h * kPT;
                if (t < lw * nc) s_W[(t % nc) * kLW + t / nc] = m[h];
            }
            __syncthreads();
            for (int r = rs + tid; r < r1; r += kPT) {
                const int rl = r - r0;
                double v[kLW];
#pragma unroll
                for (int i = 0; i < kLW; ++i) {
                    const int ci = c0 + i;
                    const double x = X[rl + min(ci, nb - 1) * xld];
                    v[i] = (i < lw && r >= ci) ? (r == ci ? 1.0 : x) : 0.0;
                }
                // Sixteen columns' loads issued together.
#pragma unroll 1
                for (int q0 = 0; q0 < nc; q0 += 16) {
                    double cv[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) cv[u] = q0 + u < nc ? X[rl + (c0 + lw + q0 + u) * xld] : 0.0;
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        if (q0 + u < nc) {
                            double s = 0.0;
#pragma unroll
                            for (int i = 0; i < kLW; ++i) s += v[i] * s_W[(q0 + u) * kLW + i];
                            X[rl + (c0 + lw + q0 + u) * xld] = cv[u] - s;
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    // Save the R diagonal block; make V's top block explicit (1 on the
    // diagonal, 0 above) so the GEMMs can use the stored panel as V.
    double* Rd = a.Rd + b * a.srd;
    for (int e = tid; e < kNB * kNB; e += kPT) {
        const int i = e % kNB, j = e / kNB;
        if ((i >= r0 && i < r1) || (g == 0 && i >= a.L)) {
            const bool in = i < nb && j < nb && i < a.L;
            const double v = in ? X[(i - r0) + j * xld] : 0.0;
            Rd[e] = (in && i <= j) ? v : 0.0;
            if (in && i <= j) X[(i - r0) + j * xld] = (i == j) ? 1.0 : 0.0;
        }
    }
    if (g == 0 && tid < kNB) {
        double* Tb = a.T + b * a.st;
        for (int l = 0; l < kNB; ++l) Tb[tid + l * kNB] = (tid <= l && l < nb) ? s_T[l * (l + 1) / 2 + tid] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Register-leaf panel.  A workgroup of NT threads owns up to NT * J rows of the
// panel, thread t the rows t, t + NT, ...; while a leaf of 16 columns is
// factored it stays in registers (J x 16 per thread), so a column touches no
// memory but the few LDS words of its reduction.
//
// The leaf's registers are a ring: the current column is entry 0, the later
// ones follow, the finished reflectors of the leaf come last.  Column k takes
//   1. the products of its entries below the pivot with all 16 entries
//      (norm, update dots and the products with the finished reflectors);
//   2. their sums over the wave by a transposing butterfly of lane swaps and
//      DPP moves (no LDS), over the waves through LDS, and for MULTI over the
//      matrix's workgroups (below);
//   3. the reflector, which every wave forms for itself from those sums (the
//      double-buffered LDS words make one barrier a column enough; MULTI takes
//      a second one after wave 0's exchange);
//   4. its application to the later columns, which also turns the ring by one:
//      new[q - 1] = old[q] - c_q v.  Coefficient q sits in lane q of each row
//      of 16 lanes and reaches the others by a DPP row broadcast.
// After 16 columns the ring is in column order again.
//
// End of a leaf: each wave stages V (its own rows, 64 x 16 at a time) in LDS
// and forms its part of W = V_s^T [V_prev, C] with 16 x 16 x 4 MFMAs; the parts are
// summed over the waves (MULTI: and workgroups).  W2 = T_s^T (V_s^T C) comes out of
// the MFMA in the layout that the update C -= V_s W2 takes as its operand.
// V_prev^T V_s goes to the packed V^T V from which the first workgroup merges
// T once, after the last leaf.
//
// J = 1 keeps the other three blocks of 16 columns in registers too, as tiles that
// are both the operand of W and the accumulator of the update: the panel is read
// once, and a leaf's columns are written once.  After a leaf its V becomes a tile
// and the next leaf's tile is turned to a row per lane through LDS.  T_s is
// formed by one wave between its MFMAs.  For J > 1 the other columns are read and
// written at every leaf end.
//
// The workgroups' exchange of a column (MULTI): wave 0 stores the workgroup's
// 16 sums, the first workgroup also the pivot row, as 16-byte slots
// {low word, tag, high word, tag}; each 8-byte half carries the exchange's
// sequence number, so a reader polls the data itself: one trip through memory
// where a flag took three (partials acknowledged, flag, partials read).  Slots
// alternate between two parities: a workgroup rewrites a slot only after every
// other one has published the exchange after the one that read it.  Tags grow
// through a factorisation and start from zeroed slots.  Every wait is bounded.
// With a matrix's workgroups on one XCD the slots stay in its L2; the accesses are
// coherent over the whole GPU, so the placement matters for speed alone.
//
// Bound: latency of the 64 dependent columns, about 250 dependent instructions each:
// in one workgroup 1500 cycles (256 rows) or 2170 (512 rows), 2600-3500 more with the
// exchange; a leaf end takes 16-20k cycles.  64-column panels, us, against the slab
// in LDS (a sweep of 16 columns per column, flag exchange) and against the leaf
// alone in registers, with square root and divisions in the column's chain and the
// exchange across the XCDs:
//   live rows       128   256   512  1024  2048  4160  8256  8 x 8256
//   slab in LDS     372   400   408   426   433   471   502       542
//   leaf            100   108   141   206   220   254   290       309
//   this kernel      73    77   106   166   179   214   246       249
// ---------------------------------------------------------------------------
typedef unsigned u4v __attribute__((ext_vector_type(4)));
typedef double dpair_u __attribute__((ext_vector_type(2), aligned(8)));
typedef double dpair __attribute__((ext_vector_type(2)));

// Sums of 16 values over the wave: lane l returns the sum of value (l >> 2) & 15.
__device__ inline double wave_sums16(double (&h)[16], int lane) {
#pragma unroll
    for (int p = 0; p < 8; ++p) h[p] = swap32_add(h[p], h[p + 8]);
#pragma unroll
    for (int p = 0; p < 4; ++p) h[p] = swap16_add(h[p], h[p + 4]);
    const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
    for (int p = 0; p < 2; ++p) h[p] = (b3 ? h[p + 2] : h[p]) + dpp<kDppRor8>(b3 ? h[p] : h[p + 2]);
    double t = (b2 ? h[1] : h[0]) + dpp<kDppHalfMirror>(b2 ? h[0] : h[1]);
    t += dpp<kDppXor1>(t);
    t += dpp<kDppXor2>(t);
    return t;
}

// xr[q - 1] = xr[q] - c_q v for q = 1..15 (c: lane q of each row of 16 holds c_q), xr[15] = last.
template <int N>
__device__ inline double row_bcast(double x) {
    return __builtin_bit_cast(double, (long long)__builtin_amdgcn_update_dpp(
                                          0ll, __builtin_bit_cast(long long, x), kDppRowBcast + N, 0xf, 0xf, true));
}
template <int Q>
__device__ __forceinline__ void ring_turn(double (&xr)[kLW], double c, double v) {
    if constexpr (Q < kLW) {
        xr[Q - 1] = fma(-row_bcast<Q>(c), v, xr[Q]);
        ring_turn<Q + 1>(xr, c, v);
    }
}

// Packed strict upper triangle: (i, j), i < j.
__device__ inline int upper_at(int i, int j) { return j * (j - 1) / 2 + i; }

// T_s of a leaf from its taus and V^T V: T[i][c] = -tau_c sum_{i <= l < c} T[i][l]
// (V^T V)[l][c], T[c][c] = tau_c.  Lane i of each row of 16 lanes holds row i of T,
// row[c] the sum so far: once column C is final its terms go to all later columns,
// which are independent of each other (a sum per column at a time is a chain of
// 120 dependent operations, 7.4k cycles).  z: row C of V^T V, the same in all lanes.
template <int C>
__device__ __forceinline__ void leaf_z(double (&z)[kLW], const double* s_G, int c0) {
#pragma unroll
    for (int c = C + 1; c < kLW; ++c) z[c] = s_G[upper_at(c0 + C, c0 + c)];
}
template <int C>
__device__ __forceinline__ void leaf_t_column(double (&row)[kLW], const double (&z)[kLW], double tau, int lw, int l16,
                                     double (*s_Ts)[kLW + 1]) {
    const double t = row_bcast<C>(tau);
    const double x = l16 == C ? t : (C > 0 && l16 < C && C < lw ? -t * row[C] : 0.0);
    s_Ts[l16][C] = x;                             // the four rows of lanes alike
#pragma unroll
    for (int c = C + 1; c < kLW; ++c) row[c] = C == 0 ? x * z[c] : fma(x, z[c], row[c]);
}
template <int C = 0>
__device__ __forceinline__ void leaf_t_all(double (&row)[kLW], const double (&z)[kLW], const double* s_G, double tau, int c0,
                                  int lw, int l16, double (*s_Ts)[kLW + 1]) {
    if constexpr (C < kLW) {
        double zn[kLW];
        leaf_z<C + 1>(zn, s_G, c0);
        leaf_t_column<C>(row, z, tau, lw, l16, s_Ts);
        __builtin_amdgcn_sched_barrier(0);
        leaf_t_all<C + 1>(row, zn, s_G, tau, c0, lw, l16, s_Ts);
    }
}
__device__ __forceinline__ void leaf_t(const double* s_G, const double* s_tau, int c0, int lw, int l16,
                              double (*s_Ts)[kLW + 1]) {
    double row[kLW], z[kLW];
    const double tau = l16 < lw ? s_tau[c0 + min(l16, lw - 1)] : 0.0;
    leaf_z<0>(z, s_G, c0);
    leaf_t_all(row, z, s_G, tau, c0, lw, l16, s_Ts);
}
// The 16 steps U of the products of a tile of V (column l % 16, at sv) with the
// NQ tiles y.  TS: column U of T_s is formed between step U's MFMAs
// (64 cycles each), which hide it.
template <bool TS, int NQ, int VS, int U = 0>
__device__ __forceinline__ void leaf_steps(const double* sv, const double (*y)[kLW], d4* w, dpair v,
                                           double (&row)[kLW], const double* s_G, double tau, int c0, int lw,
                                           int lane, double (*s_Ts)[kLW + 1]) {
    if constexpr (U < kLW) {
        const int l16 = lane & 15, lg = lane >> 4;
        double z[kLW];
        if constexpr (TS) leaf_z<U>(z, s_G, c0);
        if constexpr (U % 2 == 0) v = *reinterpret_cast<const dpair*>(&sv[l16 * VS + 4 * U + 2 * lg]);
#pragma unroll
        for (int q = 0; q < NQ; ++q) w[q] = mfma_f64_16x16x4(v[U % 2], y[q][U], w[q]);
        if constexpr (TS) {
            leaf_t_column<U>(row, z, tau, lw, l16, s_Ts);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);               // an MFMA,
                __builtin_amdgcn_sched_group_barrier(0x2, (kLW - U + 12) / NQ, 0);   // vector instructions of T_s
            }
        }
        __builtin_amdgcn_sched_barrier(0);        // one step's loads at a time (registers)
        leaf_steps<TS, NQ, VS, U + 1>(sv, y, w, v, row, s_G, tau, c0, lw, lane, s_Ts);
    }
}

template <int NT, int J, bool MULTI>
__global__ __launch_bounds__(NT) void panel_leaf_kernel(PanelArgs a) {
    constexpr int NW = NT / 64;
    constexpr int VS = 66;                        // row stride of a staged V column (16-byte loads)
    constexpr int NO = kOther / kLW;              // other blocks of 16 columns
    constexpr bool RES = J == 1;                  // the whole panel in registers
    constexpr int TW = NW - 1;                    // the wave that forms T_s
    constexpr int TS = kNB + 1;
    // The words that every column takes come first: within 64 KiB an address is
    // an instruction's offset.
    __shared__ struct __attribute__((aligned(16))) {
        double part[2][NW][kLW], prow[2][kLW], tot[2][2 * kLW];
        double tau[kNB], unused[kLW];
        double Ts[kNL][kLW][kLW + 1];             // T_s of each leaf
        double G[kNB * (kNB - 1) / 2];            // V^T V, strict upper
        double W[kLW * kOther];                   // W[i][q] at i * kOther + q
        double v[NW][kLW * VS];                   // staged V, at the end T
        double p[RES ? NW : 1][RES ? kLW * kOther : 1];   // the waves' parts of W
    } sm;
    auto &s_part = sm.part;
    auto &s_v = sm.v;
    auto &s_prow = sm.prow;
    auto &s_tot = sm.tot;
    auto &s_tau = sm.tau;
    auto &s_Ts = sm.Ts;
    auto &s_G = sm.G;
    auto &s_W = sm.W;
    auto &s_p = sm.p;
    static_assert(4 * kLW * VS >= kNB * TS, "s_v holds T");
    static_assert(NW == 4 || NW == 8, "T in s_v; sum_waves");
    // Workgroups are dealt to the XCDs round-robin: with `local` matrix b's lie on
    // XCD b % kNumXcd (and the others of the grid leave).
    const int chunk = MULTI && a.local ? kNumXcd : 1;
    const int idx = blockIdx.x / chunk;
    const int g = MULTI ? idx % a.G : 0, b = MULTI ? blockIdx.x % chunk + chunk * (idx / a.G) : blockIdx.x;
    if (MULTI && b >= a.batch) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const long long ld = a.ld;
    const int nb = a.nb;
    const int r0 = g * a.rows_per_wg;
    const int nr = min(a.L - r0, a.rows_per_wg);  // rows of this workgroup
    double* __restrict__ X = a.P + b * a.sp + r0;
    bool dead = false;                            // a bounded wait gave up: wait no more

    // Sums s_W over the matrix's workgroups (s_W on every one that wants them).
    auto leaf_exchange = [&](int leaf, bool want) __attribute__((always_inline)) {
        double* slots = a.partials + ((long long)b * 2 + (leaf & 1)) * a.G * kPanelSlot;
        for (int t = tid; t < kPanelSlot; t += NT)
            __hip_atomic_store(&slots[(long long)g * kPanelSlot + t], s_W[t], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        unsigned* flg = a.flags + (long long)b * a.G;
        const unsigned target = a.seq + kNB + leaf + 1u;
        if (tid == 0) __hip_atomic_store(&flg[g], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!want) return;
        for (int t = tid; t < a.G; t += NT) {
            unsigned spins = 0;
            while (!dead && __hip_atomic_load(&flg[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++spins > a.spin_limit) {
                    raise_flag(a.error_flag);
                    dead = true;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        __syncthreads();
        // Plain buffer loads with the agent-coherence policy: all of a round
        // are in flight together (atomic loads would be taken one by one).
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)slots, (short)0, 0x7fffffff, kBufferRsrcWord3);
        for (int t = tid; t < kPanelSlot; t += NT) {
            double sum = 0.0;
            for (int gg = 0; gg < a.G; gg += 16) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    v[u] = __builtin_bit_cast(
                        double, __builtin_amdgcn_raw_buffer_load_b64(
                                    rs, (min(gg + u, a.G - 1) * kPanelSlot + t) * 8, 0, kCoherentLoad));
#pragma unroll
                for (int u = 0; u < 16; ++u) sum += gg + u < a.G ? v[u] : 0.0;
            }
            s_W[t] = sum;
        }
        __syncthreads();
    };
    // Wave 0: val = the workgroup's sum (value lane & 15 in every row of 16
    // lanes); returns the sums over the workgroups, and in prow the pivot row.
    auto column_exchange = [&](int k, double val, double& prow) __attribute__((always_inline)) -> double {
        const unsigned tag = a.seq + k + 1u;
        unsigned long long* slots = a.colslots + ((long long)b * 2 + (k & 1)) * a.G * (4 * kLW);
        if (lane < (g == 0 ? 2 * kLW : kLW)) {
            const unsigned long long u = __builtin_bit_cast(unsigned long long, lane < kLW ? val : prow);
            unsigned long long* p = slots + (long long)g * (4 * kLW) + 2 * lane;
            __hip_atomic_store(p, ((unsigned long long)tag << 32) | (unsigned)u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p + 1, ((unsigned long long)tag << 32) | (unsigned)(u >> 32), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)slots, (short)0, 0x7fffffff, kBufferRsrcWord3);
        auto value = [](u4v x) { return __builtin_bit_cast(double, ((unsigned long long)x[2] << 32) | x[0]); };
        double sum = 0.0;
        constexpr int U = 4;                      // loads in flight: 4 U workgroups
        for (int w0 = 0; w0 < a.G; w0 += 4 * U) {
            u4v v[U + 1];
            unsigned spins = 0;
            for (;;) {
                // The addresses do not change: without this the loads, which the
                // compiler takes for ordinary ones, might be kept from turn to turn.
                asm volatile("" ::: "memory");
                bool ok = true;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int wg = min(w0 + 4 * u + lg, a.G - 1);
                    v[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, wg * (32 * kLW) + l16 * 16, 0, kCoherentLoad);
                }
                // The pivot row, from the first workgroup's second half.
                v[U] = __builtin_amdgcn_raw_buffer_load_b128(rs, (kLW + l16) * 16, 0, kCoherentLoad);
#pragma unroll
                for (int u = 0; u <= U; ++u) ok = ok && v[u][1] == tag && v[u][3] == tag;
                if (__all(ok) || dead) break;
                if (++spins > (a.spin_limit >> 4)) {   // a memory round trip each: about a second
                    if (lane == 0) raise_flag(a.error_flag);
                    dead = true;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) sum += w0 + 4 * u + lg < a.G ? value(v[u]) : 0.0;
            prow = value(v[U]);
        }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        return sum;
    };

    // A tile: 16 columns of 64 rows, element u of lane l is row 8 (u / 2) + 2 (l / 16) +
    // u % 2 of column cb + l % 16, so that a load of 16 bytes a lane takes 64
    // contiguous bytes of each column.
    auto load_tile = [&](int cb, int base, double (&y)[kLW]) __attribute__((always_inline)) {
        const int row = base + 2 * lg;
        const double* p = X + (long long)min(cb + l16, nb - 1) * ld;
        if (base + 64 <= nr) {
#pragma unroll
            for (int u = 0; u < kLW; u += 2) {
                const dpair_u t = *reinterpret_cast<const dpair_u*>(p + row + 4 * u);
                y[u] = t[0];
                y[u + 1] = t[1];
            }
        } else {
#pragma unroll
            for (int u = 0; u < kLW; ++u) y[u] = p[min(row + 4 * (u & ~1) + (u & 1), nr - 1)];
        }
    };
    // The leaf's columns, a row per lane: loads from valid addresses, then zeros
    // for rows past the slab and columns past a short leaf.
    double xr[J][kLW];
    auto load_leaf = [&](int c0, int lw) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const unsigned at = min(tid + NT * j, nr - 1);
#pragma unroll
            for (int q = 0; q < kLW; ++q) xr[j][q] = (X + (long long)(c0 + min(q, lw - 1)) * ld)[at];
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int in = opaque(tid + NT * j < nr ? -1 : 0);
#pragma unroll
            for (int q = 0; q < kLW; ++q) xr[j][q] = keep_if(xr[j][q], q < lw ? in : 0);
        }
    };
    // The other blocks in the order later ones, finished ones (V).
    double y[RES ? NO : 1][kLW];
    if constexpr (RES) {
        load_leaf(0, min(kLW, nb));
#pragma unroll
        for (int q = 0; q < NO; ++q) load_tile(kLW + kLW * q, min(64 * wv, (nr - 1) & ~63), y[q]);
#pragma unroll
        for (int q = 0; q < NO; ++q)
#pragma unroll
            for (int u = 0; u < kLW; ++u)
                y[q][u] = keep_if(y[q][u], opaque(64 * wv + 2 * lg + 4 * (u & ~1) + (u & 1) < nr &&
                                                          kLW + kLW * q + l16 < nb ? -1 : 0));
    }
    for (int c0 = 0; c0 < nb; c0 += kLW) {
        const int lw = min(kLW, nb - c0), leaf = c0 / kLW;
        if constexpr (!RES) load_leaf(c0, lw);
        for (int kk = 0; kk < lw; ++kk) {
            const int k = c0 + kk, kr = k - r0;   // kr: pivot row within the slab
            const int buf = kk & 1;
            double acc[kLW];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int row = tid + NT * j;
                const double xa = row > kr ? xr[j][0] : 0.0;
#pragma unroll
                for (int q = 0; q < kLW; ++q) acc[q] = j == 0 ? xa * xr[j][q] : fma(xa, xr[j][q], acc[q]);
            }
            if (tid == kr) {                      // pivot rows are rows 0..63: j = 0
#pragma unroll
                for (int q = 0; q < kLW; ++q) s_prow[buf][q] = xr[0][q];
            }
            const double ws = wave_sums16(acc, lane);
            if ((lane & 3) == 0) s_part[buf][wv][lane >> 2] = ws;
            __syncthreads();
            double sum, prow;
            auto sum_waves = [&]() __attribute__((always_inline)) {
                double h[NW];
#pragma unroll
                for (int w = 0; w < NW; ++w) h[w] = s_part[buf][w][l16];
                prow = s_prow[buf][l16];
                // One wait for all of the words (the compiler would take them two by two).
                if constexpr (NW == 4) asm volatile("" : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(prow));
                else asm volatile("" : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]),
                                       "+v"(h[6]), "+v"(h[7]), "+v"(prow));
#pragma unroll
                for (int s = 1; s < NW; s *= 2)
#pragma unroll
                    for (int w = 0; w + s < NW; w += 2 * s) h[w] += h[w + s];
                return h[0];
            };
            if constexpr (MULTI) {
                if (wv == 0) {
                    sum = sum_waves();
                    sum = column_exchange(k, sum, prow);
                    if (lane < 2 * kLW) s_tot[buf][lane] = lane < kLW ? sum : prow;
                }
                __syncthreads();
                sum = s_tot[buf][l16];
                prow = s_tot[buf][kLW + l16];
            } else {
                sum = sum_waves();
            }
            // Reflector k on x = [alpha; below], beta = -sign(alpha) |x|,
            // v = [1; below / (alpha - beta)]  (no cancellation in alpha - beta).
            const double s2 = uniform(sum), alpha = uniform(prow);
            double beta = alpha, tau = 0.0, scale = 0.0;
            if (s2 != 0.0) householder(alpha, s2, beta, tau, scale);
            const double w = fma(scale, sum, prow);   // v_k^T column (later) or v_l^T v_k (finished)
            const double c = l16 < kLW - kk ? tau * w : 0.0;
            // tau from lane 0, V^T V from the finished columns' lanes, in one store
            // by the wave that has the fewest rows.
            if (wv == TW && lane < kLW) {
                double* to = lane >= kLW - kk ? &s_G[upper_at(c0 + lane - (kLW - kk), k)] : &sm.unused[lane];
                to = lane == 0 ? &s_tau[k] : to;
                *to = lane == 0 ? tau : w;
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int row = tid + NT * j;
                const double x = xr[j][0];
                const double v = row > kr ? scale * x : (row == kr ? 1.0 : 0.0);
                ring_turn<1>(xr[j], c, v);
                xr[j][kLW - 1] = row > kr ? v : (row == kr ? beta : x);
            }
        }
        for (int kk = lw; kk < kLW; ++kk) {       // a short leaf: turn the ring back into column order
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const double x = xr[j][0];
#pragma unroll
                for (int q = 1; q < kLW; ++q) xr[j][q - 1] = xr[j][q];
                xr[j][kLW - 1] = x;
            }
        }
        // The leaf to memory.
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int row = tid + NT * j;
            if (row >= nr) continue;
            if (lw == kLW) {
#pragma unroll
                for (int q = 0; q < kLW; ++q) (X + (long long)(c0 + q) * ld)[(unsigned)row] = xr[j][q];
            } else {
#pragma unroll
                for (int q = 0; q < kLW; ++q)
                    if (q < lw) (X + (long long)(c0 + q) * ld)[(unsigned)row] = xr[j][q];
            }
        }
        // Tile q of 16 other columns is later, q < nlater, or finished, q >= fin, of a
        // resident panel; else they are in the order of the columns.
        const int nother = nb - lw, nblk = (nother + kLW - 1) / kLW, nc = nb - c0 - lw;
        const int nlater = (nc + kLW - 1) / kLW, fin = NO - leaf;
        const int later0 = RES ? 0 : c0, prev0 = RES ? kLW * fin : 0;
        auto tile_col = [&](int q) __attribute__((always_inline)) { return kLW * q < c0 ? kLW * q : kLW * q + lw; };
        double* const sv = s_v[wv];
        if constexpr (RES) {
            // V staged in LDS by each wave for its own 64 rows: 1 on the pivot,
            // zeros above it.
            d4 w4[NO];
#pragma unroll
            for (int q = 0; q < NO; ++q) w4[q] = d4{0, 0, 0, 0};
            if (64 * wv < nr) {
                __builtin_amdgcn_wave_barrier();
                if (wv > 0 || r0 > 0) {           // no pivots here
#pragma unroll
                    for (int q = 0; q < kLW; ++q) sv[q * VS + lane] = xr[0][q];
                } else {
#pragma unroll
                    for (int q = 0; q < kLW; ++q) {
                        const int k = c0 + q;
                        sv[q * VS + lane] = lane > k ? xr[0][q] : (lane == k && q < lw ? 1.0 : 0.0);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                double row[kLW];
                const double tau = l16 < lw ? s_tau[c0 + min(l16, lw - 1)] : 0.0;
                if (nlater + leaf == NO) {
                    if (wv == TW) {
                        leaf_steps<true, NO, VS>(sv, y, w4, dpair{}, row, s_G, tau, c0, lw, lane, s_Ts[leaf]);
                    } else {
                        leaf_steps<false, NO, VS>(sv, y, w4, dpair{}, row, s_G, tau, c0, lw, lane, s_Ts[leaf]);
                    }
                } else {
                    if (wv == TW) leaf_t(s_G, s_tau, c0, lw, l16, s_Ts[leaf]);
#pragma unroll
                    for (int q = 0; q < NO; ++q)
                        if (q < nlater || q >= fin)
                            leaf_steps<false, 1, VS>(sv, &y[q], &w4[q], dpair{}, row, s_G, tau, c0, lw, lane, s_Ts[leaf]);
                }
            } else if (wv == TW) {
                leaf_t(s_G, s_tau, c0, lw, l16, s_Ts[leaf]);
            }
            if (nother > 0) {
#pragma unroll
                for (int q = 0; q < NO; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s_p[RES ? wv : 0][Mfma<double>::row(lane, e) * kOther + kLW * q + l16] = w4[q][e];
            }
        }
        // V of the wave's rows 64 wv + NT j ... + 63, staged in LDS by the wave for
        // itself, read back so that the leaf's registers are free from here on.
        auto load_v = [&](int j, double (&v)[kLW]) __attribute__((always_inline)) {
            const unsigned at = min(tid + NT * j, nr - 1);
#pragma unroll
            for (int q = 0; q < kLW; ++q) v[q] = (X + (long long)(c0 + min(q, lw - 1)) * ld)[at];
        };
        auto stage = [&](int j, const double (&v)[kLW]) __attribute__((always_inline)) {
            const int row = tid + NT * j;
            __builtin_amdgcn_wave_barrier();
            if (j > 0 && lw == kLW) {             // no pivots here: V is the leaf as it is
                const int in = opaque(row < nr ? -1 : 0);
#pragma unroll
                for (int q = 0; q < kLW; ++q) sv[q * VS + lane] = keep_if(v[q], in);
            } else {
#pragma unroll
                for (int q = 0; q < kLW; ++q) {
                    const int kr = c0 + q - r0;
                    const int in = opaque(((row > kr) & (row < nr) & (q < lw)) ? -1 : 0);
                    sv[q * VS + lane] = row == kr && q < lw ? 1.0 : keep_if(v[q], in);
                }
            }
            __builtin_amdgcn_wave_barrier();
        };
        if constexpr (!RES) {
            d4 w4[kOther / 16];
#pragma unroll
            for (int q = 0; q < kOther / 16; ++q) w4[q] = d4{0, 0, 0, 0};
            if (nother > 0) {
                auto product = [&](const double (&yv)[16], d4 w) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < 16; u += 2) {
                        const dpair t = *reinterpret_cast<const dpair*>(&sv[l16 * VS + 4 * u + 2 * lg]);
                        w = mfma_f64_16x16x4(t[0], yv[u], w);
                        w = mfma_f64_16x16x4(t[1], yv[u + 1], w);
                    }
                    return w;
                };
#pragma unroll 1
                for (int j = 0; j < J; ++j) {
                    if (64 * wv + NT * j >= nr) break;
                    double v[kLW], yv[kOther / 16][16];
                    load_v(j, v);
#pragma unroll
                    for (int q = 0; q < kOther / 16; ++q)
                        if (q < nblk) load_tile(tile_col(q), 64 * wv + NT * j, yv[q]);
                    stage(j, v);
#pragma unroll
                    for (int q = 0; q < kOther / 16; ++q)
                        if (q < nblk) w4[q] = product(yv[q], w4[q]);
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < kOther / 16; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sv[Mfma<double>::row(lane, e) * kOther + 16 * q + l16] = w4[q][e];
            }
        }
        __syncthreads();
        if constexpr (!RES) {
            if (wv == TW) leaf_t(s_G, s_tau, c0, lw, l16, s_Ts[leaf]);
        }
        if (nother > 0) {
            for (int t = tid; t < kLW * kOther; t += NT) {
                double h = RES ? s_p[0][t] : s_v[0][t];
#pragma unroll
                for (int w = 1; w < NW; ++w) h += RES ? s_p[RES ? w : 0][t] : s_v[w][t];
                s_W[t] = h;
            }
        }
        __syncthreads();
        if (nother <= 0) break;
        if constexpr (MULTI) leaf_exchange(leaf, g == 0 || nc > 0);
        if (g == 0) {                             // V_prev^T V_s
            for (int t = tid; t < c0 * lw; t += NT) {
                const int q = t / lw, i = t % lw;
                s_G[upper_at(q, c0 + i)] = s_W[i * kOther + prev0 + q];
            }
        }
        if (nc > 0) {                             // a full leaf
            // -W2 = -T_s^T (V_s^T C): the MFMA leaves W2[l / 16 + 4 e][l % 16]
            // in element e of lane l, the operand of step e below.
            d4 w2[NO];
#pragma unroll
            for (int q = 0; q < NO; ++q) {
                w2[q] = d4{0, 0, 0, 0};
                if (q < nlater) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w2[q] = mfma_f64_16x16x4(-s_Ts[leaf][4 * e + lg][l16],
                                                 s_W[(4 * e + lg) * kOther + min(later0 + kLW * q + l16, kOther - 1)],
                                                 w2[q]);
                }
            }
            if constexpr (RES) {
                // C -= V_s W2 on the tiles as they are: their elements 4 t .. 4 t + 3 are
                // the MFMA's rows l / 16 + 4 e, so its row i is row 16 t + pr of the 64.
                if (64 * wv < nr) {
                    const int pr = 8 * (l16 >> 3) + 2 * (l16 & 3) + ((l16 >> 2) & 1);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        double av[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) av[e] = sv[(4 * e + lg) * VS + 16 * t + pr];
#pragma unroll
                        for (int q = 0; q < NO; ++q)
                            if (q < nlater) {
                                d4 x = d4{y[q][4 * t], y[q][4 * t + 1], y[q][4 * t + 2], y[q][4 * t + 3]};
#pragma unroll
                                for (int e = 0; e < 4; ++e) x = mfma_f64_16x16x4(av[e], w2[q][e], x);
#pragma unroll
                                for (int e = 0; e < 4; ++e) y[q][4 * t + e] = x[e];
                            }
                    }
                }
                // The next leaf, a row per lane; the other tiles move up, V_s last
                // (a wave without rows keeps zeros).
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int u = 0; u < kLW; u += 2) {
                    dpair* const at = reinterpret_cast<dpair*>(&sv[l16 * VS + 4 * u + 2 * lg]);
                    const dpair v = *at;
                    *at = dpair{y[0][u], y[0][u + 1]};
#pragma unroll
                    for (int q = 0; q + 1 < NO; ++q) {
                        y[q][u] = y[q + 1][u];
                        y[q][u + 1] = y[q + 1][u + 1];
                    }
                    y[NO - 1][u] = 64 * wv < nr ? v[0] : 0.0;
                    y[NO - 1][u + 1] = 64 * wv < nr ? v[1] : 0.0;
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < kLW; ++q) xr[0][q] = sv[q * VS + lane];
            } else {
                // C goes through the MFMA 16 columns x 16 rows at a time, the next
                // tile's loads issued before this tile's stores.  Rows past the slab
                // and columns past the panel load valid addresses and are not stored.
                unsigned long long off[kOther / 4];   // column offsets of this lane
#pragma unroll
                for (int q = 0; q < kOther / 4; ++q)
                    off[q] = (unsigned long long)(unsigned)min(4 * q + lg, nc - 1) * (unsigned)ld;
                double* const Cl = X + (long long)(c0 + lw) * ld;
                auto load_c = [&](int row, d4 (&cv)[kOther / 16]) __attribute__((always_inline)) {
                    const double* p = Cl + min(row, nr - 1);
#pragma unroll
                    for (int q = 0; q < kOther / 16; ++q)
                        if (16 * q < nc) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) cv[q][e] = p[off[4 * q + e]];
                        }
                };
#pragma unroll 1
                for (int j = 0; j < J; ++j) {
                    const int base = 64 * wv + NT * j;
                    if (base >= nr) break;
                    double v[kLW];
                    d4 cv[2][kOther / 16];
                    load_v(j, v);
                    load_c(base + l16, cv[0]);
                    stage(j, v);
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
                        const int row = base + 16 * rt + l16;
                        if (rt < 3) load_c(row + 16, cv[(rt + 1) & 1]);
                        double bv[4];
#pragma unroll
                        for (int s = 0; s < 4; ++s) bv[s] = sv[(4 * s + lg) * VS + 16 * rt + l16];
                        double* p = Cl + row;
#pragma unroll
                        for (int q = 0; q < kOther / 16; ++q)
                            if (16 * q < nc) {
                                d4& c = cv[rt & 1][q];
#pragma unroll
                                for (int s = 0; s < 4; ++s) c = mfma_f64_16x16x4(w2[q][s], bv[s], c);
                                if (row < nr) {
                                    if (16 * q + 16 <= nc) {
#pragma unroll
                                        for (int e = 0; e < 4; ++e) p[off[4 * q + e]] = c[e];
                                    } else {
#pragma unroll
                                        for (int e = 0; e < 4; ++e)
                                            if (16 * q + 4 * e + lg < nc) p[off[4 * q + e]] = c[e];
                                    }
                                }
                            }
                    }
                }
            }
        }
        if constexpr (!RES) __syncthreads();
    }
    __syncthreads();                              // the columns are in memory
    if (g != 0) return;
    // The first workgroup holds the top block: R's diagonal block saved, V
    // made explicit (1 on the diagonal, 0 above), so that the GEMMs can use
    // the stored panel as V.
    double* Rd = a.Rd + b * a.srd;
    {
        double v[kNB * kNB / NT];                 // all loads in flight, from valid addresses
#pragma unroll
        for (int u = 0; u < kNB * kNB / NT; ++u) {
            const int e = tid + u * NT, i = e % kNB, j = e / kNB;
            v[u] = X[min(i, min(nb, a.L) - 1) + (long long)min(j, nb - 1) * ld];
        }
#pragma unroll
        for (int u = 0; u < kNB * kNB / NT; ++u) {
            const int e = tid + u * NT, i = e % kNB, j = e / kNB;
            const bool upper = i < nb && j < nb && i < a.L && i <= j;
            Rd[e] = upper ? v[u] : 0.0;
            if (upper) X[i + j * ld] = (i == j) ? 1.0 : 0.0;
        }
    }
    // T from the leaves' T_s and V^T V: T12 = -T1 (V1^T V2) T2 for 16 and 32
    // columns a side, on the matrix cores.
    double* const T = s_v[0];                     // T[i][j] at i + j TS
#pragma unroll
    for (int u = 0; u < kNB * kNB / NT; ++u) {
        const int e = tid + u * NT, i = e % kNB, j = e / kNB;
        const double x = s_Ts[j / kLW][i % kLW][j % kLW];
        T[i + j * TS] = keep_if(x, opaque(i / kLW == j / kLW && j / kLW * kLW < nb ? -1 : 0));
    }
    __syncthreads();
    auto merge = [&](auto width) __attribute__((always_inline)) {
        constexpr int s = decltype(width)::value;
        const int ts = s / 16, per = ts * ts, total = kNB / (2 * s) * per;   // 2, 4 tiles
        const int o = wv / per * 2 * s, ti = wv % per % ts * 16, tj = wv % per / ts * 16;
#pragma unroll
        for (int phase = 0; phase < 2; ++phase) {
            d4 acc = d4{0, 0, 0, 0};
            if (wv < total) {
                double x[kNB / 8], yv[kNB / 8];   // all operands in flight
#pragma unroll
                for (int k = 0; k < s; k += 4) {
                    if (phase == 0) {             // Y = (V1^T V2) T2 into the place of T12
                        const int i = o + ti + l16, l = o + s + k + lg;
                        x[k / 4] = keep_if(s_G[upper_at(i, l)], opaque(l < nb ? -1 : 0));
                        yv[k / 4] = T[o + s + k + lg + (o + s + tj + l16) * TS];
                    } else {
                        x[k / 4] = -T[o + ti + l16 + (o + k + lg) * TS];
                        yv[k / 4] = T[o + k + lg + (o + s + tj + l16) * TS];
                    }
                }
#pragma unroll
                for (int k = 0; k < s; k += 4) acc = mfma_f64_16x16x4(x[k / 4], yv[k / 4], acc);
            }
            __syncthreads();
            if (wv < total) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    T[o + ti + Mfma<double>::row(lane, e) + (o + s + tj + l16) * TS] = acc[e];
            }
            __syncthreads();
        }
    };
    merge(std::integral_constant<int, kLW>{});
    merge(std::integral_constant<int, 2 * kLW>{});
    static_assert(4 * kLW == kNB, "two levels of merges");
    double* Tb = a.T + b * a.st;
    for (int e = tid; e < kNB * kNB; e += NT) {
        const int i = e % kNB, j = e / kNB;
        Tb[e] = i <= j && j < nb ? T[i + j * TS] : 0.0;
    }
}

// Before Q formation: zeros above the diagonal blocks of all panels (the rows
// [0, p0) of columns [p0, p0 + 64), where R was), which Q's columns start from.
__global__ void zero_above_panels_kernel(int n, double* M, long long ld, long long sm) {
    for (int j = blockIdx.y; j < n; j += gridDim.y) {
        double* col = M + blockIdx.z * sm + j * ld;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < j / kNB * kNB; i += gridDim.x * blockDim.x)
            col[i] = 0.0;
    }
}

// A panel's own columns of Q over its live rows: Q = [I; 0] - V S, S = T V_top^T
// (kNB x kNB), in place of V.  A wave forms 16 rows of all 64 columns from its
// own rows of V, all loaded before the first store, with the roles of rows and
// columns exchanged in the MFMA so that loads and stores are 128 bytes of a
// column.  Bound: launch and load latency; it replaces a product (11 us) and a
// launch for the identity and the zeros above (5 us), and S comes from one
// batched launch: structured QR 1025 x 881 x 5 5.34 -> 5.17 ms, n = 2048 24.7 -> 24.4.
__global__ __launch_bounds__(256) void orgqr_panel_kernel(int L, int nb, double* V, long long ld, long long sv,
                                                          const double* __restrict__ S, long long ss) {
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lg = lane >> 4;
    const int row0 = (blockIdx.x * 4 + wave) * 16, row = row0 + l16;
    if (row0 >= L) return;
    double* Vb = V + b * sv + min(row, L - 1);
    const double* Sb = S + b * ss;
    double v[kNB / 4], t[kNB / 16][kNB / 4];      // lane l: k-values 4 (l / 16) + u of each 16
#pragma unroll
    for (int u = 0; u < kNB / 4; ++u) v[u] = Vb[min(16 * (u >> 2) + 4 * lg + (u & 3), nb - 1) * ld];
#pragma unroll
    for (int q = 0; q < kNB / 16; ++q)
#pragma unroll
        for (int u = 0; u < kNB / 4; ++u) t[q][u] = Sb[16 * (u >> 2) + 4 * lg + (u & 3) + (16 * q + l16) * kNB];
#pragma unroll
    for (int u = 0; u < kNB / 4; ++u) v[u] = keep_if(v[u], opaque(16 * (u >> 2) + 4 * lg + (u & 3) < nb ? -1 : 0));
#pragma unroll
    for (int q = 0; q < kNB / 16; ++q) {
        d4 acc;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = row == 16 * q + lg + 4 * e ? 1.0 : 0.0;
#pragma unroll
        for (int u = 0; u < kNB / 4; ++u)         // S of a short panel is defined for k, column < nb only
            acc = mfma_f64_16x16x4(-keep_if(t[q][u], opaque((16 * (u >> 2) + 4 * lg + (u & 3) < nb) ? -1 : 0)), v[u], acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 16 * q + lg + 4 * e;
            if (row < L && j < nb) Vb[j * ld] = acc[e];
        }
    }
}

// M_b[0:m] = X (skipped when X is null), M_b[m:m+n] = p_b I.
__global__ void stack_init_kernel(int m, int n, const double* __restrict__ X, long long ldx,
                                  double* __restrict__ M, long long ld, long long sm, ShiftArgs piv) {
    const long long rows = (long long)m + n;
    const long long total = rows * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / rows, i = e - j * rows;
        if (i < m && X == nullptr) continue;  // dense block already in place
        const double x = i < m ? X[i + j * ldx] : 0.0;
        for (int b = 0; b < piv.batch; ++b)
            M[b * sm + i + j * ld] = i < m ? x : (i - m == j ? piv.shift[b] : 0.0);
    }
}

// R_b (n x n) from the factored M_b: off-diagonal blocks from M's upper part,
// diagonal blocks from the saved Rd, zeros below the diagonal.
__global__ void assemble_r_kernel(int n, const double* __restrict__ M, long long ld, long long sm,
                                  const double* __restrict__ Rd, long long srd_b, double* __restrict__ R,
                                  long long ldr, long long sr) {
    const int b = blockIdx.y;
    const long long total = (long long)n * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / n, i = e - j * n;
        double v = 0.0;
        if (i <= j) {
            const long long pi = i / kNB, pj = j / kNB;
            v = pi == pj ? Rd[b * srd_b + pi * kNB * kNB + (i % kNB) + (j % kNB) * kNB] : M[b * sm + i + j * ld];
        }
        R[b * sr + i + j * ldr] = v;
    }
}

struct Geometry {
    int G, rows;
    int variant;   // index into kLeafVariants, or -1: panel_kernel
};

// The register-leaf kernel's shapes, by the rows a workgroup holds.
struct LeafVariant {
    int nt, rows;
    const void* solo;    // one workgroup per matrix
    const void* multi;   // several, cooperative
};
const LeafVariant kLeafVariants[] = {
    {256, 256, (const void*)panel_leaf_kernel<256, 1, false>, (const void*)panel_leaf_kernel<256, 1, true>},
    {512, 512, (const void*)panel_leaf_kernel<512, 1, false>, (const void*)panel_leaf_kernel<512, 1, true>},
    {512, 1024, (const void*)panel_leaf_kernel<512, 2, false>, (const void*)panel_leaf_kernel<512, 2, true>},
    {512, 2048, (const void*)panel_leaf_kernel<512, 4, false>, (const void*)panel_leaf_kernel<512, 4, true>},
};
constexpr int kNumLeafVariants = sizeof(kLeafVariants) / sizeof(kLeafVariants[0]);

// One workgroup per matrix up to this many live rows.  Measured on gfx950, one
// 64-column panel, one workgroup against 256-row workgroups with their column
// exchange: 513 rows 155 against 166 us, 764 rows 170 against 172, 1024 rows 194
// against 166-176 (one matrix or eight alike).
constexpr int kSoloRows = 768;

// Rows each workgroup owns when the slab stays in global memory.
constexpr int kPanelRowsTarget = 256;

// Panels of the solves of zolo_pd_batched with at most this many live rows
// take one workgroup per matrix: an ordinary launch on the solve's own
// stream, instead of a cooperative launch on the panel stream that all
// concurrent solves share: about 410 us at 2048 rows where a cooperative panel takes
// 180, but the panels of sixteen solves overlap.
constexpr int kSinglePanelRows = 2048;

// At most this many workgroups share a matrix's panel: every column polls
// and sums one slot per workgroup.
constexpr int kPanelMaxG = 64;

int cu_count() {
    static int v = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        return cus;
    }();
    return v;
}

// Co-resident workgroups of a multi-workgroup register-leaf shape.
int leaf_coresident(int v) {
    static int cache[kNumLeafVariants] = {};
    static std::mutex mu;
    std::lock_guard<std::mutex> lock(mu);
    if (cache[v] == 0) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kLeafVariants[v].multi, kLeafVariants[v].nt, 0) !=
            hipSuccess)
            per_cu = 0;
        cache[v] = per_cu > 0 ? per_cu * cu_count() : -1;
    }
    return cache[v] > 0 ? cache[v] : 0;
}

// Co-resident workgroups of the global-memory panel kernel.
int global_coresident() {
    static int v = [] {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)panel_kernel, kPT, 0) != hipSuccess)
            return 0;
        return per_cu * cu_count();
    }();
    return v;
}

// Shapes that keep the whole panel in registers: one row per thread.
inline bool resident(int v) { return kLeafVariants[v].rows == kLeafVariants[v].nt; }
// The grid that puts each matrix's G workgroups on one XCD (workgroups are dealt
// to the XCDs round-robin; those without a matrix leave at once).
inline long long panel_spread(int G, int batch) { return (long long)kNumXcd * ((batch + kNumXcd - 1) / kNumXcd) * G; }

// One workgroup per matrix where that is enough (above), else a resident shape
// whose grid can put each matrix on one XCD, 256 rows a workgroup before 512, else
// the smallest workgroups that all fit on the GPU at once, at most kPanelMaxG a
// matrix.  The exchange within one XCD's L2 against across them, 64-column panel:
// 2048 rows 179 against 195 us, 4160 rows 214 against 232, eight of 8256 rows (512
// a workgroup) 249 against 266; one of 8256 rows with 512-row workgroups on one XCD
// 246 against 270 with 256 rows across all.  Matrices too tall for the last shape go to
// panel_kernel.
Geometry panel_geometry(int L, int batch, bool single) {
    if (L <= (single ? kSinglePanelRows : kSoloRows)) {
        int v = 0;
        while (L > kLeafVariants[v].rows) ++v;
        return {1, L, v};
    }
    for (int pass = 0; pass < 2; ++pass) {
        for (int v = 0; v < kNumLeafVariants; ++v) {
            int G = (L + kLeafVariants[v].rows - 1) / kLeafVariants[v].rows;
            if (pass == 0 && (!resident(v) || panel_spread(G, batch) > leaf_coresident(v))) continue;
            if (G > kPanelMaxG || G * (long long)batch > leaf_coresident(v)) continue;
            const int rows = ((L + G - 1) / G + 15) / 16 * 16;
            G = (L + rows - 1) / rows;
            return {G, rows, v};
        }
    }
    const int target = kPanelRowsTarget;
    int G = (L + target - 1) / target;
    if (G < 1) G = 1;
    int cap = global_coresident() / batch;
    if (cap < 1) cap = 1;
    if (G > cap) G = cap;
    int rows = (L + G - 1) / G;
    if (rows < 64) rows = 64;
    G = (L + rows - 1) / rows;
    return {G, rows, -1};
}

inline int live_rows(int m, int e, int p0, int nb) {
    const int end = m + p0 + nb < m + e ? m + p0 + nb : m + e;
    return end - p0;
}

}  // namespace

// The most panel workgroups one launch of any shape can use; sizes the buffers of
// per-workgroup partial sums, flags and column slots.
int panel_max_coresident() {
    int v = global_coresident();
    for (int i = 0; i < kNumLeafVariants; ++i) v = std::max(v, leaf_coresident(i));
    return v;
}

__global__ void cooperative_noop_kernel() {}

// One empty cooperative launch per device, before the library's first own
// stream beside the callers'.  The HIP runtime runs cooperative kernels on a queue of its own, made for the first of
// them; made after the process's streams have taken the hardware queues (4 by
// default) it shares one, and every later panel launch waits for it: a
// structured QR of 1025 x 881 x 5 took 10.0 ms where it takes 6.5.
hipError_t open_cooperative_queue(int device, hipStream_t st) {
    static std::mutex mu;
    static unsigned long long opened = 0;
    if (device < 0 || device >= 64) return hipSuccess;
    std::lock_guard<std::mutex> lock(mu);
    if (opened >> device & 1) return hipSuccess;
    void* args[] = {nullptr};
    const hipError_t e =
        hipLaunchCooperativeKernel((const void*)cooperative_noop_kernel, dim3(1), dim3(64), args, 0, st);
    if (e == hipSuccess) opened |= 1ull << device;
    return e;
}

hipError_t stack_init(int m, int n, const double* X, long long ldx, double* M, long long ld, long long sm,
                      const double* pivots, int batch, hipStream_t st) {
    if (batch > kMaxInlineAlpha) return hipErrorInvalidValue;
    ShiftArgs piv;
    piv.batch = batch;
    for (int b = 0; b < batch; ++b) piv.shift[b] = pivots[b];
    const long long total = ((long long)m + n) * n;
    long long grid = (total + 255) / 256;
    if (grid > 8192) grid = 8192;
    stack_init_kernel<<<(int)grid, 256, 0, st>>>(m, n, X, ldx, M, ld, sm, piv);
    return hipGetLastError();
}

hipError_t assemble_r(int n, const double* M, long long ld, long long sm, int batch, const QrWork& w, double* R,
                      long long ldr, long long sr, hipStream_t st) {
    const int npanels = (n + kNB - 1) / kNB;
    long long grid = ((long long)n * n + 255) / 256;
    if (grid > 4096) grid = 4096;
    assemble_r_kernel<<<dim3((int)grid, batch), 256, 0, st>>>(n, M, ld, sm, w.Rd, (long long)npanels * kNB * kNB,
                                                             R, ldr, sr);
    return hipGetLastError();
}

namespace {

// Launch of the panel kernel for panel p (columns p0 .. p0+nb-1).
hipError_t run_panel(int m, int e, int p, int nb, double* M, long long ld, long long sm, int batch, const QrWork& w,
                     long long stT, hipStream_t st) {
    const int p0 = p * kNB;
    const int L = live_rows(m, e, p0, nb);
    const Geometry geo = panel_geometry(L, batch, w.single_panels);
    // The partial-sum and flag buffers hold max_coresident workgroups.
    if ((long long)geo.G * batch > w.max_coresident && geo.G > 1) return hipErrorInvalidValue;
    PanelArgs pa;
    pa.L = L; pa.nb = nb; pa.G = geo.G; pa.rows_per_wg = geo.rows; pa.batch = batch;
    const long long spread = panel_spread(geo.G, batch);
    pa.local = geo.variant >= 0 && geo.G > 1 && spread <= leaf_coresident(geo.variant);
    pa.P = M + p0 + (long long)p0 * ld; pa.ld = ld; pa.sp = sm;
    pa.T = w.T + (long long)p * kNB * kNB; pa.st = stT;
    pa.Rd = w.Rd + (long long)p * kNB * kNB; pa.srd = stT;
    pa.partials = w.partials;
    pa.colslots = w.colslots;
    pa.flags = w.flags;
    pa.seq = (unsigned)p * kPanelExchanges;
    pa.error_flag = w.error_flag;
    pa.spin_limit = 1u << 24;
    const double flops = 4.0 * L * (double)nb * nb * batch, bytes = 16.0 * L * (double)nb * batch;
    void* args[] = {&pa};
    hipError_t err;
    if (geo.variant >= 0 && geo.G == 1) {
        // One workgroup per matrix needs no co-residency: an ordinary launch
        // on the solve's own stream, free to overlap other solves.
        const LeafVariant& v = kLeafVariants[geo.variant];
        StatScope sc("panel_leaf<one workgroup>", st, flops, bytes);
        err = hipLaunchKernel(v.solo, dim3(batch), dim3(v.nt), args, 0, st);
        sc.end();
        return err;
    }
    // Several solves at once (zolo_pd_batched): every cooperative panel goes
    // to one shared stream, so two panels never wait for each other's
    // workgroups to become resident; events order it against this solve.
    hipStream_t ps = st;
    if (w.panel_stream && w.panel_stream != st) {
        ps = w.panel_stream;
        if ((err = hipEventRecord(w.ev_ready, st)) != hipSuccess) return err;
        if ((err = hipStreamWaitEvent(ps, w.ev_ready, 0)) != hipSuccess) return err;
    }
    StatScope sc(geo.variant >= 0 ? "panel_leaf<workgroups>" : "panel_kernel<global>", ps, flops, bytes);
    if (geo.variant >= 0) {
        const LeafVariant& v = kLeafVariants[geo.variant];
        err = hipLaunchCooperativeKernel(v.multi, dim3(pa.local ? (int)spread : pa.G * batch), dim3(v.nt), args, 0, ps);
    } else {
        err = hipLaunchCooperativeKernel((const void*)panel_kernel, dim3(pa.G * batch), dim3(kPT), args, 0, ps);
    }
    sc.end();
    if (err == hipSuccess && ps != st) {
        if ((err = hipEventRecord(w.ev_done, ps)) != hipSuccess) return err;
        err = hipStreamWaitEvent(st, w.ev_done, 0);
    }
    return err;
}

// Reflectors and columns of C up to which wy_t_kernel takes W2: the updates
// inside a superblock (7-14 us against 16-20 in two launches).  With 256
// reflectors the depth of the product takes it to 25 us.
constexpr int kWyMaxRefl = 128, kWyMaxTrail = 256;

// W2 = op(T) W of a block reflector for few columns: W given as `pieces`
// partial products (sums over the split k-range, in order), T upper triangular
// with stored zeros below its diagonal.  A workgroup sums 16 columns of W into
// LDS and multiplies them on the matrix cores, a 16-row tile of the result per
// wave at a time.  Lane l takes the k-values 4 (l / 16) + u, u = 0..3, of each
// 16, so that T^T is read 32 contiguous bytes per lane.  Bound: launch and load
// latency; it replaces the sum of the pieces and a product, two launches of 5.5
// and 10-14 us, by one of 7-14.  With merge_wy_kernel: n = 2048 25.5 -> 24.7 ms,
// 1000 x 777 11.8 -> 11.2, structured QR 1025 x 881 x 5 5.65 -> 5.3, 32 uneven
// matrices 27.5 -> 25.9.
constexpr int kWyCols = 16, kWyThreads = 512;
__global__ __launch_bounds__(kWyThreads) void wy_t_kernel(int nbv, int trail, int transpose, const double* __restrict__ Tm,
                                                   long long ldt, long long stt, const double* __restrict__ Wp,
                                                   int pieces, long long ldw, long long sw, long long sz,
                                                   double* __restrict__ W2, long long ldw2, long long sw2) {
    __shared__ double s_w[kWyMaxRefl][kWyCols + 1];
    const int b = blockIdx.y, c0 = blockIdx.x * kWyCols, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int rows = (nbv + 15) / 16 * 16;
    const double* Tb = Tm + b * stt;
    const double* Wb = Wp + b * sw;
    constexpr int UE = 4, UZ = 8;                 // elements and pieces whose loads are in flight together
    for (int e0 = tid; e0 < rows * kWyCols; e0 += kWyThreads * UE) {
        const double* p[UE];
        double s[UE];
#pragma unroll
        for (int u = 0; u < UE; ++u) {
            const int e = min(e0 + kWyThreads * u, rows * kWyCols - 1);
            p[u] = Wb + min(e % rows, nbv - 1) + (long long)min(c0 + e / rows, trail - 1) * ldw;
            s[u] = 0.0;
        }
        for (int z = 0; z < pieces; z += UZ) {
            double v[UE][UZ];
#pragma unroll
            for (int u = 0; u < UE; ++u)
#pragma unroll
                for (int q = 0; q < UZ; ++q) v[u][q] = p[u][min(z + q, pieces - 1) * sz];
#pragma unroll
            for (int u = 0; u < UE; ++u)
#pragma unroll
                for (int q = 0; q < UZ; ++q) s[u] += keep_if(v[u][q], opaque(z + q < pieces ? -1 : 0));
        }
#pragma unroll
        for (int u = 0; u < UE; ++u) {
            const int e = e0 + kWyThreads * u;
            if (e < rows * kWyCols) s_w[e % rows][e / rows] = keep_if(s[u], opaque(e % rows < nbv ? -1 : 0));
        }
    }
    __syncthreads();
    for (int rt = tid >> 6; rt * 16 < rows; rt += kWyThreads / 64) {
        d4 acc = d4{0, 0, 0, 0};
        const int i = 16 * rt + l16, ic = min(i, nbv - 1);
        const int k0 = transpose ? 0 : 16 * rt, k1 = transpose ? 16 * rt + 16 : rows;   // T's nonzeros
        for (int k = k0; k < k1; k += 64) {       // four blocks' loads in flight
            double t[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int kc = min(k + 16 * (u >> 2) + 4 * lg + (u & 3), nbv - 1);
                t[u] = transpose ? Tb[kc + ic * ldt] : Tb[ic + kc * ldt];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + 16 * q < k1) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        acc = mfma_f64_16x16x4(t[4 * q + u], s_w[k + 16 * q + 4 * lg + u][l16], acc);
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 16 * rt + Mfma<double>::row(lane, e);
            if (r < nbv && c0 + l16 < trail) W2[b * sw2 + r + (long long)(c0 + l16) * ldw2] = acc[e];
        }
    }
}

// Applies the block reflector I - V T V^T (forward: its transpose, as in the
// factorisation; backward: itself, as in forming Q) of the nbv columns of V
// starting at column c0 to `trail` columns C starting at column c0 + nbv, over
// the live rows [c0, c0 + L).  T (ld ldt, batch stride stt) is upper
// triangular.  V's zeros above its unit diagonal, including an R block stored
// there by an earlier panel of the same block, are masked by the GEMM's
// triangular flags.  col_off skips that many columns of C first.
hipError_t apply_block(int L, int c0, int nbv, int trail, const double* Tm, long long ldt, long long stt,
                       bool transpose_t, double* M, long long ld, long long sm, int batch, const QrWork& w,
                       hipStream_t st, int col_off = 0) {
    if (trail <= 0) return hipSuccess;
    const double* V = M + c0 + (long long)c0 * ld;
    double* C = M + c0 + (long long)(c0 + nbv + col_off) * ld;
    const long long sw = (long long)kQrSuper * trail;
    GemmDesc g1;  // W = V^T C
    g1.m = nbv; g1.n = trail; g1.k = L; g1.transa = 1;
    g1.A = V; g1.lda = ld; g1.strideA = sm;
    g1.B = C; g1.ldb = ld; g1.strideB = sm;
    g1.C = w.W; g1.ldc = kQrSuper; g1.strideC = sw;
    g1.batch = batch; g1.flags = kAUpper;
    hipError_t err;
    if (nbv <= kWyMaxRefl && trail <= kWyMaxTrail) {  // W2 = T^T W (forward) or T W (backward)
        int pieces = 1;
        if ((err = gemm_split(g1, w.splitk, w.splitk_elems, st, &pieces)) != hipSuccess) return err;
        const long long per = (long long)nbv * trail;
        const bool split = pieces > 1;
        wy_t_kernel<<<dim3((trail + kWyCols - 1) / kWyCols, batch), kWyThreads, 0, st>>>(
            nbv, trail, transpose_t ? 1 : 0, Tm, ldt, stt, split ? w.splitk : w.W, pieces, split ? nbv : kQrSuper,
            split ? per : sw, per * batch, w.W2, kQrSuper, sw);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    } else {
        if ((err = gemm_split(g1, w.splitk, w.splitk_elems, st)) != hipSuccess) return err;
        GemmDesc g2;
        g2.m = nbv; g2.n = trail; g2.k = nbv; g2.transa = transpose_t ? 1 : 0;
        g2.A = Tm; g2.lda = ldt; g2.strideA = stt;
        g2.B = w.W; g2.ldb = kQrSuper; g2.strideB = sw;
        g2.C = w.W2; g2.ldc = kQrSuper; g2.strideC = sw;
        g2.batch = batch; g2.flags = transpose_t ? kALower : kAUpper;
        if ((err = gemm(g2, st)) != hipSuccess) return err;
    }
    GemmDesc g3;  // C -= V W2
    g3.m = L; g3.n = trail; g3.k = nbv;
    g3.A = V; g3.lda = ld; g3.strideA = sm;
    g3.B = w.W2; g3.ldb = kQrSuper; g3.strideB = sw;
    g3.Cin = C; g3.ldcin = ld; g3.strideCin = sm;
    g3.C = C; g3.ldc = ld; g3.strideC = sm;
    g3.alpha = -1.0; g3.beta = 1.0; g3.batch = batch; g3.flags = kALower;
    return gemm(g3, st);
}

// To = [T1, -T1 P T2; 0, T2], P = V1^T V2: the compact-WY factor of the product
// of the block reflectors of columns [c1, c1 + n1) (factor T1) and [c2, c2 + n2),
// c2 = c1 + n1 (factor T2); n1 a multiple of 16.  A workgroup takes 16 columns of
// T2: Y = P T2 into LDS, then -T1 Y, on the matrix cores; the blocks copied and
// zeroed are spread over the workgroups of a matrix.  Bound: launch and load
// latency; it replaces two products and a copy, 26-30 us in three launches.
constexpr int kMergeCols = 16, kMergeThreads = 512;
__global__ __launch_bounds__(kMergeThreads) void merge_wy_kernel(int n1, int n2, const double* __restrict__ P,
                                                                 long long ldp, long long sp,
                                                                 const double* __restrict__ T1, long long ld1,
                                                                 long long st1, const double* __restrict__ T2,
                                                                 long long ld2, long long st2,
                                                                 double* __restrict__ To, long long ldo,
                                                                 long long sto) {
    __shared__ double s_y[kQrBlock][kMergeCols + 1];
    const int b = blockIdx.y, c0 = blockIdx.x * kMergeCols, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lg = lane >> 4;
    const double* Pb = P + b * sp;
    const double* T1b = T1 + b * st1;
    const double* T2b = T2 + b * st2;
    double* Tob = To + b * sto;
    constexpr int NW = kMergeThreads / 64;
    // Four blocks of 16 along k have their loads in flight together; lane l
    // takes the k-values 4 (l / 16) + u of each block.
    for (int i0 = 16 * wave; i0 < n1; i0 += 16 * NW) {   // Y[:, c] = P T2[:, c], T2 zero below its diagonal
        const int jc = min(c0 + l16, n2 - 1), kend = min(n2, c0 + kMergeCols);
        d4 acc = d4{0, 0, 0, 0};
        for (int k = 0; k < kend; k += 64) {
            double x[16], y[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int kc = min(k + 16 * (u >> 2) + 4 * lg + (u & 3), n2 - 1);
                x[u] = Pb[i0 + l16 + kc * ldp];
                y[u] = T2b[kc + jc * ld2];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int in = opaque(k + 16 * (u >> 2) + 4 * lg + (u & 3) < n2 ? -1 : 0);
                acc = mfma_f64_16x16x4(keep_if(x[u], in), keep_if(y[u], in), acc);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) s_y[i0 + Mfma<double>::row(lane, e)][l16] = acc[e];
    }
    __syncthreads();
    for (int i0 = 16 * wave; i0 < n1; i0 += 16 * NW) {   // T12 = -T1 Y, T1 upper triangular
        d4 acc = d4{0, 0, 0, 0};
        for (int k = i0; k < n1; k += 64) {
            double x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                x[u] = T1b[i0 + l16 + min(k + 16 * (u >> 2) + 4 * lg + (u & 3), n1 - 1) * ld1];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + 16 * q < n1) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        acc = mfma_f64_16x16x4(-x[4 * q + u], s_y[k + 16 * q + 4 * lg + u][l16], acc);
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c0 + l16 < n2) Tob[i0 + Mfma<double>::row(lane, e) + (n1 + c0 + l16) * ldo] = acc[e];
    }
    // The copied and the zero blocks.
    const int nt = n1 + n2, stride = gridDim.x * kMergeThreads;
    for (int e0 = blockIdx.x * kMergeThreads + tid; e0 < nt * nt; e0 += 8 * stride) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = min(e0 + u * stride, nt * nt - 1), i = e % nt, j = e / nt;
            const double* src = j < n1 ? T1b + min(i, n1 - 1) + j * ld1 : T2b + max(i - n1, 0) + (j - n1) * ld2;
            v[u] = *src;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + u * stride, i = e % nt, j = e / nt;
            if (e < nt * nt && (i >= n1 || j < n1))   // not T12
                Tob[i + j * ldo] = keep_if(v[u], opaque(((i < n1) == (j < n1)) ? -1 : 0));
        }
    }
}

hipError_t merge_wy(int m, int e, int c1, int n1, const double* T1, long long ld1, long long st1, int n2,
                    const double* T2, long long ld2, long long st2, double* M, long long ld, long long sm, int batch,
                    const QrWork& w, double* To, long long ldo, long long sto, hipStream_t st) {
    const int c2 = c1 + n1;
    const int k = live_rows(m, e, c1, n1) - n1;  // rows [c2, end of V1's live rows): V1 is zero below
    const long long ss = (long long)kQrBlock * kQrBlock;
    double* P = w.S;
    GemmDesc g;  // P = V1^T V2 (n1 x n2); V2's part above its diagonal (zeros, or R of an
                 // earlier panel of its block) is masked
    g.m = n1; g.n = n2; g.k = k; g.transa = 1;
    g.A = M + c2 + (long long)c1 * ld; g.lda = ld; g.strideA = sm;
    g.B = M + c2 + (long long)c2 * ld; g.ldb = ld; g.strideB = sm;
    g.C = P; g.ldc = kQrBlock; g.strideC = ss;
    g.batch = batch; g.flags = kBLower;
    hipError_t err = gemm_split(g, w.splitk, w.splitk_elems, st);
    if (err != hipSuccess) return err;
    merge_wy_kernel<<<dim3((n2 + kMergeCols - 1) / kMergeCols, batch), kMergeThreads, 0, st>>>(
        n1, n2, P, kQrBlock, ss, T1, ld1, st1, T2, ld2, st2, To, ldo, sto);
    return hipGetLastError();
}

}  // namespace

// Panels of 64 columns, paired into 128-column blocks (factor Tb), paired
// into 256-column superblocks (factor Ts).  Inside a superblock each block's
// reflectors update the superblock's remaining columns; the rest of the
// matrix takes one rank-256 block-reflector update per superblock, so the
// trailing matrix is read and written once per 256 columns.  That update
// is done in two parts: the next superblock's 256 columns first, then the
// far columns.  With one matrix per launch (whose panels leave most of the
// GPU idle) and a second stream, the far part runs there while the next
// superblock's panels and inner updates proceed on the caller's stream
// (look-ahead); the next superblock's own trailing update waits for it.
// Both orders compute the same products in the same way (the same two
// column ranges), so the results do not depend on the stream.
hipError_t structured_geqrf(int m, int e, int n, double* M, long long ld, long long sm, int batch, const QrWork& w,
                            hipStream_t st) {
    if (batch > kMaxInlineAlpha || batch < 1) return hipErrorInvalidValue;
    const int npanels = (n + kNB - 1) / kNB;
    const int nblocks = (n + kQrBlock - 1) / kQrBlock;
    const int nsuper = (n + kQrSuper - 1) / kQrSuper;
    const long long stT = (long long)npanels * kNB * kNB;
    const long long stb = (long long)nblocks * kQrBlock * kQrBlock;
    const long long sts = (long long)nsuper * kQrSuper * kQrSuper;
    hipError_t err = hipSuccess;
    // Tags and flags start from zero; the first panel has the most live rows.
    if (panel_geometry(live_rows(m, e, 0, std::min(n, kNB)), batch, w.single_panels).G > 1) {
        if ((err = zero_ints(reinterpret_cast<int*>(w.flags), (int)w.flag_elems, st)) != hipSuccess) return err;
        if ((err = zero_ints(reinterpret_cast<int*>(w.colslots), (int)(2 * w.colslot_elems), st)) != hipSuccess)
            return err;
    }
    const bool lookahead = batch == 1 && !w.single_panels && w.side_stream && w.side_stream != st &&
                           w.ev_side_ready && w.ev_side_done && w.W_side && w.W2_side && w.splitk_side &&
                           (size_t)kQrSuper * n <= qr_w_elems(n, 1);
    bool side_pending = false;
    for (int Q = 0; Q < nsuper; ++Q) {
        const int s0 = Q * kQrSuper;
        const int nsq = n - s0 < kQrSuper ? n - s0 : kQrSuper, send = s0 + nsq;
        const int trail_s = n - send;
        for (int q = 2 * Q; q < 2 * Q + 2 && q < nblocks; ++q) {
            const int p0 = q * kQrBlock, p = 2 * q;
            const int nbq = n - p0 < kQrBlock ? n - p0 : kQrBlock;
            const int nb1 = nbq < kNB ? nbq : kNB, nb2 = nbq - nb1;
            const int trail_in = send - p0 - nbq;  // columns to the right inside the superblock
            const double* T1 = w.T + (long long)p * kNB * kNB;
            if ((err = run_panel(m, e, p, nb1, M, ld, sm, batch, w, stT, st)) != hipSuccess) return err;
            if (nb2 == 0) {
                err = apply_block(live_rows(m, e, p0, nb1), p0, nb1, trail_in, T1, kNB, stT, true, M, ld, sm, batch,
                                  w, st);
                if (err != hipSuccess) return err;
                continue;
            }
            err = apply_block(live_rows(m, e, p0, nb1), p0, nb1, nb2, T1, kNB, stT, true, M, ld, sm, batch, w, st);
            if (err != hipSuccess) return err;
            if ((err = run_panel(m, e, p + 1, nb2, M, ld, sm, batch, w, stT, st)) != hipSuccess) return err;
            if (trail_in <= 0 && trail_s <= 0) continue;  // no later update needs Tb
            double* Tb = w.Tb + (long long)q * kQrBlock * kQrBlock;
            err = merge_wy(m, e, p0, kNB, T1, kNB, stT, nb2, T1 + kNB * kNB, kNB, stT, M, ld, sm, batch, w, Tb,
                           kQrBlock, stb, st);
            if (err != hipSuccess) return err;
            err = apply_block(live_rows(m, e, p0, nbq), p0, nbq, trail_in, Tb, kQrBlock, stb, true, M, ld, sm, batch,
                              w, st);
            if (err != hipSuccess) return err;
        }
        if (trail_s <= 0) continue;
        // The superblock (two full blocks when anything follows it) on the rest.
        const int nB = nsq - kQrBlock;
        const double* TA = w.Tb + (long long)(2 * Q) * kQrBlock * kQrBlock;
        const double* TB = nB > kNB ? w.Tb + (long long)(2 * Q + 1) * kQrBlock * kQrBlock
                                    : w.T + (long long)(4 * Q + 2) * kNB * kNB;
        const long long ldB = nB > kNB ? kQrBlock : kNB, stB = nB > kNB ? stb : stT;
        double* Ts = w.Ts + (long long)Q * kQrSuper * kQrSuper;
        err = merge_wy(m, e, s0, kQrBlock, TA, kQrBlock, stb, nB, TB, ldB, stB, M, ld, sm, batch, w, Ts, kQrSuper, sts,
                       st);
        if (err != hipSuccess) return err;
        // Columns the far part of the previous superblock's update wrote are
        // read from here on.
        if (side_pending) {
            if ((err = hipStreamWaitEvent(st, w.ev_side_done, 0)) != hipSuccess) return err;
            side_pending = false;
        }
        const int L = live_rows(m, e, s0, nsq);
        const int ahead = trail_s < kQrSuper ? trail_s : kQrSuper;
        err = apply_block(L, s0, nsq, ahead, Ts, kQrSuper, sts, true, M, ld, sm, batch, w, st);
        if (err != hipSuccess) return err;
        const int far = trail_s - ahead;
        if (far <= 0) continue;
        // One matrix: the far part runs on the side buffers (batch 1 sizes)
        // on either stream, since its split-K depends on the buffer size.
        QrWork ws = w;
        if (batch == 1 && w.W_side && w.W2_side && w.splitk_side) {
            ws.W = w.W_side;
            ws.W2 = w.W2_side;
            ws.splitk = w.splitk_side;
            ws.splitk_elems = w.splitk_side_elems;
        }
        if (lookahead) {
            if ((err = hipEventRecord(w.ev_side_ready, st)) != hipSuccess) return err;
            if ((err = hipStreamWaitEvent(w.side_stream, w.ev_side_ready, 0)) != hipSuccess) return err;
            err = apply_block(L, s0, nsq, far, Ts, kQrSuper, sts, true, M, ld, sm, batch, ws, w.side_stream, ahead);
            if (err != hipSuccess) return err;
            if ((err = hipEventRecord(w.ev_side_done, w.side_stream)) != hipSuccess) return err;
            side_pending = true;
        } else {
            err = apply_block(L, s0, nsq, far, Ts, kQrSuper, sts, true, M, ld, sm, batch, ws, st, ahead);
            if (err != hipSuccess) return err;
        }
    }
    if (side_pending) return hipStreamWaitEvent(st, w.ev_side_done, 0);
    return hipSuccess;
}

hipError_t structured_orgqr(int m, int e, int n, double* M, long long ld, long long sm, int batch, const QrWork& w,
                            hipStream_t st) {
    const int npanels = (n + kNB - 1) / kNB;
    const int nblocks = (n + kQrBlock - 1) / kQrBlock;
    const int nsuper = (n + kQrSuper - 1) / kQrSuper;
    const long long stT = (long long)npanels * kNB * kNB;
    const long long stb = (long long)nblocks * kQrBlock * kQrBlock;
    const long long sts = (long long)nsuper * kQrSuper * kQrSuper;
    hipError_t err;
    // S_p = T_p V_top^T of every panel at once, into Rd (R's diagonal blocks
    // are not needed any more), and the zeros above the panels.
    const int full = n / kNB;
    for (int part = 0; part < 2; ++part) {
        const int p = part == 0 ? 0 : full, nb = part == 0 ? kNB : n - full * kNB;
        GemmDesc s;
        s.m = nb; s.n = nb; s.k = nb; s.transb = 1;
        s.batch = part == 0 ? full : 1; s.batch2 = batch;
        if (nb <= 0 || s.batch <= 0) continue;
        s.A = w.T + (long long)p * kNB * kNB; s.lda = kNB; s.strideA = (long long)kNB * kNB; s.strideA2 = stT;
        s.B = M + (long long)p * kNB * (ld + 1); s.ldb = ld; s.strideB = (long long)kNB * (ld + 1); s.strideB2 = sm;
        s.C = w.Rd + (long long)p * kNB * kNB; s.ldc = kNB; s.strideC = (long long)kNB * kNB; s.strideC2 = stT;
        s.flags = kAUpper | kBUpper;
        if ((err = gemm(s, st)) != hipSuccess) return err;
    }
    if (n > kNB) {
        zero_above_panels_kernel<<<dim3(std::min(8, (n + 255) / 256), std::min(n, 4096), batch), 256, 0, st>>>(n, M, ld, sm);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    for (int Q = nsuper - 1; Q >= 0; --Q) {
        const int s0 = Q * kQrSuper;
        const int nsq = n - s0 < kQrSuper ? n - s0 : kQrSuper, send = s0 + nsq;
        // The superblock's reflectors on the columns already formed to its right
        // (a superblock that is followed by columns holds two full blocks).
        if (n - send > 0) {
            err = apply_block(live_rows(m, e, s0, nsq), s0, nsq, n - send, w.Ts + (long long)Q * kQrSuper * kQrSuper,
                              kQrSuper, sts, false, M, ld, sm, batch, w, st);
            if (err != hipSuccess) return err;
        }
        for (int q = (2 * Q + 1 < nblocks ? 2 * Q + 1 : 2 * Q); q >= 2 * Q; --q) {
            const int p0 = q * kQrBlock;
            const int nbq = n - p0 < kQrBlock ? n - p0 : kQrBlock;
            const int trail = send - p0 - nbq;
            // The block's reflectors on the superblock's columns to its right.
            if (trail > 0) {
                if (nbq > kNB)
                    err = apply_block(live_rows(m, e, p0, nbq), p0, nbq, trail,
                                      w.Tb + (long long)q * kQrBlock * kQrBlock, kQrBlock, stb, false, M, ld, sm, batch,
                                      w, st);
                else
                    err = apply_block(live_rows(m, e, p0, nbq), p0, nbq, trail, w.T + (long long)(2 * q) * kNB * kNB,
                                      kNB, stT, false, M, ld, sm, batch, w, st);
                if (err != hipSuccess) return err;
            }
            // The block's own columns, panel by panel from the last.
            for (int p = (nbq > kNB ? 2 * q + 1 : 2 * q); p >= 2 * q; --p) {
                const int pp0 = p * kNB;
                const int nb = n - pp0 < kNB ? n - pp0 : kNB;
                const int L = live_rows(m, e, pp0, nb);
                const double* Tp = w.T + (long long)p * kNB * kNB;
                double* V = M + pp0 + (long long)pp0 * ld;
                const int inblock = p0 + nbq - pp0 - nb;
                if ((err = apply_block(L, pp0, nb, inblock, Tp, kNB, stT, false, M, ld, sm, batch, w, st)) !=
                    hipSuccess)
                    return err;
                orgqr_panel_kernel<<<dim3((L + 63) / 64, batch), 256, 0, st>>>(
                    L, nb, V, ld, sm, w.Rd + (long long)p * kNB * kNB, stT);
                if ((err = hipGetLastError()) != hipSuccess) return err;
            }
        }
    }
    return hipSuccess;
}

}  // namespace zolo
