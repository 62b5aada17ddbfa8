// Plain FP64 symmetric eigensolver of Zolo-SVD (Algorithm 2: H = V diag(S) V^T
// once A = Qp H), on gfx950.  Three stages, as in the eigensolvers the paper
// builds on (Section 2.3):
//
//  1. Householder tridiagonalisation Q^T H Q = T, blocked: panels of kTB
//     columns, each column's reflector from a matrix-vector product with the
//     trailing matrix corrected by the panel's earlier reflectors (the
//     trailing matrix itself is updated once per panel by a rank-2 kTB
//     product on the matrix cores).  The matrix-vector product reads the
//     trailing matrix once per column: this stage is bound by HBM bandwidth.
//  2. Divide and conquer on T (Cuppen's method): T splits into 1 x 1 blocks
//     by removing every off-diagonal coupling (a rank-one term each); blocks
//     are merged pairwise, bottom up, each merge solving the eigenproblem of
//     D + rho z z^T: deflation, the secular equation by a bracketed rational
//     iteration (one wave per root), Gu-Eisenstat eigenvectors, and the product of the
//     merged block's eigenvectors with that solution (matrix cores).
//  3. Back-transformation V = Q V_T with the reflectors of stage 1 in
//     blocks of kBT, on the matrix cores.
// The eigenvalues come back in descending order with matching columns.
#include "eig_dc.hpp"
#include "misc.hpp"

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <numeric>
#include <vector>

namespace zolo {
namespace {

constexpr int kTB = 32;       // tridiagonalisation panel width
constexpr int kBT = 256;      // reflectors per block of the back-transformation
constexpr int kFT = 128;      // reflectors whose T factor one workgroup forms in LDS
constexpr int kET = 256;      // threads per workgroup
constexpr int kMaxG = 512;    // workgroups of trd_product (partial sums)

__device__ inline double block_sum256(double v, double* sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// ---------------------------------------------------------------------------
// Stage 1.  Panel starting at column j0; column j = j0 + c.  V's columns are
// the reflectors v_{j0..j-1}, stored in A below their explicit unit (row
// j' + 1 of column j'); W holds w'_c (before the alpha_c v_c term, which
// consumers add on the fly: w_c = w'_c + alpha_c v_c).
//
// Two launches per column.  trd_product multiplies the trailing matrix by the
// column x below its first subdiagonal entry as it stands, before the norm of x
// is known: with v = [1; s x], A v = A e_1 + s A x, and the same for V^T v, W^T v and
// v^T A v.  trd_column then forms the reflector, w' of its column and the
// update of the next column on the same rows, so that V and W are read once.
// ---------------------------------------------------------------------------
struct TrdArgs {
    int n, j, j0, c;
    double* A; long long lda;
    double* W; long long ldw;      // n x kTB, w'_c
    double* alpha;                 // kTB: alpha_c
    double* tau;                   // n: tau_j
    double* d; double* e;          // n: diagonal, off-diagonal of T
    double* xa;                    // n: first subdiagonal entry of each column before its reflector
    double* yr; double* a1;        // n: (A x)_i over rows >= j + 2, and A[j + 1][i]
    double* pq;                    // 2 kTB: V^T x, W'^T x over the same rows
    const double* sq;              // sums of squares of x of column j - 1, gA of them
    double* sq_next;               // row groups: those of column j
    double* partY;                 // 2 kMaxG: sums of a1_i x_i and yr_i x_i, i >= j + 2
    int gA, gY;                    // partial counts written by the producers (sq, partY)
    double* P; double* Q;          // n x 2 kTB: [V W] and [W V] of the panel's trailing rows
};

constexpr int kTrdRows = 64;       // rows per workgroup of trd_column

// With c > 0: the reflector of column p = j - 1 (beta, tau, v), then
//   w' = tau (y - V (W^T v) - W (V^T v)) on rows >= j, y = A22 v,
//   alpha = -tau (w'^T v) / 2,  w'^T v = tau (v^T y - 2 (V^T v)^T (W^T v)),
// v and w' stored.  Then, unless `finish`, column j takes the panel's update,
//   A[j:n, j] -= V[j:n] W[j]^T + W[j:n] V[j]^T,
// with its diagonal, its first subdiagonal entry and the partial sums of
// a[j+2:n, j]^2; `finish` (end of a panel) writes the operands [V W], [W V] of
// the trailing update instead.  One row per lane, the earlier columns of V
// and W spread over the four waves; what every row needs of row j is formed
// by each workgroup for itself.  Nothing orders the workgroups of a launch: a
// word that one of them writes is read by no other.  The sums of squares of
// column j - 1 and of column j therefore lie in two arrays that change places
// from launch to launch, and the columns of V and W and the words of column
// j - 1 that this launch forms (A[j:n, j - 1], W[:, c - 1], alpha[c - 1], xa[j])
// are not among those read for all rows (columns up to c - 2, xa[j - 1]).
__global__ __launch_bounds__(kET) void trd_column(TrdArgs a, int finish) {
    __shared__ double sh[3][4];
    __shared__ double s_p[kTB], s_q[kTB], s_al[kTB], s_wj[kTB], s_vj[kTB], s_sc[4];
    __shared__ double s_acc[4][kTrdRows][2];
    const int n = a.n, j = a.j, c = a.c, j0 = a.j0, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Everything that does not wait for the reflector is loaded first: the
    // wave's share of the earlier columns on this lane's row, and what wave 0
    // needs of row j and of the row itself.
    const int row = j + blockIdx.x * kTrdRows + lane, rc = min(row, n - 1);
    constexpr int S = kTB / 4;
    // With fewer than two earlier columns none of these words is used: they then
    // come from a column that this launch leaves alone (a branch around the
    // loads cost 1 % of the eigensolver).
    const int last = c > 1 ? c - 2 : min(c + 1, n - 1 - j0), w0 = c > 1 ? wave : last;
    double vr[S], wr[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int k = min(w0 + 4 * u, last);
        vr[u] = a.A[rc + (long long)(j0 + k) * a.lda];
        wr[u] = a.W[rc + (long long)k * a.ldw];
    }
    const int kl = min(c > 1 ? lane : last, last);
    const double rv = a.A[j + (long long)(j0 + kl) * a.lda], rw = a.W[j + (long long)kl * a.ldw];
    const double ral = a.alpha[kl], rpv = a.pq[kl], rpw = a.pq[kTB + kl];
    const double x1 = a.xa[j > 0 ? j - 1 : 1], y1 = a.a1[j], y2 = a.yr[j];
    const double ca1 = a.a1[rc], cyr = a.yr[rc], cp = a.A[rc + (long long)max(j - 1, 0) * a.lda];
    const double cj = a.A[rc + (long long)j * a.lda];
    if (c > 0) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int i = tid; i < a.gA; i += kET) s0 += a.sq[i];
        for (int i = tid; i < a.gY; i += kET) {
            s1 += a.partY[2 * i];
            s2 += a.partY[2 * i + 1];
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane == 0) {
            sh[0][wave] = s0;
            sh[1][wave] = s1;
            sh[2][wave] = s2;
        }
        __syncthreads();
        if (wave == 0) {
            const double xx = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]);
            const double ax = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
            const double yx = (sh[2][0] + sh[2][1]) + (sh[2][2] + sh[2][3]);
            double beta = x1, t = 0.0, scale = 0.0;
            if (xx > 0.0) householder(x1, xx, beta, t, scale);
            const int k = lane;
            double vk = 0.0, wk = 0.0, pk = 0.0, qk = 0.0, alk = 0.0;
            if (k < c - 1) {
                alk = ral;
                vk = rv;
                pk = vk + scale * rpv;                                   // V^T v
                qk = rw + scale * rpw + alk * pk;                        // W^T v
                wk = rw + alk * vk;                                      // W[j][k]
            }
            const double pq = wave_sum(pk * qk), vq = wave_sum(vk * qk + wk * pk);
            const double yj = y1 + scale * y2;
            const double al = -0.5 * t * t * (yj + scale * (ax + scale * yx) - 2.0 * pq);
            if (k == c - 1) {
                alk = al;
                vk = 1.0;
                wk = t * (yj - vq) + al;
            }
            if (k < c) {
                s_p[k] = pk;
                s_q[k] = qk;
                s_al[k] = alk;
                s_vj[k] = vk;
                s_wj[k] = wk;
            }
            if (lane == 0) {
                s_sc[0] = t;
                s_sc[1] = scale;
                if (blockIdx.x == 0) {
                    a.e[j - 1] = beta;
                    a.tau[j - 1] = t;
                    a.alpha[c - 1] = al;
                }
            }
        }
        __syncthreads();
    }
    // This lane's row: the sums over the wave's share of the earlier columns.
    double u0 = 0.0, u1 = 0.0;
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int k = wave + 4 * u;
        if (k >= c - 1) break;
        const double v = vr[u], w = wr[u] + s_al[k] * v;
        u0 += v * s_q[k] + w * s_p[k];
        u1 += v * s_wj[k] + w * s_vj[k];
        if (finish && row < n) {
            const long long at = row + (long long)k * n, jb = (long long)c * n;
            a.P[at] = v;
            a.P[at + jb] = w;
            a.Q[at] = w;
            a.Q[at + jb] = v;
        }
    }
    s_acc[wave][lane][0] = u0;
    s_acc[wave][lane][1] = u1;
    __syncthreads();
    if (wave != 0) return;
    double part = 0.0;
    if (row < n) {
        u0 = (s_acc[0][lane][0] + s_acc[1][lane][0]) + (s_acc[2][lane][0] + s_acc[3][lane][0]);
        u1 = (s_acc[0][lane][1] + s_acc[1][lane][1]) + (s_acc[2][lane][1] + s_acc[3][lane][1]);
        double v = 0.0, w = 0.0;
        if (c > 0) {
            const double t = s_sc[0], scale = s_sc[1];
            v = row == j ? 1.0 : scale * cp;
            const double w1 = t * (ca1 + scale * cyr - u0);
            a.A[row + (long long)(j - 1) * a.lda] = v;
            a.W[row + (long long)(c - 1) * a.ldw] = w1;
            w = w1 + s_al[c - 1] * v;
        }
        if (finish) {
            const long long at = row + (long long)(c - 1) * n, jb = (long long)c * n;
            a.P[at] = v;
            a.P[at + jb] = w;
            a.Q[at] = w;
            a.Q[at + jb] = v;
        } else {
            double x = cj;
            if (c > 0) x -= u1 + v * s_wj[c - 1] + w * s_vj[c - 1];
            a.A[row + (long long)j * a.lda] = x;
            if (row == j) a.d[j] = x;
            if (row == j + 1) a.xa[j] = x;
            if (row >= j + 2) part = x * x;
        }
    }
    if (finish) return;
    part = wave_sum(part);
    if (lane == 0) a.sq_next[blockIdx.x] = part;
}

// x = A[j+2:n, j]: yr_i = A[j+2:n, i]^T x and a1_i = A[j+1][i] for the trailing
// columns i > j, V^T x and W'^T x, and per workgroup the sums of a1_i x_i and
// yr_i x_i.  A wave takes C columns at a time (x is read once for them), two
// rows per lane and load.  Bound: the trailing matrix read once per column,
// n^3 / 3 doubles over the reduction: 4.8 TB/s at n = 2048-4096 (15.9 us a
// column), launch latency below.  One wave per column with one 8-byte load at a
// time took 20 us a column over the whole reduction of n = 4096, and the column
// update and w two launches of 5.3 us; with these two kernels and one rank-64
// trailing update per panel in place of two of rank 32, Zolo-SVD went from 231 to
// 166 ms, 900 x 600 from 20.5 to 16.6 ms; with the sums over a wave in registers and
// the reflector without divisions from 153.5 to 149.7 and 14.2 to 13.5.
template <int C>
__global__ __launch_bounds__(kET) void trd_product(TrdArgs a) {
    typedef double pair_u __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int U = C == 1 ? 4 : (C == 2 ? 4 : 2);   // 16-byte loads in flight per column
    __shared__ double sh[2][4];
    const int n = a.n, j = a.j, c = a.c, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nt = n - j - 1, items = nt + 2 * c, nw = gridDim.x * 4;
    const double* x = a.A + (long long)j * a.lda;
    double ax = 0.0, yx = 0.0;
    for (int g = blockIdx.x * 4 + wave; g * C < items; g += nw) {
        const double* col[C];
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const int it = min(g * C + u, items - 1);
            col[u] = it < nt ? a.A + (long long)(j + 1 + it) * a.lda
                             : (it < nt + c ? a.A + (long long)(a.j0 + it - nt) * a.lda
                                            : a.W + (long long)(it - nt - c) * a.ldw);
        }
        double s[C][2];
#pragma unroll
        for (int u = 0; u < C; ++u) s[u][0] = s[u][1] = 0.0;
        int r0 = j + 2;
        for (; r0 + 128 * U <= n; r0 += 128 * U) {
            pair_u xv[U], cv[C][U];
#pragma unroll
            for (int q = 0; q < U; ++q) xv[q] = *reinterpret_cast<const pair_u*>(x + r0 + 128 * q + 2 * lane);
#pragma unroll
            for (int u = 0; u < C; ++u)
#pragma unroll
                for (int q = 0; q < U; ++q) cv[u][q] = *reinterpret_cast<const pair_u*>(col[u] + r0 + 128 * q + 2 * lane);
#pragma unroll
            for (int u = 0; u < C; ++u)
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    s[u][0] += cv[u][q][0] * xv[q][0];
                    s[u][1] += cv[u][q][1] * xv[q][1];
                }
        }
        // The rest (fewer than 128 U rows), single rows from clamped addresses.
        if (r0 < n) {
            double xv[2 * U], cv[C][2 * U];
#pragma unroll
            for (int q = 0; q < 2 * U; ++q) xv[q] = x[min(r0 + 64 * q + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < C; ++u)
#pragma unroll
                for (int q = 0; q < 2 * U; ++q) cv[u][q] = col[u][min(r0 + 64 * q + lane, n - 1)];
#pragma unroll
            for (int q = 0; q < 2 * U; ++q) {
                const double xq = keep_if(xv[q], opaque(r0 + 64 * q + lane < n ? -1 : 0));
#pragma unroll
                for (int u = 0; u < C; ++u) s[u][q & 1] += cv[u][q] * xq;
            }
        }
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const double y = wave_sum(s[u][0] + s[u][1]);
            const int it = g * C + u;
            if (lane == 0 && it < items) {
                if (it < nt) {
                    const double first = col[u][j + 1];
                    a.yr[j + 1 + it] = y;
                    a.a1[j + 1 + it] = first;
                    if (it > 0) {
                        const double xi = x[j + 1 + it];
                        ax += first * xi;
                        yx += y * xi;
                    }
                } else {
                    a.pq[it < nt + c ? it - nt : kTB + it - nt - c] = y;
                }
            }
        }
    }
    if (lane == 0) {
        sh[0][wave] = ax;
        sh[1][wave] = yx;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double* p = sh[threadIdx.x];
        a.partY[2 * blockIdx.x + threadIdx.x] = (p[0] + p[1]) + (p[2] + p[3]);
    }
}

// The reduction forms x^T A x of raw columns x, of the order of ||A||^3: right
// for norms from about 1e-100 to 1e100 alone (with entries of 1e-106 the
// eigenvalues were off by 1e-2 ||A||, with 1e104 NaN).  A matrix whose largest
// entry lies outside 2^+-32 is therefore scaled into [1, 2) by a power of two, and
// its eigenvalues are scaled back on the host: every operation of the solver
// commutes with that, so the eigenvectors keep their bits.  One pass over the
// lower triangle for the largest entry (partial maxima, one per workgroup), and
// the launch that makes the identity of the merges applies the scale.  From
// subnormal entries up the scale stays a normal number.  A matrix with a NaN or an
// infinity is refused (scale 0) and solved as zero: NaN eigenvalues have no ranks,
// and the merges index by rank.
constexpr int kMaxParts = 256;     // workgroups of trd_max
constexpr int kScaleFree = 32, kScaleMost = 1000;

__device__ inline double block_max256(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

__global__ __launch_bounds__(kET) void trd_max(int n, const double* A, long long lda, double* part) {
    __shared__ double sh[4];
    double m = 0.0;
    for (int j = blockIdx.x; j < n; j += gridDim.x)
        for (int i = j + threadIdx.x; i < n; i += kET) {
            const double v = fabs(A[i + j * lda]);
            m = fmax(m, v <= DBL_MAX ? v : INFINITY);
        }
    m = block_max256(m, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// A <- scale A where that is needed (0 A = 0 for a refused one), *scale, and Q = I.
__global__ __launch_bounds__(kET) void trd_scale(int n, double* A, long long lda, const double* part, int nparts,
                                                 double* scale, double* Q, long long ldq) {
    __shared__ double sh[4];
    const double m = block_max256((int)threadIdx.x < nparts ? part[threadIdx.x] : 0.0, sh);
    const bool apply = m > 0.0 && (m < ldexp(1.0, -kScaleFree) || m >= ldexp(1.0, kScaleFree));
    double s = 1.0;
    if (apply) s = m <= DBL_MAX ? ldexp(1.0, max(-kScaleMost, min(kScaleMost, -ilogb(m)))) : 0.0;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *scale = s;
    const int step = gridDim.x * kET;
    for (int j = blockIdx.y; j < n; j += gridDim.y)
        for (int i = blockIdx.x * kET + threadIdx.x; i < n; i += step) {
            if (apply) A[i + j * lda] = s > 0.0 ? s * A[i + j * lda] : 0.0;
            Q[i + j * ldq] = i == j ? 1.0 : 0.0;
        }
}

// After the reduction: d[n-1], and zeros on and above the diagonal of A so
// that the reflector blocks read as unit lower trapezoidal matrices.
__global__ void trd_cleanup(int n, double* A, long long lda, double* d) {
    if (blockIdx.x == 0 && threadIdx.x == 0) d[n - 1] = A[(n - 1) + (long long)(n - 1) * lda];
    __syncthreads();
    const long long total = (long long)n * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long col = e / n, row = e - col * n;
        if (row <= col && !(row == n - 1 && col == n - 1)) A[row + col * lda] = 0.0;
    }
}

// T factors (compact WY) of kFT reflectors each from S = V^T V, one workgroup
// of 8 waves per factor: workgroup x forms the diagonal block of columns
// kFT x ... of the reflectors, half x % 2 of back-transformation block x / 2.
// Each wave first forms the T of its own 16 reflectors (lane = row, in
// registers), then neighbouring factors are merged in LDS,
//   T12 = -T1 (S12 T2),
// on the matrix cores for 16, 32 and 64 reflectors a side.  Reflectors past
// nref get tau = 0, so their rows and columns of T are zero.  Bound: latency of
// the 16-column recurrence and of the three merges.  One thread per row with
// T in global memory and a barrier per column took 0.73-0.87 ms for 128
// reflectors (28 ms of Zolo-SVD at n = 4096; 900 x 600: 3.6 of 36 ms).  With
// this kernel, one launch for all blocks, S and V aligned for the pipelined
// GEMM and 256 reflectors a block, the two calls went from 288 to 248 and from
// 36.0 to 32.1 ms.  Up to kFT reflectors in all there is one factor, of leading
// dimension ld = kFT: one workgroup clears, merges and stores the columns there are, and
// S need not hold zeros past them (with the blocks' whole 256 columns, cleared and merged
// by two more products, order 2 took 204 us instead of 150, order 24 506 instead of 469).
constexpr int kFTld = kFT + 2;
constexpr size_t kFormTLds = (size_t)kFTld * kFT * sizeof(double);
__global__ __launch_bounds__(512) void form_t(int nref, const double* S, const double* tau, double* T, int ld) {
    extern __shared__ double Tl[];               // T[i][j] at i + j kFTld
    __shared__ double Sl[kFT / 16][16][17];      // S's 16 x 16 diagonal blocks
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int c0 = blockIdx.x * kFT, half = (blockIdx.x & 1) * kFT;
    const long long blk = (long long)(blockIdx.x >> 1) * ld * ld;
    const double* Sb = S + blk + half + (long long)half * ld;
    const int cols = ld == kFT ? (nref + 15) / 16 * 16 : kFT;
    for (int e = tid; e < kFTld * cols; e += 512) Tl[e] = 0.0;
    for (int e = tid; e < cols * 16; e += 512) {
        const int q = e / 256, r = e % 16, c = (e / 16) % 16;
        Sl[q][r][c] = r < c && c0 + 16 * q + c < nref ? Sb[16 * q + r + (long long)(16 * q + c) * ld] : 0.0;
    }
    __syncthreads();
    if (16 * w < cols) {
        // T[i][c] = -tau_c sum_{i <= k < c} T[i][k] S[k][c], T[c][c] = tau_c.
        const int i = lane & 15;
        double row[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const int gc = c0 + 16 * w + c;
            const double t = gc < nref ? tau[gc] : 0.0;
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < c; ++k) s += row[k] * Sl[w][k][c];
            row[c] = i == c ? t : (i < c ? -t * s : 0.0);
        }
        if (lane < 16) {
#pragma unroll
            for (int c = 0; c < 16; ++c) Tl[16 * w + i + (16 * w + c) * kFTld] = row[c];
        }
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    for (int s = 16; s < cols; s *= 2) {
        const int ts = s / 16, per = ts * ts;    // 16 x 16 tiles of one merge
        const int total = kFT / (2 * s) * per;   // 4, 8, 16
        d4 acc[2];
        // Y = S12 T2 into the place of T12, then T12 = -T1 Y.
        for (int phase = 0; phase < 2; ++phase) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = w + 8 * u;
                acc[u] = d4{0, 0, 0, 0};
                if (tile >= total) continue;
                const int o = tile / per * 2 * s, ti = tile % per % ts * 16, tj = tile % per / ts * 16;
                if (o + s + tj >= cols) continue;      // no columns there
                const int kend = phase == 0 ? min(s, tj + 16) : s;   // T2 is zero below its diagonal
                for (int k = 0; k < kend; k += 4) {
                    double x, y;
                    if (phase == 0) {
                        const int at = o + s + k + lk;
                        x = c0 + at < nref ? Sb[o + ti + li + (long long)at * ld] : 0.0;
                        y = Tl[at + (o + s + tj + li) * kFTld];
                    } else {
                        x = Tl[o + ti + li + (o + k + lk) * kFTld];
                        y = Tl[o + k + lk + (o + s + tj + li) * kFTld];
                    }
                    acc[u] = mfma_f64_16x16x4(x, y, acc[u]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = w + 8 * u;
                if (tile >= total) continue;
                const int o = tile / per * 2 * s, ti = tile % per % ts * 16, tj = tile % per / ts * 16;
                if (o + s + tj >= cols) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    Tl[o + ti + Mfma<double>::row(lane, e) + (o + s + tj + li) * kFTld] =
                        phase == 0 ? acc[u][e] : -acc[u][e];
            }
            __syncthreads();
        }
    }
    // The diagonal block of T, and zeros below it.
    double* Tb = T + blk + (long long)half * ld;
    for (int e = tid; e < kFT * cols; e += 512) {
        const int i = e % kFT, j = e / kFT;
        Tb[half + i + (long long)j * ld] = Tl[i + j * kFTld];
        if (half == 0 && ld == kBT) Tb[kFT + i + (long long)j * ld] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// Stage 2.  Divide and conquer.  Level with half-width s: group g covers
// [A0, A0 + k), A0 = 2 s g, k = min(2 s, n - A0); it is a merge when
// A0 + s < n, else the block is carried unchanged.  Every block keeps its
// eigenvalues in ascending order (and its eigenvector columns to match), so
// the poles of a merge come in order by merging two sorted lists.  Per-group
// arrays live at offset A0 of length-n arrays.
// ---------------------------------------------------------------------------
struct DcArgs {
    int n, s;
    const double* e;                 // couplings
    double* D;                       // eigenvalues of the current blocks (ascending per block)
    double* Qa; double* Qb; double* U; long long ld;
    double *ds, *zs, *pole, *zp, *dval, *rc, *rs, *tau, *zh, *vals, *rho;
    int *colsrc, *src, *ri, *rj, *org, *inv, *K, *nrot;
};

__global__ void dc_init(int n, const double* d, const double* e, double* D) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) D[i] = d[i] - (i > 0 ? fabs(e[i - 1]) : 0.0) - (i + 1 < n ? fabs(e[i]) : 0.0);
}

constexpr int kScanChunk = 1024;

// One workgroup per group: the merged poles in ascending order with their z
// (from the facing rows of the two blocks), normalisation, and the
// deflation scan (thread 0, over chunks staged in LDS).  Bound: that scan, 85 -> 36 ns a
// pole with the last kept pole in a register and no root and divisions for poles
// that are clearly apart: all merges of n = 4096 3.6 -> 1.8 ms.
__global__ __launch_bounds__(kET) void dc_prepare(DcArgs a) {
    __shared__ double sh[4];
    __shared__ double cd[kScanChunk], cz[kScanChunk];
    const int g = blockIdx.x, s = a.s, n = a.n, A0 = 2 * s * g, k = min(2 * s, n - A0);
    if (A0 + s >= n) {
        if (threadIdx.x == 0) a.K[g] = -1;
        return;
    }
    const double beta = a.e[A0 + s - 1], sg = beta >= 0.0 ? 1.0 : -1.0;
    const double* D = a.D + A0;
    for (int c = threadIdx.x; c < k; c += kET) {
        const double x = D[c];
        int lo, hi;
        if (c < s) {             // count of the second block's values < x
            lo = s; hi = k;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (D[mid] < x) lo = mid + 1;
                else hi = mid;
            }
            lo -= s;
        } else {                 // count of the first block's values <= x
            lo = 0; hi = s;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (D[mid] <= x) lo = mid + 1;
                else hi = mid;
            }
        }
        const int pos = (c < s ? c : c - s) + lo;
        const long long col = (long long)(A0 + c) * a.ld;
        a.ds[A0 + pos] = x;
        a.zs[A0 + pos] = c < s ? a.Qa[(A0 + s - 1) + col] : sg * a.Qa[(A0 + s) + col];
        a.colsrc[A0 + pos] = c;
    }
    __syncthreads();
    double zz = 0.0, dm = 0.0;
    for (int t = threadIdx.x; t < k; t += kET) {
        const double z = a.zs[A0 + t];
        zz += z * z;
        dm = fmax(dm, fabs(a.ds[A0 + t]));
    }
    zz = block_sum256(zz, sh);
    // max over the workgroup
    for (int off = 32; off > 0; off >>= 1) dm = fmax(dm, __shfl_xor(dm, off, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = dm;
    __syncthreads();
    dm = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    const double zn = sqrt(zz);
    double zm = 0.0;
    for (int t = threadIdx.x; t < k; t += kET) {
        const double z = zn > 0.0 ? a.zs[A0 + t] / zn : 0.0;
        a.zs[A0 + t] = z;
        zm = fmax(zm, fabs(z));
    }
    for (int off = 32; off > 0; off >>= 1) zm = fmax(zm, __shfl_xor(zm, off, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = zm;
    __syncthreads();
    zm = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    const double r = fabs(beta) * zn * zn;
    dc::DeflateScan sc;
    sc.pole = a.pole + A0; sc.zp = a.zp + A0; sc.dval = a.dval + A0; sc.rc = a.rc + A0; sc.rs = a.rs + A0;
    sc.src = a.src + A0; sc.ri = a.ri + A0; sc.rj = a.rj + A0;
    sc.begin(k, r, 8.0 * dc::kEps * fmax(dm, r * zm));
    for (int c0 = 0; c0 < k; c0 += kScanChunk) {
        const int cn = min(kScanChunk, k - c0);
        __syncthreads();
        for (int t = threadIdx.x; t < cn; t += kET) {
            cd[t] = a.ds[A0 + c0 + t];
            cz[t] = a.zs[A0 + c0 + t];
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int t = 0; t < cn; ++t) sc.step(c0 + t, cd[t], cz[t]);
    }
    if (threadIdx.x == 0) {
        a.K[g] = sc.finish();
        a.nrot[g] = sc.nrot;
        a.rho[g] = r;
    }
}

// The deflating rotations on the block columns of each merge (row-parallel;
// rotation indices are sorted positions, mapped to block columns).
__global__ void dc_rotate(DcArgs a) {
    const int g = blockIdx.y, s = a.s, A0 = 2 * s * g;
    if (a.K[g] < 0) return;
    const int k = min(2 * s, a.n - A0), nr = a.nrot[g];
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < k; r += gridDim.x * blockDim.x) {
        double* row = a.Qa + (A0 + r);
        for (int t = 0; t < nr; ++t) {
            const long long ci = (long long)(A0 + a.colsrc[A0 + a.ri[A0 + t]]) * a.ld;
            const long long cj = (long long)(A0 + a.colsrc[A0 + a.rj[A0 + t]]) * a.ld;
            const double x = row[ci], y = row[cj], c = a.rc[A0 + t], sn = a.rs[A0 + t];
            row[ci] = c * x + sn * y;
            row[cj] = c * y - sn * x;
        }
    }
}

// One wave per root: the sums over the K poles are spread over its lanes, so
// a root costs about a dozen evaluations of K / 64 terms per lane.  Bound: FP64
// division (one per term).  One thread per root with plain bisection (some 60
// evaluations of K terms, one wave per 64 roots) left most of the chip idle:
// 111 ms of the 401 ms of Zolo-SVD at n = 4096, 19 of 55 ms at 900 x 600;
// with this kernel (and dc_lowner and dc_rank spread the same way) the two
// calls take 288 and 36 ms.
__global__ __launch_bounds__(kET) void dc_secular(DcArgs a) {
    const int p = blockIdx.x * (kET / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= a.n) return;
    const int g = p / (2 * a.s), A0 = 2 * a.s * g, t = p - A0, K = a.K[g];
    if (K < 0 || t >= K) return;
    const double* pole = a.pole + A0;
    const double* zp = a.zp + A0;
    const double rho = a.rho[g];
    auto sums = [&](double origin, double x, int split) {
        double f = 0.0, dpsi = 0.0, dphi = 0.0;
#pragma unroll 4
        for (int j = lane; j < K; j += 64) {
            const double z = zp[j], q = z / ((pole[j] - origin) - x);
            f += z * q;
            if (j <= split) dpsi += q * q;
            else dphi += q * q;
        }
        return dc::SecularSums{1.0 / rho + wave_sum(f), wave_sum(dpsi), wave_sum(dphi)};
    };
    int o;
    double tau;
    dc::secular_root(K, pole, rho, t, &o, &tau, sums);
    if (lane == 0) {
        a.org[p] = o;
        a.tau[p] = tau;
    }
}

// Gu-Eisenstat z and the new eigenvalues (roots, then deflated values), one
// wave per entry.
__global__ __launch_bounds__(kET) void dc_lowner(DcArgs a) {
    const int p = blockIdx.x * (kET / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= a.n) return;
    const int g = p / (2 * a.s), A0 = 2 * a.s * g, t = p - A0, K = a.K[g];
    if (K < 0 || t >= K) {
        if (lane == 0) a.vals[p] = K < 0 ? a.D[p] : a.dval[p];
        return;
    }
    double prod = dc::lowner_product(K, a.pole + A0, a.org + A0, a.tau + A0, t, lane, 64);
    for (int off = 32; off > 0; off >>= 1) prod *= __shfl_xor(prod, off, 64);
    if (lane == 0) {
        a.zh[p] = dc::lowner_z(K, a.pole + A0, a.zp[p], a.rho[g], a.org + A0, a.tau + A0, t, prod);
        a.vals[p] = a.pole[A0 + a.org[p]] + a.tau[p];
    }
}

// Ascending order of the new eigenvalues of each group: inv[A0 + rank] = t
// (one wave per value).
__global__ __launch_bounds__(kET) void dc_rank(DcArgs a) {
    const int p = blockIdx.x * (kET / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= a.n) return;
    const int g = p / (2 * a.s), A0 = 2 * a.s * g, t = p - A0, K = a.K[g];
    if (K < 0) {
        if (lane == 0) a.inv[p] = t;
        return;
    }
    const int k = min(2 * a.s, a.n - A0);
    const double x = a.vals[p];
    int rank = 0;
    for (int u = lane; u < k; u += 64) {
        const double y = a.vals[A0 + u];
        rank += (y < x || (y == x && u < t)) ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) rank += __shfl_xor(rank, off, 64);
    if (lane == 0) a.inv[A0 + rank] = t;
}

// One workgroup per output column p of the group's k x k block of U, and the
// eigenvalue D[p].  Carried blocks get identity columns.
__global__ __launch_bounds__(kET) void dc_vectors(DcArgs a) {
    __shared__ double sh[4];
    const int p = blockIdx.x;
    const int g = p / (2 * a.s), A0 = 2 * a.s * g, K = a.K[g];
    const int k = min(2 * a.s, a.n - A0);
    const int t = a.inv[p];
    double* col = a.U + A0 + (long long)p * a.ld;
    for (int r = threadIdx.x; r < k; r += kET) col[r] = 0.0;
    __syncthreads();
    if (K < 0) {
        if (threadIdx.x == 0) col[t] = 1.0;
        return;
    }
    if (threadIdx.x == 0) a.D[p] = a.vals[A0 + t];
    if (t >= K) {
        if (threadIdx.x == 0) col[a.colsrc[A0 + a.src[A0 + t]]] = 1.0;
        return;
    }
    const double* pole = a.pole + A0;
    const int o = a.org[A0 + t];
    const double tau = a.tau[A0 + t];
    double sum = 0.0;
    for (int j = threadIdx.x; j < K; j += kET) {
        const double u = a.zh[A0 + j] / dc::pole_minus_root(pole, j, o, tau);
        sum += u * u;
    }
    sum = block_sum256(sum, sh);
    const double inv = 1.0 / sqrt(sum);
    for (int j = threadIdx.x; j < K; j += kET)
        col[a.colsrc[A0 + a.src[A0 + j]]] = a.zh[A0 + j] / dc::pole_minus_root(pole, j, o, tau) * inv;
}

// Qb block = Qa block * U block for groups of at most 64 columns (one
// workgroup per group; the matrix cores take the larger ones).
__global__ __launch_bounds__(kET) void dc_small_product(DcArgs a, int ngroups) {
    const int g = blockIdx.x;
    if (g >= ngroups) return;
    const int A0 = 2 * a.s * g, k = min(2 * a.s, a.n - A0);
    for (int e = threadIdx.x; e < k * k; e += kET) {
        const int r = e % k, c = e / k;
        double acc = 0.0;
        for (int q = 0; q < k; ++q)
            acc += a.Qa[(A0 + r) + (long long)(A0 + q) * a.ld] * a.U[(A0 + q) + (long long)(A0 + c) * a.ld];
        a.Qb[(A0 + r) + (long long)(A0 + c) * a.ld] = acc;
    }
}

// Vs[:, k] = V[:, perm[k]] (n x n).
__global__ void gather_columns(int n, const double* V, long long ldv, const int* perm, double* Vs, long long lds) {
    const int k = blockIdx.y;
    const int src = perm[k];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        Vs[i + (long long)k * lds] = V[i + (long long)src * ldv];
}

template <class T>
T* carve(char*& p, size_t count) {
    T* r = reinterpret_cast<T*>(p);
    p += ((count * sizeof(T) + 255) / 256) * 256;
    return r;
}

}  // namespace

// Leading dimension of the T factors (and of S): one of at most kFT reflectors, or
// blocks of kBT.
static int factor_ld(int nref) { return nref <= kFT ? kFT : kBT; }
static size_t row_groups_max(int n) { return ((size_t)n + kTrdRows - 1) / kTrdRows; }

size_t syevd_work_bytes(int n) {
    const size_t nn = (size_t)n * n, N = (size_t)n + 64;
    const size_t nblk = ((size_t)n - 1 + kBT - 1) / kBT, ldf = factor_ld(n - 1);
    return 3 * (nn * 8 + 256) + (size_t)n * kTB * 8 + 256 + nblk * (2 * ldf * ldf + kFT * kFT) * 8 + 768 +
           2 * ((size_t)n * 2 * kTB * 8 + 256) + 22 * (N * 8 + 256) + 10 * (N * 4 + 256) +
           2 * (row_groups_max(n) * 8 + 256) + 2 * kMaxG * 8 + kMaxParts * 8 + 4096;
}

// Eigen-decomposition of the symmetric n x n matrix A (both triangles stored
// and used; A is overwritten).  w_host: eigenvalues, descending; Z (ldz): the matching
// orthonormal eigenvectors.  work: syevd_work_bytes(n) bytes of device memory.
// host: pinned buffer of at least n + 1 doubles.  Synchronises the stream.
// *finite: false when A holds a NaN or an infinity; w_host and Z are then not written.
hipError_t syevd(int n, double* A, long long lda, double* w_host, double* Z, long long ldz, char* work,
                 double* host, hipStream_t st, bool* finite) {
    if (n < 1) return hipErrorInvalidValue;
    char* p = work;
    const long long ld = n;
    double* Qa = carve<double>(p, (size_t)n * n);
    double* Qb = carve<double>(p, (size_t)n * n);
    double* U = carve<double>(p, (size_t)n * n);
    double* W = carve<double>(p, (size_t)n * kTB);
    const int nref = n - 1, nblk = (nref + kBT - 1) / kBT;
    const int ldf = factor_ld(nref);
    double* S = carve<double>(p, (size_t)nblk * ldf * ldf);
    double* Tf = carve<double>(p, (size_t)nblk * ldf * ldf);
    double* Y = carve<double>(p, (size_t)nblk * kFT * kFT);
    const size_t N = (size_t)n + 64;
    double *d = carve<double>(p, N), *e = carve<double>(p, N), *tau = carve<double>(p, N), *xa = carve<double>(p, N);
    double *yr = carve<double>(p, N), *a1 = carve<double>(p, N), *pq = carve<double>(p, N), *alpha = carve<double>(p, N);
    double *P = carve<double>(p, (size_t)n * 2 * kTB), *Q = carve<double>(p, (size_t)n * 2 * kTB);
    double *D = carve<double>(p, N), *ds = carve<double>(p, N), *zs = carve<double>(p, N);
    double *pole = carve<double>(p, N), *zp = carve<double>(p, N), *dval = carve<double>(p, N);
    double *rc = carve<double>(p, N), *rs = carve<double>(p, N), *dtau = carve<double>(p, N);
    double *zh = carve<double>(p, N), *vals = carve<double>(p, N), *rho = carve<double>(p, N);
    int *colsrc = carve<int>(p, N), *src = carve<int>(p, N), *ri = carve<int>(p, N), *rj = carve<int>(p, N);
    int *org = carve<int>(p, N), *inv = carve<int>(p, N), *Kc = carve<int>(p, N), *nrot = carve<int>(p, N);
    int* perm = carve<int>(p, N);
    double *sq = carve<double>(p, row_groups_max(n)), *sq_next = carve<double>(p, row_groups_max(n));
    double* partY = carve<double>(p, 2 * kMaxG);
    double* partM = carve<double>(p, kMaxParts);
    double* const scale = D + n;     // read back behind the eigenvalues
    hipError_t err;

    // --- Stage 1: tridiagonalisation ----------------------------------------
    const int gM = std::min(kMaxParts, n);
    trd_max<<<gM, kET, 0, st>>>(n, A, lda, partM);
    trd_scale<<<dim3(std::min(8, (n + kET - 1) / kET), std::min(n, 1024)), kET, 0, st>>>(n, A, lda, partM, gM, scale, Qa, ld);
    TrdArgs ta;
    ta.n = n; ta.A = A; ta.lda = lda; ta.W = W; ta.ldw = n; ta.alpha = alpha; ta.tau = tau;
    ta.d = d; ta.e = e; ta.xa = xa; ta.yr = yr; ta.a1 = a1; ta.pq = pq; ta.partY = partY;
    ta.P = P; ta.Q = Q;
    auto row_groups = [](int rows) { return (rows + kTrdRows - 1) / kTrdRows; };
    for (int j0 = 0; j0 < n - 1; j0 += kTB) {
        const int jb = std::min(kTB, n - 1 - j0);
        ta.j0 = j0;
        for (int c = 0; c < jb; ++c) {
            const int j = j0 + c;
            ta.j = j; ta.c = c;
            ta.sq = sq; ta.sq_next = sq_next;
            trd_column<<<row_groups(n - j), kET, 0, st>>>(ta, 0);
            std::swap(sq, sq_next);
            ta.gA = row_groups(n - j);
            // Columns per wave: enough waves to fill the chip first (256 CUs,
            // four waves a workgroup), then fewer reads of x.
            const int items = (n - j - 1) + 2 * c, C = items >= 4096 ? 4 : (items >= 2048 ? 2 : 1);
            ta.gY = std::min(kMaxG, ((items + C - 1) / C + 3) / 4);
            if (C == 4) trd_product<4><<<ta.gY, kET, 0, st>>>(ta);
            else if (C == 2) trd_product<2><<<ta.gY, kET, 0, st>>>(ta);
            else trd_product<1><<<ta.gY, kET, 0, st>>>(ta);
        }
        const int r0 = j0 + jb;
        const int nt = n - r0;
        ta.j = r0; ta.c = jb;
        ta.sq = sq;
        trd_column<<<row_groups(nt), kET, 0, st>>>(ta, 1);
        GemmDesc g;  // A22 -= [V W] [W V]^T
        g.m = nt; g.n = nt; g.k = 2 * jb; g.transb = 1;
        g.A = P + r0; g.lda = n;
        g.B = Q + r0; g.ldb = n;
        g.Cin = A + r0 + (long long)r0 * lda; g.ldcin = lda; g.beta = 1.0; g.alpha = -1.0;
        g.C = A + r0 + (long long)r0 * lda; g.ldc = lda;
        if ((err = gemm(g, st)) != hipSuccess) return err;
    }
    trd_cleanup<<<std::max(1, std::min(2048, (int)(((long long)n * n + kET - 1) / kET))), kET, 0, st>>>(n, A, lda, d);
    if ((err = hipGetLastError()) != hipSuccess) return err;

    // --- Stage 2: divide and conquer on T ------------------------------------
    dc_init<<<(n + kET - 1) / kET, kET, 0, st>>>(n, d, e, D);
    DcArgs da;
    da.n = n; da.e = e; da.D = D; da.ld = ld; da.ds = ds; da.zs = zs; da.pole = pole; da.zp = zp;
    da.dval = dval; da.rc = rc; da.rs = rs; da.tau = dtau; da.zh = zh; da.vals = vals; da.rho = rho;
    da.colsrc = colsrc; da.src = src; da.ri = ri; da.rj = rj; da.org = org; da.inv = inv; da.K = Kc;
    da.nrot = nrot;
    for (int s = 1; s < n; s *= 2) {
        const int ngroups = (n + 2 * s - 1) / (2 * s);
        da.s = s; da.Qa = Qa; da.Qb = Qb; da.U = U;
        dc_prepare<<<ngroups, kET, 0, st>>>(da);
        {
            const int k = std::min(2 * s, n);
            dc_rotate<<<dim3(std::max(1, std::min(64, (k + kET - 1) / kET)), ngroups), kET, 0, st>>>(da);
        }
        const int gwave = (n + kET / 64 - 1) / (kET / 64);   // one wave per root
        dc_secular<<<gwave, kET, 0, st>>>(da);
        dc_lowner<<<gwave, kET, 0, st>>>(da);
        dc_rank<<<gwave, kET, 0, st>>>(da);
        dc_vectors<<<n, kET, 0, st>>>(da);
        if ((err = fill_matrix<double>(n, n, Qb, ld, 0, 1, 0.0, 0.0, st)) != hipSuccess) return err;
        if (2 * s <= 64) {
            dc_small_product<<<ngroups, kET, 0, st>>>(da, ngroups);
        } else {
            const int full = n / (2 * s), k2 = 2 * s;
            const long long stride = (long long)k2 * (ld + 1);
            if (full > 0) {
                GemmDesc g;
                g.m = k2; g.n = k2; g.k = k2;
                g.A = Qa; g.lda = ld; g.strideA = stride;
                g.B = U; g.ldb = ld; g.strideB = stride;
                g.C = Qb; g.ldc = ld; g.strideC = stride;
                g.batch = full;
                if ((err = gemm(g, st)) != hipSuccess) return err;
            }
            const int tail = n - full * k2;
            if (tail > 0) {
                const long long off = (long long)full * stride;
                GemmDesc g;
                g.m = tail; g.n = tail; g.k = tail;
                g.A = Qa + off; g.lda = ld; g.B = U + off; g.ldb = ld; g.C = Qb + off; g.ldc = ld;
                if ((err = gemm(g, st)) != hipSuccess) return err;
            }
        }
        if ((err = hipGetLastError()) != hipSuccess) return err;
        std::swap(Qa, Qb);
    }

    // Eigenvalues to the host, descending order; matching columns.
    if ((err = hipMemcpyAsync(host, D, sizeof(double) * (n + 1), hipMemcpyDeviceToHost, st)) != hipSuccess) return err;
    if ((err = hipStreamSynchronize(st)) != hipSuccess) return err;
    const double unscale = host[n];
    *finite = unscale > 0.0;
    if (!*finite) return hipSuccess;
    std::vector<int> order(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y2) { return host[x] > host[y2]; });
    for (int i = 0; i < n; ++i) w_host[i] = host[order[i]] / unscale;
    int* hperm = reinterpret_cast<int*>(host);
    for (int i = 0; i < n; ++i) hperm[i] = order[i];
    if ((err = hipMemcpyAsync(perm, hperm, sizeof(int) * n, hipMemcpyHostToDevice, st)) != hipSuccess) return err;
    gather_columns<<<dim3(std::max(1, std::min(64, (n + kET - 1) / kET)), n), kET, 0, st>>>(n, Qa, ld, perm, Z, ldz);

    // --- Stage 3: Z <- Q Z with the reflectors of stage 1 --------------------
    // Blocks of kBT reflectors.  A block's V is taken from row b0 on, one row
    // above its first unit entry: that row is zero in V, and the operands keep
    // the alignment of A's columns.
    if (nref > 0) {
        // S = V^T V of every block at once (upper tiles; the rows above a
        // block are zero), then the T factors.
        const bool one = ldf == kFT;
        if (!one && (err = fill_matrix<double>(kBT, kBT * nblk, S, kBT, 0, 1, 0.0, 0.0, st)) != hipSuccess) return err;
        const int fullb = nref / kBT;
        for (int part = 0; part < 2; ++part) {
            const long long b0 = part == 0 ? 0 : (long long)fullb * kBT;
            GemmDesc g;
            g.m = g.n = part == 0 ? kBT : nref - (int)b0;
            g.k = n - (int)b0; g.transa = 1;
            g.batch = part == 0 ? fullb : 1;
            if (g.m <= 0 || g.batch <= 0) continue;
            g.A = g.B = A + b0 + b0 * lda; g.lda = g.ldb = lda;
            g.strideA = g.strideB = (long long)kBT * lda;
            g.C = S + (b0 / kBT) * kBT * kBT; g.ldc = ldf; g.strideC = (long long)kBT * kBT;
            g.flags = kCUpperTiles | kCStoreUpper;
            if ((err = gemm(g, st)) != hipSuccess) return err;
        }
        if ((err = hipFuncSetAttribute((const void*)form_t, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kFormTLds)) != hipSuccess)
            return err;
        form_t<<<one ? 1 : 2 * nblk, 512, kFormTLds, st>>>(nref, S, tau, Tf, ldf);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        GemmDesc y;  // Y = S12 T2
        y.m = y.n = y.k = kFT; y.batch = nblk;
        y.A = S + (long long)kFT * kBT; y.lda = kBT; y.strideA = (long long)kBT * kBT;
        y.B = Tf + kFT + (long long)kFT * kBT; y.ldb = kBT; y.strideB = (long long)kBT * kBT;
        y.C = Y; y.ldc = kFT; y.strideC = (long long)kFT * kFT;
        y.flags = kBUpper;
        if (!one && (err = gemm(y, st)) != hipSuccess) return err;
        GemmDesc t;  // T12 = -T1 Y
        t.m = t.n = t.k = kFT; t.batch = nblk;
        t.A = Tf; t.lda = kBT; t.strideA = (long long)kBT * kBT;
        t.B = Y; t.ldb = kFT; t.strideB = (long long)kFT * kFT;
        t.C = Tf + (long long)kFT * kBT; t.ldc = kBT; t.strideC = (long long)kBT * kBT;
        t.alpha = -1.0; t.flags = kAUpper;
        if (!one && (err = gemm(t, st)) != hipSuccess) return err;
    }
    const long long ldt = std::min(kBT, n);   // scratch U, Qb hold nb x n with nb <= ldt
    for (int q = nblk - 1; q >= 0; --q) {
        const int b0 = q * kBT, nb = std::min(kBT, nref - b0);
        const int rows = n - b0;
        const double* V = A + b0 + (long long)b0 * lda;
        GemmDesc w1;  // U = V^T Z[b0:, :]   (nb x n, in U)
        w1.m = nb; w1.n = n; w1.k = rows; w1.transa = 1;
        w1.A = V; w1.lda = lda; w1.B = Z + b0; w1.ldb = ldz; w1.C = U; w1.ldc = ldt;
        w1.flags = kAUpper;
        if ((err = gemm(w1, st)) != hipSuccess) return err;
        GemmDesc w2;  // Qb = T U
        w2.m = nb; w2.n = n; w2.k = nb;
        w2.A = Tf + (long long)q * kBT * kBT; w2.lda = ldf; w2.B = U; w2.ldb = ldt; w2.C = Qb; w2.ldc = ldt;
        w2.flags = kAUpper;
        if ((err = gemm(w2, st)) != hipSuccess) return err;
        GemmDesc w3;  // Z[b0:, :] -= V Qb
        w3.m = rows; w3.n = n; w3.k = nb;
        w3.A = V; w3.lda = lda; w3.B = Qb; w3.ldb = ldt;
        w3.Cin = Z + b0; w3.ldcin = ldz; w3.beta = 1.0; w3.alpha = -1.0;
        w3.C = Z + b0; w3.ldc = ldz;
        w3.flags = kALower;
        if ((err = gemm(w3, st)) != hipSuccess) return err;
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    return hipStreamSynchronize(st);
}

}  // namespace zolo
