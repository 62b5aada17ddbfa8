// Batched upper Cholesky and triangular inverse (FP64, and FP32 for the mixed
// precision schedule) for the Cholesky-type step of Zolo-PD (Algorithm 1
// step 4(d)): Z_j = X^T X + c_{2j-1} I = R_j^T R_j for all j at once, then
// R_j^{-1}.
//
// POTRF is right-looking with 64-column blocks grouped in bands of 256: a
// 64 x 64 diagonal block is factored in LDS by one workgroup per matrix
// (which also inverts it), the row panel to its right becomes R_kk^{-T} Z_12
// (one GEMM), the rows of the band below the block take its rank-64 update,
// and once the band is done the matrix below it takes one rank-256 update on
// its upper tiles.  The trailing matrix is thus read and written once per
// 256 columns rather than once per 64.
//
// TRTRI is recursive and level-batched: all 64 x 64 diagonal blocks are
// inverted at once, then for block sizes s = 64, 128, 256, ... every pair of
// neighbouring s-blocks is merged with two GEMMs,
//     inv([R11 R12; 0 R22]) = [R11^{-1}, -R11^{-1} R12 R22^{-1}; 0, R22^{-1}],
// batched over all pairs of a level and all matrices.
#include "misc.hpp"
#include "stats.hpp"

#include <limits>

namespace zolo {
namespace {

constexpr int kB = 64;
constexpr int kBand = 256;   // columns whose trailing update is applied at once

constexpr int kDB = 16;  // column block of the in-LDS factorisation

// Wave-uniform broadcast of lane l's value (readlane, no LDS round trip).
template <class T>
__device__ inline T lane_bcast(T x, int l) {
    if constexpr (sizeof(T) == 8) {
        const long long v = __double_as_longlong(x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, l);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), l);
        return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    } else {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
    }
}

// The upper triangle of the kb x kb block at Z into S (LDS), the identity
// beyond it, by 256 threads with all loads in flight together.
template <class T>
__device__ void load_upper(const T* Z, long long ld, int kb, T (*S)[kB + 1]) {
    const int i = threadIdx.x % kB, j0 = threadIdx.x / kB;
    T v[kB / 4];
#pragma unroll
    for (int u = 0; u < kB / 4; ++u) v[u] = Z[min(i, kb - 1) + (long long)min(j0 + 4 * u, kb - 1) * ld];
#pragma unroll
    for (int u = 0; u < kB / 4; ++u) {
        const int j = j0 + 4 * u;
        const int in = opaque(((i < kb) & (j < kb) & (i <= j)) ? -1 : 0);
        S[i][j] = keep_if(v[u], in) + (T)(((i == j) & (i >= kb)) ? 1 : 0);
    }
}

// Inverse of the 16 x 16 diagonal block at o of the upper triangular S into Si (LDS),
// by one wave: lane j of each row of 16 lanes back-substitutes column j.  rcp
// holds 1 / S[i][i], with DIV S[i][i] itself.  Each entry found goes to all the sums above it, which are
// independent of each other (a sum per entry at a time is one chain of 120
// operations: 11.4k cycles for the four blocks at once, now 2.5k).
template <class T, int K, bool DIV>
__device__ __forceinline__ void inverse16_steps(const T (*S)[kB + 1], const T* rcp, T (*Si)[kB + 1], T (&x)[kDB],
                                                const T (&z)[kDB], T r, int o, int l16) {
    if constexpr (K >= 0) {
        T zn[kDB], rn = 0;
        if constexpr (K > 0) {
            rn = rcp[o + K - 1];
#pragma unroll
            for (int i = 0; i < K - 1; ++i) zn[i] = S[o + i][o + K - 1];
        }
        const T xk = K <= l16 ? (DIV ? x[K] / r : x[K] * r) : (T)0;
        Si[o + K][o + l16] = xk;                  // the four rows of lanes alike
#pragma unroll
        for (int i = 0; i < K; ++i) x[i] -= z[i] * xk;
        __builtin_amdgcn_sched_barrier(0);        // one column's loads ahead (registers)
        inverse16_steps<T, K - 1, DIV>(S, rcp, Si, x, zn, rn, o, l16);
    }
}
template <class T, bool DIV = false>
__device__ __forceinline__ void inverse16(const T (*S)[kB + 1], const T* rcp, T (*Si)[kB + 1], int o, int l16) {
    T x[kDB], z[kDB];
#pragma unroll
    for (int i = 0; i < kDB; ++i) x[i] = i == l16 ? (T)1 : (T)0;
#pragma unroll
    for (int i = 0; i < kDB - 1; ++i) z[i] = S[o + i][o + kDB - 1];
    inverse16_steps<T, kDB - 1, DIV>(S, rcp, Si, x, z, rcp[o + kDB - 1], o, l16);
}
// A 16 x 16 tile of S12 Si22 (phase 0) or -Si11 times it (phase 1) for blocks of
// W at o and o + W, the tile's rows and columns at ti and tj, on the matrix cores.
template <class T, int W>
__device__ __forceinline__ typename Mfma<T>::acc merge_tile(const T (*S)[kB + 1], const T (*Si)[kB + 1], int phase, int o,
                                                            int ti, int tj, int l16, int lg) {
    T x[W / 4], y[W / 4];                         // all operands in flight
#pragma unroll
    for (int k = 0; k < W; k += 4) {
        x[k / 4] = phase == 0 ? S[o + ti + l16][o + W + k + lg] : -Si[o + ti + l16][o + k + lg];
        y[k / 4] = phase == 0 ? Si[o + W + k + lg][o + W + tj + l16] : Si[o + k + lg][o + W + tj + l16];
    }
    typename Mfma<T>::acc acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < W; k += 4) acc = Mfma<T>::run(x[k / 4], y[k / 4], acc);
    return acc;
}
template <class T, int W>
__device__ __forceinline__ void merge_store(T (*Si)[kB + 1], const typename Mfma<T>::acc& acc, int o, int ti, int tj,
                                            int lane) {
#pragma unroll
    for (int e = 0; e < 4; ++e) Si[o + ti + Mfma<T>::row(lane, e)][o + W + tj + (lane & 15)] = acc[e];
}
// Si12 = -Si11 (S12 Si22): blocks of 16 by one wave, of 32 by the workgroup.
template <class T>
__device__ __forceinline__ void merge16(const T (*S)[kB + 1], T (*Si)[kB + 1], int o, int lane) {
    for (int phase = 0; phase < 2; ++phase) {
        const typename Mfma<T>::acc acc = merge_tile<T, kDB>(S, Si, phase, o, 0, 0, lane & 15, lane >> 4);
        __builtin_amdgcn_wave_barrier();
        merge_store<T, kDB>(Si, acc, o, 0, 0, lane);
        __builtin_amdgcn_wave_barrier();
    }
}
template <class T>
__device__ __forceinline__ void merge32(const T (*S)[kB + 1], T (*Si)[kB + 1], int wave, int lane) {
    const int ti = wave % 2 * kDB, tj = wave / 2 * kDB;
    for (int phase = 0; phase < 2; ++phase) {
        const typename Mfma<T>::acc acc = merge_tile<T, 2 * kDB>(S, Si, phase, 0, ti, tj, lane & 15, lane >> 4);
        __syncthreads();
        merge_store<T, 2 * kDB>(Si, acc, 0, ti, tj, lane);
        __syncthreads();
    }
}

// Inverse of the upper-triangular 64 x 64 matrix S (LDS; identity beyond the
// matrix) into Si (LDS), by the workgroup's 256 threads: the four 16 x 16
// diagonal blocks at once (rcp and DIV as above), then neighbouring blocks of 16
// and of 32 merged.
template <class T, bool DIV>
__device__ void lds_upper_inverse(const T (*S)[kB + 1], const T* rcp, T (*Si)[kB + 1]) {
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < kB * kB; e += 256) {
        const int i = e / kB, j = e % kB;
        if (i / kDB != j / kDB) Si[i][j] = 0;
    }
    inverse16<T, DIV>(S, rcp, Si, w * kDB, lane & 15);
    __syncthreads();
    if (w < 2) merge16<T>(S, Si, 2 * w * kDB, lane);
    __syncthreads();
    merge32<T>(S, Si, w, lane);
}

// sqrt(d) and 1 / sqrt(d) of a positive, finite d: the hardware's estimate of the
// reciprocal root refined by Goldschmidt's and Newton's iterations without a branch,
// 1 / sqrt(d) first, which the next pivot waits for, then the root from it and
// its residual.  Small d is scaled by an even power of two, so that no residual
// underflows.  Largest errors over all exponents: root 1.11e-16, as correctly
// rounded, and reciprocal 1.38e-16, where a division by it leaves 1.65e-16 (FP32:
// 5.96e-8, and 7.4e-8 against 8.9e-8).
__device__ __forceinline__ void sqrt_rcp(double d, double& r, double& ri) {
    const bool small = d < 0x1p-900;
    d *= small ? 0x1p512 : 1.0;
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
    const double t = fma(-h, g, 0.5);
    h = fma(h, t, h);
    const double z = h + h;
    const double x = fma(fma(-(d * z), z, 1.0), h, z);
    g = d * x;
    r = fma(fma(-g, g, d), h, g) * (small ? 0x1p-256 : 1.0);
    ri = x * (small ? 0x1p256 : 1.0);
}
__device__ __forceinline__ void sqrt_rcp(float d, float& r, float& ri) {
    const bool small = d < 0x1p-96f;
    d *= small ? 0x1p64f : 1.0f;
    const float y = __builtin_amdgcn_rsqf(d), h = 0.5f * y;
    const float x = fmaf(fmaf(-(d * y), y, 1.0f), h, y);
    const float g = d * x;
    r = fmaf(fmaf(-g, g, d), h, g) * (small ? 0x1p-32f : 1.0f);
    ri = x * (small ? 0x1p32f : 1.0f);
}

// Upper Cholesky of the kb x kb diagonal block at (k0, k0) of each matrix
// (one workgroup per matrix), its inverse into inv.  Four steps of 16 rows:
// wave 0 holds the 16 rows of all 64 columns (lane = column) and factors them
// in registers, the diagonal block and the row panel to its right in the same
// instructions (the multipliers of a row reach all lanes by readlane); then the
// rows below take their rank-16 update on the matrix cores, a 16 x 16 tile per
// wave.  While wave 0 factors, the others invert and store the blocks before and
// merge the first two inverses.  Rows and columns past kb are those of the
// identity.  A non-positive pivot is reported (1-based global column) and
// replaced by 1 so that every wave finishes; the caller discards the result.
// The pivots run without a branch, so that one's reciprocal square root overlaps
// the updates of the one before.  Bound: latency of the 64 dependent pivots.  One
// launch in a solve takes 19 us (FP32: 15); with inverse, merges and stores after the
// factor and two branches per pivot it took 28 (23), with the panel of a block
// solved one thread per column and sums element by element 58 (51): 3001 x 1501 by
// Cholesky-type steps 10.9, 6.8 and 6.3 ms, four FP32 factors at n = 2000 4.1, 3.2
// and 2.9 ms.
template <class T>
__global__ __launch_bounds__(256) void potrf_diag_kernel(int k0, int kb, T* Z, long long ldz, long long sz,
                                                         int* info, T* inv, long long ldi, long long si) {
    __shared__ T S[kB][kB + 1];
    __shared__ T Si[kB][kB + 1];
    __shared__ T s_rcp[kB];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    T* Zb = Z + b * sz + k0 + (long long)k0 * ldz;
    load_upper<T>(Zb, ldz, kb, S);
    __syncthreads();
    // Rows [o, o + 16) of R to memory by `nw` waves, this one the w-th: 16 rows of 4
    // columns at a time.
    auto store_rows = [&](int o, int w, int nw) __attribute__((always_inline)) {
        const int i = o + l16;
        for (int j = 4 * w + lg; j < kb; j += 4 * nw)
            if (i < kb) Zb[i + (long long)j * ldz] = i <= j ? S[i][j] : (T)0;
    };
    int bad = 0;
#pragma unroll 1
    for (int jb = 0; jb < kB; jb += kDB) {
        if (wave == 0) {
            T c[kDB];
#pragma unroll
            for (int i = 0; i < kDB; ++i) c[i] = S[jb + i][lane];
#pragma unroll
            for (int i = 0; i < kDB; ++i) {
                T d = lane_bcast(c[i], jb + i);
                asm("" : "+v"(d));                // tested in vector registers: no turns to the scalar unit
                const bool ok = d > (T)0 && d <= std::numeric_limits<T>::max();
                bad = ok || bad != 0 ? bad : k0 + jb + i + 1;
                d = ok ? d : (T)1;
                T r, ri;
                sqrt_rcp(d, r, ri);
                c[i] = lane == jb + i ? r : c[i] * ri;
                s_rcp[jb + i] = ri;               // all lanes alike
#pragma unroll
                for (int l = i + 1; l < kDB; ++l) c[l] -= lane_bcast(c[i], jb + l) * c[i];   // R[i][jb + l]
            }
#pragma unroll
            for (int i = 0; i < kDB; ++i) S[jb + i][lane] = lane >= jb + i ? c[i] : (T)0;
        } else if (jb == 0) {
            for (int e = tid - 64; e < kB * kB; e += 192) {
                const int i = e / kB, j = e % kB;
                if (i / kDB != j / kDB) Si[i][j] = 0;
            }
        } else if (wave == 1) {
            inverse16<T>(S, s_rcp, Si, jb - kDB, l16);
        } else {
            store_rows(jb - kDB, wave - 2, 2);
            if (jb == kB - kDB && wave == 2) merge16<T>(S, Si, 0, lane);
        }
        __syncthreads();
        // Rows below (upper tiles): S[i][j] -= sum_k R[jb+k][i] R[jb+k][j].
        const int c0 = jb + kDB, nt = (kB - c0) / kDB;
        for (int t = wave; t < nt * (nt + 1) / 2; t += 4) {
            int ti = 0, tj = t;
            while (tj >= nt - ti) tj -= nt - ti++;
            tj += ti;
            T* const row = &S[c0 + kDB * ti][c0 + kDB * tj + l16];
            typename Mfma<T>::acc acc;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = row[Mfma<T>::row(lane, e) * (kB + 1)];
#pragma unroll
            for (int k = 0; k < kDB; k += 4)
                acc = Mfma<T>::run(-S[jb + k + lg][c0 + kDB * ti + l16], S[jb + k + lg][c0 + kDB * tj + l16], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) row[Mfma<T>::row(lane, e) * (kB + 1)] = acc[e];
        }
        __syncthreads();
    }
    if (wave == 0) {
        inverse16<T>(S, s_rcp, Si, kB - kDB, l16);
        __builtin_amdgcn_wave_barrier();
        merge16<T>(S, Si, 2 * kDB, lane);
    } else {
        store_rows(kB - kDB, wave - 1, 3);
    }
    __syncthreads();
    merge32<T>(S, Si, wave, lane);
    T* wb = inv + b * si + lane;
    if (lane < kb)
        for (int j = wave; j < kb; j += 4) wb[(long long)j * ldi] = Si[lane][j];
    if (tid == 0 && bad != 0 && info[b] == 0) info[b] = bad;
}

// Invert every 64 x 64 diagonal block of R_b into Rinv_b.
template <class T>
__global__ __launch_bounds__(256) void trtri_diag_kernel(int n, const T* R, long long ldr, long long sr, T* Rinv,
                                                         long long ldi, long long si) {
    __shared__ T S[kB][kB + 1];
    __shared__ T Si[kB][kB + 1];
    const int blk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int o = blk * kB, kb = min(kB, n - o);
    const T* Rb = R + b * sr + o + (long long)o * ldr;
    T* Ib = Rinv + b * si + o + (long long)o * ldi;
    load_upper<T>(Rb, ldr, kb, S);
    __syncthreads();
    __shared__ T s_rcp[kB];
    // A diagonal entry so small or so large that its reciprocal is no normal number
    // (zero and infinity among them) is divided by: 0 times a reciprocal that
    // overflows would be NaN.
    bool plain = true;
    if (tid < kB) {
        const T r = (T)1 / S[tid][tid];
        plain = fabs(r) >= std::numeric_limits<T>::min() && fabs(r) <= std::numeric_limits<T>::max();
        s_rcp[tid] = r;
    }
    if (__syncthreads_and(plain)) {
        lds_upper_inverse<T, false>(S, s_rcp, Si);
    } else {
        if (tid < kB) s_rcp[tid] = S[tid][tid];
        __syncthreads();
        lds_upper_inverse<T, true>(S, s_rcp, Si);
    }
    for (int e = tid; e < kb * kb; e += 256) {
        const int i = e % kb, j = e / kb;
        Ib[i + (long long)j * ldi] = Si[i][j];
    }
}

}  // namespace

// The factorisation.  The inverse of the diagonal block at (j0, j0) goes to
// inv + j0 * step (leading dimension ldi, batch stride si).
template <class T>
static hipError_t potrf_blocks(int n, T* Z, long long ldz, long long sz, int batch, int* info_dev, T* inv,
                               long long step, long long ldi, long long si, hipStream_t st) {
    hipError_t e;
    for (int k0 = 0; k0 < n; k0 += kBand) {
        const int band = n - k0 < kBand ? n - k0 : kBand;
        for (int j0 = k0; j0 < k0 + band; j0 += kB) {
            const int kb = k0 + band - j0 < kB ? k0 + band - j0 : kB;
            StatScope sc(sizeof(T) == 8 ? "potrf_diag_kernel<double>" : "potrf_diag_kernel<float>", st,
                         batch * (double)kb * kb * kb / 3.0);
            T* Ik = inv + j0 * step;
            potrf_diag_kernel<T><<<batch, 256, 0, st>>>(j0, kb, Z, ldz, sz, info_dev, Ik, ldi, si);
            sc.end();
            if ((e = hipGetLastError()) != hipSuccess) return e;
            const int rest = n - j0 - kb;
            if (rest <= 0) break;
            T* Z12 = Z + j0 + (long long)(j0 + kb) * ldz;
            // R12 = R_kk^{-T} Z12 over the whole width, in place (one tile
            // row covers all kb rows).
            GemmDescT<T> g;
            g.m = kb; g.n = rest; g.k = kb; g.transa = 1; g.transb = 0;
            g.A = Ik; g.lda = ldi; g.strideA = si;
            g.B = Z12; g.ldb = ldz; g.strideB = sz;
            g.C = Z12; g.ldc = ldz; g.strideC = sz;
            g.beta = 0.0; g.batch = batch; g.flags = kALower;
            if ((e = gemm(g, st)) != hipSuccess) return e;
            // Rows of the band below this block take its rank-kb update now
            // (the next blocks of the band need them); the matrix below the
            // band waits for the band's combined update.
            const int rows = k0 + band - j0 - kb;
            if (rows > 0) {
                T* Z22 = Z + (j0 + kb) + (long long)(j0 + kb) * ldz;
                GemmDescT<T> u;
                u.m = rows; u.n = rest; u.k = kb; u.transa = 1; u.transb = 0;
                u.A = Z12; u.lda = ldz; u.strideA = sz;
                u.B = Z12; u.ldb = ldz; u.strideB = sz;
                u.Cin = Z22; u.ldcin = ldz; u.strideCin = sz;
                u.C = Z22; u.ldc = ldz; u.strideC = sz;
                u.alpha = -1.0; u.beta = 1.0; u.batch = batch;
                u.flags = kCUpperTiles | kCStoreUpper;
                if ((e = gemm(u, st)) != hipSuccess) return e;
            }
        }
        // Below the band: Z22 -= P^T P with P = the band's rows of R to the
        // right of the band (one rank-`band` update instead of band/64).
        const int rest = n - k0 - band;
        if (rest <= 0) break;
        T* P = Z + k0 + (long long)(k0 + band) * ldz;
        T* Z22 = Z + (k0 + band) + (long long)(k0 + band) * ldz;
        GemmDescT<T> s;
        s.m = rest; s.n = rest; s.k = band; s.transa = 1; s.transb = 0;
        s.A = P; s.lda = ldz; s.strideA = sz;
        s.B = P; s.ldb = ldz; s.strideB = sz;
        s.Cin = Z22; s.ldcin = ldz; s.strideCin = sz;
        s.C = Z22; s.ldc = ldz; s.strideC = sz;
        s.alpha = -1.0; s.beta = 1.0; s.batch = batch;
        s.flags = kCUpperTiles | kCStoreUpper;
        if ((e = gemm(s, st)) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <class T>
hipError_t potrf_batched(int n, T* Z, long long ldz, long long sz, int batch, int* info_dev, T* work,
                         hipStream_t st) {
    hipError_t e = zero_ints(info_dev, batch, st);
    if (e != hipSuccess) return e;
    e = potrf_blocks<T>(n, Z, ldz, sz, batch, info_dev, work, 0, kB, (long long)kB * kB, st);
    return e != hipSuccess ? e : zero_strict_lower<T>(n, Z, ldz, sz, batch, st);
}
template hipError_t potrf_batched<double>(int, double*, long long, long long, int, int*, double*, hipStream_t);
template hipError_t potrf_batched<float>(int, float*, long long, long long, int, int*, float*, hipStream_t);

// The merges of the triangular inverse, its 64 x 64 diagonal blocks in place.
template <class T>
static hipError_t trtri_merges(int n, const T* R, long long ldr, long long sr, T* Rinv, long long ldi, long long si,
                               int batch, T* work, long long work_elems, hipStream_t st) {
    hipError_t e;
    for (long long s = kB; s < n; s *= 2) {
        const long long full = n / (2 * s);           // pairs with both blocks of size s
        const long long o_rag = full * 2 * s;          // a ragged pair starts here if o_rag + s < n
        const long long s2_rag = n - o_rag - s;
        const long long per_b = full * s * s + (s2_rag > 0 ? s * s2_rag : 0);
        if (per_b * batch > work_elems) return hipErrorInvalidValue;
        for (int part = 0; part < 2; ++part) {
            const long long npairs = part == 0 ? full : (s2_rag > 0 ? 1 : 0);
            if (npairs == 0) continue;
            const long long o = part == 0 ? 0 : o_rag;
            const long long s2 = part == 0 ? s : s2_rag;
            T* Wp = work + (part == 0 ? 0 : full * s * s);
            // W = R12 * R22^{-1}
            GemmDescT<T> g;
            g.m = (int)s; g.n = (int)s2; g.k = (int)s2;
            g.A = R + o + (o + s) * ldr; g.lda = ldr; g.strideA = 2 * s * (ldr + 1);
            g.B = Rinv + (o + s) + (o + s) * ldi; g.ldb = ldi; g.strideB = 2 * s * (ldi + 1);
            g.C = Wp; g.ldc = s; g.strideC = s * s2;
            g.batch = (int)npairs; g.flags = kBUpper;
            g.batch2 = batch; g.strideA2 = sr; g.strideB2 = si; g.strideC2 = per_b;
            if ((e = gemm(g, st)) != hipSuccess) return e;
            // Rinv12 = -R11^{-1} W
            GemmDescT<T> h;
            h.m = (int)s; h.n = (int)s2; h.k = (int)s;
            h.A = Rinv + o + o * ldi; h.lda = ldi; h.strideA = 2 * s * (ldi + 1);
            h.B = Wp; h.ldb = s; h.strideB = s * s2;
            h.C = Rinv + o + (o + s) * ldi; h.ldc = ldi; h.strideC = 2 * s * (ldi + 1);
            h.alpha = -1.0; h.batch = (int)npairs; h.flags = kAUpper;
            h.batch2 = batch; h.strideA2 = si; h.strideB2 = per_b; h.strideC2 = si;
            if ((e = gemm(h, st)) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

template <class T>
hipError_t trtri_batched(int n, const T* R, long long ldr, long long sr, T* Rinv, long long ldi, long long si,
                         int batch, T* work, long long work_elems, hipStream_t st) {
    hipError_t e = fill_matrix<T>(n, n, Rinv, ldi, si, batch, 0.0, 0.0, st);
    if (e != hipSuccess) return e;
    const int nblk = (n + kB - 1) / kB;
    trtri_diag_kernel<T><<<dim3(nblk, batch), 256, 0, st>>>(n, R, ldr, sr, Rinv, ldi, si);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return trtri_merges<T>(n, R, ldr, sr, Rinv, ldi, si, batch, work, work_elems, st);
}

template <class T>
hipError_t potrf_inverse_batched(int n, T* Z, long long ldz, long long sz, T* Rinv, long long ldi, long long si,
                                 int batch, int* info_dev, T* work, long long work_elems, hipStream_t st) {
    const hipError_t e = potrf_blocks<T>(n, Z, ldz, sz, batch, info_dev, Rinv, ldi + 1, ldi, si, st);
    return e != hipSuccess ? e : trtri_merges<T>(n, Z, ldz, sz, Rinv, ldi, si, batch, work, work_elems, st);
}
template hipError_t potrf_inverse_batched<double>(int, double*, long long, long long, double*, long long, long long,
                                                  int, int*, double*, long long, hipStream_t);
template hipError_t potrf_inverse_batched<float>(int, float*, long long, long long, float*, long long, long long, int,
                                                 int*, float*, long long, hipStream_t);

template hipError_t trtri_batched<double>(int, const double*, long long, long long, double*, long long, long long,
                                          int, double*, long long, hipStream_t);
template hipError_t trtri_batched<float>(int, const float*, long long, long long, float*, long long, long long, int,
                                         float*, long long, hipStream_t);

}  // namespace zolo
