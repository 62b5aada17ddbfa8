// Shared definitions for the gfx950 Zolo-PD library (device helpers, launch
// descriptors).  Every kernel of the library is written for CDNA4: 64-lane
// wavefronts, FP64 MFMA 16x16x4 tiles, LDS staging.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace zolo {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// GEMM descriptor:  D_b = alpha * alpha_b * op(A_b) op(B_b) + beta * Cin_b
// (or, with `reduce`, one D = beta * Cin + sum_b alpha*alpha_b op(A_b) op(B_b)).
// Column-major, op(X) = X or X^T.  Structural flags let a tile skip k-blocks
// that are known to be zero (triangular operands) and skip whole tiles of a
// symmetric result.  The zero region of a triangular operand may hold anything,
// NaN included: whole blocks of it are skipped, and its elements in the blocks
// on the diagonal are replaced by zeros element by element.  The Cholesky-type
// step, whose factors are undefined there, relies on it.
// ---------------------------------------------------------------------------
enum GemmFlags : unsigned {
    kAUpper = 1u,        // op(A)[i][k] == 0 for k < i   (k-range starts at tile row 0)
    kALower = 2u,        // op(A)[i][k] == 0 for k > i   (k-range ends at last tile row)
    kBUpper = 4u,        // op(B)[k][j] == 0 for k > j   (k-range ends at last tile column)
    kBLower = 8u,        // op(B)[k][j] == 0 for k < j   (k-range starts at tile column 0)
    kCUpperTiles = 16u,  // compute only tiles that meet the upper triangle (i <= j)
    kCStoreUpper = 32u,  // store only elements with i <= j
    kCStoreLower = 64u,  // store only elements with i >= j
};

constexpr int kMaxInlineAlpha = 16;

// T = double (FP64 path) or float (the FP32 steps of the mixed schedule).
template <class T>
struct GemmDescT {
    int m = 0, n = 0, k = 0;
    int transa = 0, transb = 0;
    const T* A = nullptr; long long lda = 0, strideA = 0;
    const T* B = nullptr; long long ldb = 0, strideB = 0;
    const T* Cin = nullptr; long long ldcin = 0, strideCin = 0;
    T* C = nullptr; long long ldc = 0, strideC = 0;
    double alpha = 1.0;
    double beta = 0.0;
    int batch = 1;
    int reduce = 0;          // sum the batch into one output
    // Optional second (outer) batch dimension, never reduced.
    int batch2 = 1;
    long long strideA2 = 0, strideB2 = 0, strideCin2 = 0, strideC2 = 0;
    unsigned flags = 0;
    int nalpha = 0;          // if > 0, alpha_b = alphas[b] (b < nalpha <= 16)
    double alphas[kMaxInlineAlpha] = {};
    // Split-K (batch2 must be 1): the k-range is cut into `splitk` pieces whose
    // partial products go to `work` (splitk x outputs x m x n, ld m) and a
    // second kernel sums them in order into C.
    int splitk = 1;
    T* work = nullptr;
    int keep_pieces = 0;     // leave the pieces in `work` (the caller sums them)
    // Set by the launcher when the work per tile is uneven (triangular
    // operands, upper-tile outputs): XCD x takes the tiles [xsplit[x],
    // xsplit[x+1]) of the launch order, ranges cut to equal estimated work.
    int xbal = 0;
    int xsplit[9] = {};
};
using GemmDesc = GemmDescT<double>;
using SGemmDesc = GemmDescT<float>;

// Launches D = ... on `stream`.  Returns hipSuccess or the launch error.
hipError_t gemm(const GemmDesc& d, hipStream_t stream);
hipError_t gemm(const SGemmDesc& d, hipStream_t stream);
// As gemm(), but a product whose output has too few tiles to fill the chip
// and a long k-range is split along k into `work` (up to work_elems doubles).
// With `pieces`, the pieces are left unsummed in `work` and *pieces says how
// many there are (1: the product is in C as usual).
hipError_t gemm_split(GemmDesc d, double* work, size_t work_elems, hipStream_t stream, int* pieces = nullptr);
hipError_t gemm_few(const GemmDesc& d, double* work, size_t work_elems, hipStream_t stream);
inline hipError_t gemm_few(const SGemmDesc& d, float*, size_t, hipStream_t stream) { return gemm(d, stream); }

// Nonzeros of a trapezoidal operand with `r` rows (the side that is not k)
// and depth k: "from diagonal" = zero where k < r-index (upper op(A), lower
// op(B)), otherwise zero where k > r-index.
inline double trapezoid_nnz(double r, double k, bool from_diagonal) {
    if (from_diagonal) {
        const double s = r < k ? r : k;
        return s * k - s * (s - 1) / 2;
    }
    return r <= k ? r * (r + 1) / 2 : k * (k + 1) / 2 + (r - k) * k;
}

// Floating-point operations a descriptor executes: 2 m n k per product, a
// triangular or trapezoidal operand counted by its nonzeros (both
// triangular: one third of the full product, as for square triangles), and
// half for upper-tile outputs.
template <class T>
double gemm_flops(const GemmDescT<T>& d) {
    const double nb = (double)d.batch * d.batch2, m = d.m, n = d.n, k = d.k;
    const bool ta = d.flags & (kAUpper | kALower), tb = d.flags & (kBUpper | kBLower);
    double f;
    if (ta && tb) f = 2.0 * m * n * k / 3.0;
    else if (ta) f = 2.0 * n * trapezoid_nnz(m, k, d.flags & kAUpper);
    else if (tb) f = 2.0 * m * trapezoid_nnz(n, k, d.flags & kBLower);
    else f = 2.0 * m * n * k;
    if (d.flags & kCUpperTiles) f *= 0.5;
    return f * nb;
}

// Algorithmic memory traffic of a descriptor in bytes: the nonzeros of A and
// B once per batch, Cin when beta != 0 and C once per output (upper-tile
// outputs halved).
template <class T>
double gemm_bytes(const GemmDescT<T>& d) {
    const double nb = (double)d.batch * d.batch2, nout = (double)(d.reduce ? 1 : d.batch) * d.batch2;
    double a = (double)d.m * d.k, b = (double)d.k * d.n, c = (double)d.m * d.n;
    if (d.flags & (kAUpper | kALower)) a = trapezoid_nnz(d.m, d.k, d.flags & kAUpper);
    if (d.flags & (kBUpper | kBLower)) b = trapezoid_nnz(d.n, d.k, d.flags & kBLower);
    if (d.flags & kCUpperTiles) c *= 0.5;
    const double cin = (d.Cin && d.beta != 0.0) ? c : 0.0;
    return sizeof(T) * (nb * (a + b) + nout * (c + cin));
}

// ---------------------------------------------------------------------------
// Small device helpers
// ---------------------------------------------------------------------------
__device__ inline d4 mfma_f64_16x16x4(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 16 x 16 x 4 MFMA tiles for either precision.  Both take A[l % 16][l / 16]
// and B[l / 16][l % 16] from lane l; the accumulator rows differ:
// FP64 holds D[l / 16 + 4 e][l % 16], FP32 holds D[4 (l / 16) + e][l % 16].
template <class T> struct Mfma;
template <> struct Mfma<double> {
    typedef d4 acc;
    __device__ static acc run(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int lane, int e) { return (lane >> 4) + 4 * e; }
};
template <> struct Mfma<float> {
    typedef f4 acc;
    __device__ static acc run(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int lane, int e) { return 4 * (lane >> 4) + e; }
};

// x where mask is -1, +0 where it is 0.  With a mask the compiler cannot see
// through (opaque), a load into x stays unconditional: `in ? load : 0` may
// become a branch around each load, which then waits for them one by one.
__device__ inline double keep_if(double x, int mask) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)u & (unsigned)mask, hi = (unsigned)(u >> 32) & (unsigned)mask;
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline float keep_if(float x, int mask) { return __int_as_float(__float_as_int(x) & mask); }
__device__ inline int opaque(int x) {
    asm("" : "+v"(x));
    return x;
}

// Sets a flag that the host may hold (pinned memory): a store that every
// setter makes alike, no read-modify-write across the bus.
__device__ inline void raise_flag(int* flag) {
    __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int CTRL>
__device__ inline double dpp(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;             // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppRor8 = 0x128, kDppHalfMirror = 0x141;     // lane ^ 8; lane ^ 7
constexpr int kDppRowBcast = 0x150;                         // row_newbcast:0 (+ n: lane n of each row of 16)

// a' = [a.low half, b.low half] and b' = [a.high half, b.high half] over the
// 32-lane halves; the sum adds each value's two halves, a in lanes 0-31, b above.
__device__ inline double swap32_add(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
// The same over neighbouring rows of 16 lanes: a in rows 0 and 2, b in rows 1 and 3.
__device__ inline double swap16_add(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// The sum over a full wave, in every lane: six register moves instead of six
// trips through LDS (some 180 against 900 cycles).
__device__ inline double wave_sum(double v) {
    v = swap32_add(v, v);
    v = swap16_add(v, v);
    v += dpp<kDppRor8>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppXor1>(v);
    return v + dpp<kDppXor2>(v);
}

// Householder reflector of [alpha; x], s2 = |x|^2 > 0: beta = -sign(alpha) |(alpha, x)|,
// tau = (beta - alpha) / beta, scale = 1 / (alpha - beta).  The norm and the two
// reciprocals come from the hardware's estimates of a reciprocal square root and a
// reciprocal by Goldschmidt's coupled iteration (nrm -> sqrt(t), h -> 1 / (2 sqrt(t))) and
// Newton's: half the dependent operations of a square root and two divisions.
// Largest errors over the exponents without underflow, as with those: beta
// 1.6e-16, tau 2.3e-16 (without the last step of its quotient 4.0e-16), scale 3.0e-16.
__device__ __forceinline__ void householder(double alpha, double s2, double& beta, double& tau, double& scale) {
    const double t = fma(alpha, alpha, s2);
    double h = __builtin_amdgcn_rsq(t);
    double nrm = t * h;
    h *= 0.5;
    double e = fma(-h, nrm, 0.5);
    nrm = fma(nrm, e, nrm);
    h = fma(h, e, h);
    const double d = fma(-nrm, nrm, t);
    e = fma(-h, nrm, 0.5);
    nrm = fma(d, h, nrm);
    h = fma(h, e, h);                             // 1 / (2 nrm)
    const double den = fabs(alpha) + nrm;
    double x = __builtin_amdgcn_rcp(den);
    e = fma(-den, x, 1.0);
    x = fma(x, e, x);
    e = fma(-den, x, 1.0);
    x = fma(x, e, x);
    beta = alpha >= 0.0 ? -nrm : nrm;
    const double q = den * (h + h);
    tau = fma(fma(-q, nrm, den), h + h, q);       // the quotient to the last bit, beside the steps of x
    scale = alpha >= 0.0 ? x : -x;
}

// Number of XCDs on MI355X; consecutive workgroup ids are dealt round-robin.
constexpr int kNumXcd = 8;

// Bijective remap of a linear block id so that consecutive logical ids land
// on the same XCD (and so share its L2).
__device__ inline int xcd_remap(int b, int nblocks) {
    if (nblocks < 2 * kNumXcd) return b;
    int q = nblocks / kNumXcd, rem = nblocks % kNumXcd;
    int x = b % kNumXcd, idx = b / kNumXcd;
    int base = x < rem ? x * (q + 1) : rem * (q + 1) + (x - rem) * q;
    return base + idx;
}

}  // namespace zolo
