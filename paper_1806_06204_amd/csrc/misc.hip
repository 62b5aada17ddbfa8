// Memory-bound helper kernels of the Zolo-PD iteration: scaling, copies with
// structure, deterministic two-pass reductions (Frobenius norms, the
// orthogonality residual of a Gram matrix), symmetrisation of H, and the
// matrix-vector products of the power iteration for alpha.
//
// Reductions write one partial per workgroup and a second single-workgroup
// pass sums them in a fixed order, so results do not depend on scheduling.
#include "misc.hpp"

namespace zolo {
namespace {

constexpr int kThreads = 256;

__device__ inline double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
    __syncthreads();
    return s;  // valid in thread 0
}

// X = A * s, reporting non-finite entries of A in *flag.
__global__ void scale_copy_kernel(int m, int n, const double* __restrict__ A, long long lda,
                                  double* __restrict__ X, long long ldx, double s, int* flag) {
    const long long total = (long long)m * n;
    int bad = 0;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / m, i = e - j * m;
        const double v = A[i + j * lda];
        if (!isfinite(v)) bad = 1;
        X[i + j * ldx] = v * s;
    }
    if (bad && flag) raise_flag(flag);
}

// Z_b = G (upper triangle and diagonal) + shift_b I, strict lower part zero.
template <class T>
__global__ void shift_copy_kernel(int n, const T* __restrict__ G, long long ldg,
                                  T* __restrict__ Z, long long ldz, long long sz,
                                  ShiftArgs sh) {
    const long long total = (long long)n * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / n, i = e - j * n;
        const T g = i <= j ? G[i + j * ldg] : (T)0;
        for (int b = 0; b < sh.batch; ++b)
            Z[b * sz + i + j * ldz] = (i == j) ? g + (T)sh.shift[b] : g;
    }
}

// Y = s * X with a change of precision (FP64 <-> FP32).
template <class S, class D>
__global__ void convert_kernel(int m, int n, const S* __restrict__ X, long long ldx, D* __restrict__ Y,
                               long long ldy, double s) {
    const long long total = (long long)m * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / m, i = e - j * m;
        Y[i + j * ldy] = (D)(s * (double)X[i + j * ldx]);
    }
}

// Fill an n x n matrix (batched) with value `diag` on the diagonal and `off` elsewhere,
// or only the strict lower triangle with zero (mode 1).
template <class T>
__global__ void fill_kernel(int m, int n, T* __restrict__ Z, long long ldz, long long sz, int batch,
                            int mode, double diag, double off) {
    const long long total = (long long)m * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / m, i = e - j * m;
        for (int b = 0; b < batch; ++b) {
            T* p = Z + b * sz + i + j * ldz;
            if (mode == 0) *p = (T)((i == j) ? diag : off);
            else if (i > j) *p = (T)0;
        }
    }
}

// Mode 0: S = (C + C^T)/2 (full C); mode 1: S[i][j] = C[min][max] + add_diag * delta_ij
// (mirror the upper triangle); mode 2: the same from the lower triangle.
template <class T>
__global__ void symmetrize_kernel(int n, const T* __restrict__ C, long long ldc,
                                  T* __restrict__ S, long long lds, int mode, double add_diag) {
    const long long total = (long long)n * n;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / n, i = e - j * n;
        T v;
        if (mode == 0) v = (T)0.5 * (C[i + j * ldc] + C[j + i * ldc]);
        else v = ((i <= j) == (mode == 1) ? C[i + j * ldc] : C[j + i * ldc]) + (i == j ? (T)add_diag : (T)0);
        S[i + j * lds] = v;
    }
}

// Partial sums for ||X - Y||_F^2 and ||X||_F^2 (Y may be null).
__global__ void frob_partial_kernel(int m, int n, const double* __restrict__ X, long long ldx,
                                    const double* __restrict__ Y, long long ldy, double* part) {
    __shared__ double sh[kThreads / 64];
    const long long total = (long long)m * n;
    double sd = 0.0, sx = 0.0;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / m, i = e - j * m;
        const double x = X[i + j * ldx];
        sx += x * x;
        if (Y) {
            const double dd = x - Y[i + j * ldy];
            sd += dd * dd;
        }
    }
    const double a = block_sum(sd, sh);
    const double b = block_sum(sx, sh);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = a;
        part[2 * blockIdx.x + 1] = b;
    }
}

// Partial sums of ||G - I||_F^2 from the upper triangle of a symmetric G.
__global__ void orth_partial_kernel(int n, const double* __restrict__ G, long long ldg, double* part) {
    __shared__ double sh[kThreads / 64];
    const long long total = (long long)n * n;
    double s = 0.0;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const long long j = e / n, i = e - j * n;
        if (i <= j) {
            const double v = G[i + j * ldg] - (i == j ? 1.0 : 0.0);
            s += (i == j ? 1.0 : 2.0) * v * v;
        }
    }
    const double a = block_sum(s, sh);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = a;
        part[2 * blockIdx.x + 1] = 0.0;
    }
}

// out[0..1] = sums of the (pairs of) partials, in order.
__global__ void finish_sum_kernel(int nparts, const double* part, double* out) {
    __shared__ double sh[kThreads / 64];
    double a = 0.0, b = 0.0;
    for (int p = threadIdx.x; p < nparts; p += blockDim.x) {
        a += part[2 * p];
        b += part[2 * p + 1];
    }
    const double sa = block_sum(a, sh);
    const double sb = block_sum(b, sh);
    if (threadIdx.x == 0) {
        out[0] = sa;
        out[1] = sb;
    }
}

// y = A x / ||x||  (A m x n, column-major), the first half of a power step.
// A workgroup of 16 waves owns kPowRows rows (one 128-byte line of a column),
// its 64 lane groups every 64th column, so that the rows of a few hundred
// columns are a dozen independent loads per lane; n = 777, m = 1000 runs 63
// workgroups.  One thread per row, the form before, kept 4 workgroups busy with
// one dependent load chain each: 92 us, 9.2 of the 30 ms of a 1000 x 777 solve
// with alpha estimated (now 21 ms).  Every workgroup takes ||x|| itself, so the vectors need
// no normalising pass.  The first workgroup also reports the step before:
// *lam = prev^T x / ||prev|| (x = A^T A prev / ||prev||), skipped when lam is null.
constexpr int kPowRows = 16, kPowThreads = 1024;
__global__ __launch_bounds__(kPowThreads) void power_gemv_kernel(int m, int n, const double* __restrict__ A,
                                                                 long long lda, const double* __restrict__ x,
                                                                 const double* __restrict__ prev,
                                                                 double* __restrict__ y, double* lam) {
    __shared__ double sh[kPowThreads / 64];
    __shared__ double part[kPowThreads / 64][kPowRows];
    __shared__ double s_inv;
    double xx = 0.0, pp = 0.0, px = 0.0;
    const bool report = lam != nullptr && blockIdx.x == 0;
    for (int j = threadIdx.x; j < n; j += kPowThreads) {
        xx += x[j] * x[j];
        if (report) {
            pp += prev[j] * prev[j];
            px += prev[j] * x[j];
        }
    }
    xx = block_sum(xx, sh);
    if (threadIdx.x == 0) s_inv = xx > 0.0 ? 1.0 / sqrt(xx) : 0.0;
    if (report) {
        pp = block_sum(pp, sh);
        px = block_sum(px, sh);
        if (threadIdx.x == 0) *lam = pp > 0.0 ? px / sqrt(pp) : 0.0;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * kPowRows + (lane & (kPowRows - 1));
    const double* col = A + min(row, m - 1);
    double s = 0.0;
#pragma unroll 8
    for (int j = wave * 4 + (lane >> 4); j < n; j += kPowThreads / kPowRows) s += col[(long long)j * lda] * x[j];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < kPowRows) part[wave][lane] = s;
    __syncthreads();
    if (threadIdx.x < kPowRows && row < m) {
        double t = part[0][threadIdx.x];
        for (int w = 1; w < kPowThreads / 64; ++w) t += part[w][threadIdx.x];
        y[row] = t * s_inv;
    }
}

// y = A^T x: one workgroup per column.
__global__ void gemv_t_kernel(int m, int n, const double* __restrict__ A, long long lda,
                              const double* __restrict__ x, double* __restrict__ y) {
    __shared__ double sh[kThreads / 64];
    const int j = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < m; i += blockDim.x) s += A[i + (long long)j * lda] * x[i];
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) y[j] = t;
}

// After the last step: *lam = prev^T w / ||prev||, v <- w / ||w|| (single
// workgroup; v may be prev or w).
__global__ void power_finish_kernel(int n, const double* prev, const double* w, double* v, double* lam) {
    __shared__ double sh[kThreads / 64];
    __shared__ double s_inv;
    double pp = 0.0, pw = 0.0, ww = 0.0;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        pp += prev[j] * prev[j];
        pw += prev[j] * w[j];
        ww += w[j] * w[j];
    }
    pp = block_sum(pp, sh);
    pw = block_sum(pw, sh);
    ww = block_sum(ww, sh);
    if (threadIdx.x == 0) {
        *lam = pp > 0.0 ? pw / sqrt(pp) : 0.0;
        s_inv = ww > 0.0 ? 1.0 / sqrt(ww) : 0.0;
    }
    __syncthreads();
    const double inv = s_inv;
    for (int j = threadIdx.x; j < n; j += blockDim.x) v[j] = w[j] * inv;
}

__global__ void fill_vec_kernel(int n, double* v, double val) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) v[j] = val;
}

// max_j sum_i |R[i][j]| over the upper triangle: one workgroup per column,
// partial column sums written to colsum[j].
__global__ void colsum_abs_upper_kernel(int n, const double* __restrict__ R, long long ldr, double* colsum) {
    __shared__ double sh[kThreads / 64];
    const int j = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i <= j && i < n; i += blockDim.x) s += fabs(R[i + (long long)j * ldr]);
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) colsum[j] = t;
}

__global__ void max_kernel(int n, const double* v, double* out) {
    __shared__ double sh[kThreads];
    double m = 0.0;
    for (int j = threadIdx.x; j < n; j += blockDim.x) m = fmax(m, v[j]);
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

inline int grid_for(long long total) {
    long long g = (total + kThreads - 1) / kThreads;
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace

hipError_t scale_copy(int m, int n, const double* A, long long lda, double* X, long long ldx, double s,
                      int* flag, hipStream_t st) {
    scale_copy_kernel<<<grid_for((long long)m * n), kThreads, 0, st>>>(m, n, A, lda, X, ldx, s, flag);
    return hipGetLastError();
}

template <class T>
hipError_t shift_copy(int n, const T* G, long long ldg, T* Z, long long ldz, long long sz, const ShiftArgs& sh,
                      hipStream_t st) {
    shift_copy_kernel<T><<<grid_for((long long)n * n), kThreads, 0, st>>>(n, G, ldg, Z, ldz, sz, sh);
    return hipGetLastError();
}
template hipError_t shift_copy<double>(int, const double*, long long, double*, long long, long long,
                                       const ShiftArgs&, hipStream_t);
template hipError_t shift_copy<float>(int, const float*, long long, float*, long long, long long, const ShiftArgs&,
                                      hipStream_t);

template <class T>
hipError_t fill_matrix(int m, int n, T* Z, long long ldz, long long sz, int batch, double diag, double off,
                       hipStream_t st) {
    fill_kernel<T><<<grid_for((long long)m * n), kThreads, 0, st>>>(m, n, Z, ldz, sz, batch, 0, diag, off);
    return hipGetLastError();
}
template hipError_t fill_matrix<double>(int, int, double*, long long, long long, int, double, double, hipStream_t);
template hipError_t fill_matrix<float>(int, int, float*, long long, long long, int, double, double, hipStream_t);

template <class T>
hipError_t zero_strict_lower(int n, T* Z, long long ldz, long long sz, int batch, hipStream_t st) {
    fill_kernel<T><<<grid_for((long long)n * n), kThreads, 0, st>>>(n, n, Z, ldz, sz, batch, 1, 0.0, 0.0);
    return hipGetLastError();
}
template hipError_t zero_strict_lower<double>(int, double*, long long, long long, int, hipStream_t);
template hipError_t zero_strict_lower<float>(int, float*, long long, long long, int, hipStream_t);

template <class T>
hipError_t symmetrize(int n, const T* C, long long ldc, T* S, long long lds, int mode, double add_diag,
                      hipStream_t st) {
    symmetrize_kernel<T><<<grid_for((long long)n * n), kThreads, 0, st>>>(n, C, ldc, S, lds, mode, add_diag);
    return hipGetLastError();
}
template hipError_t symmetrize<double>(int, const double*, long long, double*, long long, int, double, hipStream_t);
template hipError_t symmetrize<float>(int, const float*, long long, float*, long long, int, double, hipStream_t);

template <class S, class D>
hipError_t convert(int m, int n, const S* X, long long ldx, D* Y, long long ldy, double s, hipStream_t st) {
    convert_kernel<S, D><<<grid_for((long long)m * n), kThreads, 0, st>>>(m, n, X, ldx, Y, ldy, s);
    return hipGetLastError();
}
template hipError_t convert<double, float>(int, int, const double*, long long, float*, long long, double,
                                           hipStream_t);
template hipError_t convert<float, double>(int, int, const float*, long long, double*, long long, double,
                                           hipStream_t);

hipError_t frob2(int m, int n, const double* X, long long ldx, const double* Y, long long ldy, double* part,
                 double* out, hipStream_t st) {
    const int g = grid_for((long long)m * n) > 1024 ? 1024 : grid_for((long long)m * n);
    frob_partial_kernel<<<g, kThreads, 0, st>>>(m, n, X, ldx, Y, ldy, part);
    finish_sum_kernel<<<1, kThreads, 0, st>>>(g, part, out);
    return hipGetLastError();
}

hipError_t orth2(int n, const double* G, long long ldg, double* part, double* out, hipStream_t st) {
    const int g = grid_for((long long)n * n) > 1024 ? 1024 : grid_for((long long)n * n);
    orth_partial_kernel<<<g, kThreads, 0, st>>>(n, G, ldg, part);
    finish_sum_kernel<<<1, kThreads, 0, st>>>(g, part, out);
    return hipGetLastError();
}

hipError_t power_steps(int m, int n, const double* A, long long lda, int steps, double* v, double* u, double* w,
                       double* lam, hipStream_t st) {
    double* src = v;   // the current vector; dst takes A^T A src / ||src|| and holds the one before until then
    double* dst = w;
    for (int t = 0; t < steps; ++t) {
        power_gemv_kernel<<<(m + kPowRows - 1) / kPowRows, kPowThreads, 0, st>>>(m, n, A, lda, src, dst, u,
                                                                              t > 0 ? lam + t - 1 : nullptr);
        gemv_t_kernel<<<n, kThreads, 0, st>>>(m, n, A, lda, u, dst);
        double* next = dst;
        dst = src;
        src = next;
    }
    if (steps > 0) power_finish_kernel<<<1, kThreads, 0, st>>>(n, dst, src, v, lam + steps - 1);
    return hipGetLastError();
}

__global__ void zero_ints_kernel(int* p, int count) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) p[i] = 0;
}

hipError_t zero_ints(int* p, int count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    int grid = (count + kThreads - 1) / kThreads;
    if (grid > 1024) grid = 1024;
    zero_ints_kernel<<<grid, kThreads, 0, st>>>(p, count);
    return hipGetLastError();
}

hipError_t fill_vector(int n, double* v, double val, hipStream_t st) {
    fill_vec_kernel<<<(n + kThreads - 1) / kThreads, kThreads, 0, st>>>(n, v, val);
    return hipGetLastError();
}

hipError_t norm1_upper(int n, const double* R, long long ldr, double* colsum, double* out, hipStream_t st) {
    colsum_abs_upper_kernel<<<n, kThreads, 0, st>>>(n, R, ldr, colsum);
    max_kernel<<<1, kThreads, 0, st>>>(n, colsum, out);
    return hipGetLastError();
}

}  // namespace zolo
