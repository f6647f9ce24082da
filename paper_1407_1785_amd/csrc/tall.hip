// Tall slices in the FP32 form: the SVD of an m x n slice, m >> n, through
// its n x n Gram matrix in FP64.
//
// The vectorised baselines (Sec. 3's unfoldings) give one slice of 10^4 rows
// and tens of columns.  One-sided Jacobi on its columns streams the whole
// slice once per column pairing, some 2 x 63 launches a sweep of a
// 20480 x 64 unfolding, 2.2 ms an ADMM iteration.  Here
//   G = A^H A           products exact and sums in FP64 (the data are FP32),
//   G = R^H R           Cholesky with complete pivoting, rows in pivot order,
//   R V                 the FP64 Jacobi of jacobi_persist.hip on an n x n slice,
// and V is the slice's right singular vectors: G carries singular values down
// to sqrt(eps64) = 1.5e-8 of the largest, under the FP32 rounding of A's own
// entries, so V and sigma come out closer to the exact ones than the FP32
// rotations left them.  The thresholded slice is A (V diag(d) V^H), one
// product; where the left vectors are asked for, A V is swept orthogonal once
// more (left_vectors in capi.hip).  In FP64 the Gram matrix would lose half the digits, so FP64
// unfoldings keep the global-memory Jacobi (jacobi.hip).
//
// gram_partial: one workgroup per chunk of rows, the chunk staged through LDS
// 64 rows at a time, FP64 16 x 16 x 4 matrix products over the tiles on and
// above the diagonal (one real product for a matrix, four for a complex slice).
// Bound: the FP64 matrix rate (8 m n^2 flops halved by symmetry; a 20480 x 64
// matrix is 0.17 GFLOP) beside one read of the slice.
//
// Measured, completion of a 20480 x 64 matrix: 2.50 -> 0.45 ms an iteration
// (Gram 30 + 6 us, Cholesky 44, Jacobi 270 in 4.2 sweeps of 64 us, products 23 +
// 4 x 7, the transforms 61 + 66 -> 6 + 14 us), 30 iterations 3e-4 -> 9e-8 from
// 64-bit LAPACK.

#include "kernels.h"

#include <algorithm>

namespace tsvd {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kGramRows = 64;                  // rows staged at a time
constexpr int kGramLd = kGramRows + 2;         // LDS column stride (elements)
constexpr int kGramTiles = 6;                  // 16 x 16 tiles a wave accumulates
static_assert(kMaxGramCols / 16 * (kMaxGramCols / 16 + 1) / 2 <= kGramTiles * (kBlock / 64) &&
                  kMaxGramCols % 16 == 0,
              "the tiles on and above the diagonal fit the waves' accumulators");
static_assert(kMaxGramCols * kGramLd * sizeof(cplx<float>) <= 64 * 1024, "the staged rows fit the default LDS limit");

// partial[(chunk * h + s) * n^2 + col * n + row], every entry of the n x n
// matrix of chunk `chunk` of slice s.
template <bool REAL>
__global__ __launch_bounds__(kBlock) void gram_partial_kernel(const cplx<float>* A, int m, int n, int h, int rows_per,
                                                              cplx<double>* partial, const Ctrl* ctrl) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (ctrl && ctrl->done) return;
    cplx<float>* const buf = reinterpret_cast<cplx<float>*>(smem);   // [col < np][row]
    const int chunk = blockIdx.x, s = blockIdx.y;
    const int r0 = chunk * rows_per, r1 = min(r0 + rows_per, m);
    const cplx<float>* const a = A + (int64_t)s * n * m;
    const int nt = (n + 15) / 16, np = nt * 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c16 = lane & 15, kq = lane >> 4;
    v4d re[kGramTiles], im[kGramTiles];
#pragma unroll
    for (int i = 0; i < kGramTiles; ++i) re[i] = im[i] = v4d{0.0, 0.0, 0.0, 0.0};
    for (int b0 = r0; b0 < r1; b0 += kGramRows) {
        __syncthreads();
        // rows past the chunk and columns past n are zero
        for (int c = wave; c < np; c += kBlock / 64) {
            const bool in = c < n && b0 + lane < r1;
            const cplx<float> v = in ? a[(int64_t)c * m + b0 + lane] : cplx<float>{0.f, 0.f};
            buf[c * kGramLd + lane] = v;
        }
        __syncthreads();
        int t = 0;
        for (int ti = 0, ix = 0; ti < nt; ++ti)
            for (int tj = ti; tj < nt; ++tj, ++ix) {
                if ((ix & 3) != wave) continue;
                const cplx<float>* pi = buf + (ti * 16 + c16) * kGramLd + kq;
                const cplx<float>* pj = buf + (tj * 16 + c16) * kGramLd + kq;
                v4d tr = v4d{0.0, 0.0, 0.0, 0.0}, tm = tr;
#pragma unroll 4
                for (int k = 0; k < kGramRows; k += 4) {
                    const cplx<float> x = pi[k], y = pj[k];
                    tr = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x.re, (double)y.re, tr, 0, 0, 0);
                    if (!REAL) {
                        // conj(x) y = (xr yr + xi yi) + i (xr yi - xi yr)
                        tr = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x.im, (double)y.im, tr, 0, 0, 0);
                        tm = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x.re, (double)y.im, tm, 0, 0, 0);
                        tm = __builtin_amdgcn_mfma_f64_16x16x4f64(-(double)x.im, (double)y.re, tm, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int i = 0; i < kGramTiles; ++i)
                    if (i == t) {
                        re[i] += tr;
                        if (!REAL) im[i] += tm;
                    }
                ++t;
            }
    }
    cplx<double>* const out = partial + ((int64_t)chunk * h + s) * n * n;
    int t = 0;
    for (int ti = 0, ix = 0; ti < nt; ++ti)
        for (int tj = ti; tj < nt; ++tj, ++ix) {
            if ((ix & 3) != wave) continue;
            v4d tr = v4d{0.0, 0.0, 0.0, 0.0}, tm = tr;
#pragma unroll
            for (int i = 0; i < kGramTiles; ++i)
                if (i == t) {
                    tr = re[i];
                    tm = im[i];
                }
            ++t;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = ti * 16 + 4 * v + kq, j = tj * 16 + c16;   // G(i, j)
                if (i >= n || j >= n) continue;
                out[(int64_t)j * n + i] = cplx<double>{tr[v], tm[v]};
                if (ti != tj) out[(int64_t)i * n + j] = cplx<double>{tr[v], -tm[v]};
            }
        }
}

// G = sum of the chunks in a fixed order: four threads per entry.
__global__ __launch_bounds__(kBlock) void gram_sum_kernel(const cplx<double>* partial, int chunks, int64_t total,
                                                          cplx<double>* G, const Ctrl* ctrl) {
    if (ctrl && ctrl->done) return;
    __shared__ cplx<double> part[4][64];
    const int e = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + e;
    cplx<double> acc{0.0, 0.0};
    if (i < total) {
        const int per = (chunks + 3) / 4, c1 = min((q + 1) * per, chunks);
#pragma unroll 8
        for (int c = q * per; c < c1; ++c) {
            const cplx<double> v = partial[(int64_t)c * total + i];
            acc.re += v.re;
            acc.im += v.im;
        }
    }
    part[q][e] = acc;
    __syncthreads();
    if (q == 0 && i < total)
        G[i] = cplx<double>{(part[0][e].re + part[1][e].re) + (part[2][e].re + part[3][e].re),
                            (part[0][e].im + part[1][e].im) + (part[2][e].im + part[3][e].im)};
}

// G = R^H R with complete pivoting, one workgroup of 8 waves per slice, the
// remaining matrix in registers: wave w holds the columns w + 8 c, a lane the
// rows lane + 64 k (NC columns and NR rows).  Row k of R (over the original
// columns) is the pivot row of the remaining matrix over the root of its
// pivot; the steps end at pivots under n eps of the first, and the rows after
// them are zero.  Every wave follows the remaining diagonal itself, so a step
// has one barrier: the pivot column's wave puts the row of R into LDS, and
// every wave subtracts its product.  With the matrix in LDS and two barriers
// a step the factorisation of a 64 x 64 matrix took 142 us.
constexpr int kCholThreads = 512, kCholWaves = kCholThreads / 64;
static_assert(kMaxGramCols <= 2 * 64 && kMaxGramCols % kCholWaves == 0,
              "two rows a lane and whole columns a wave hold the largest matrix");

template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
    return fmax(v, __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                                    __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true)));
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

__device__ __forceinline__ double wave_max(double v) {
    v = dpp_max<0xB1>(v);
    v = dpp_max<0x4E>(v);
    v = dpp_max<0x141>(v);
    v = dpp_max<0x140>(v);
    return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}

template <int NR, int NC>
__global__ __launch_bounds__(kCholThreads) void chol_kernel(const cplx<double>* G, int n, cplx<double>* R,
                                                            const Ctrl* ctrl) {
    __shared__ cplx<double> row[2][64 * NR];
    if (ctrl && ctrl->done) return;
    const int64_t s = blockIdx.x;
    const cplx<double>* const g = G + s * n * n;
    cplx<double>* const out = R + s * n * n;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double sr[NC][NR], si[NC][NR], d[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int i = lane + 64 * k;
        d[k] = i < n ? g[(int64_t)i * n + i].re : -1.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int j = wave + kCholWaves * c;
            const cplx<double> v = i < n && j < n ? g[(int64_t)j * n + i] : cplx<double>{0.0, 0.0};
            sr[c][k] = v.re;
            si[c][k] = v.im;
        }
    }
    // rows of R not reached stay zero
    for (int idx = threadIdx.x; idx < n * n; idx += kCholThreads) out[idx] = cplx<double>{0.0, 0.0};
    __syncthreads();
    double stop = 0.0;
    for (int k = 0; k < n; ++k) {
        double m = d[0];
#pragma unroll
        for (int q = 1; q < NR; ++q) m = fmax(m, d[q]);
        m = wave_max(m);
        if (k == 0) stop = 2.220446049250313e-16 * n * m;
        if (!(m > stop) || !(m > 0.0)) break;   // the same in every wave
        // the pivot: the lowest column with that diagonal
        int p = 0;
#pragma unroll
        for (int q = NR - 1; q >= 0; --q) {
            const unsigned long long b = __ballot(d[q] == m);
            if (b) p = 64 * q + __builtin_ctzll(b);
        }
        cplx<double>* const rw = row[k & 1];
        if (p % kCholWaves == wave) {
            const double inv = 1.0 / sqrt(m);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (c == p / kCholWaves) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        // R(k, i) = S(p, i) / root = conj(S(i, p)) / root; taken columns are 0
                        const bool live = d[q] >= 0.0;
                        const cplx<double> r{live ? sr[c][q] * inv : 0.0, live ? -si[c][q] * inv : 0.0};
                        rw[lane + 64 * q] = r;
                        if (lane + 64 * q < n) out[(int64_t)(lane + 64 * q) * n + k] = r;
                    }
                }
        }
        __syncthreads();
        cplx<double> ri[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            ri[q] = rw[lane + 64 * q];
            // a remaining diagonal entry stays >= 0; the pivot's leaves
            if (d[q] >= 0.0) d[q] = lane + 64 * q == p ? -1.0 : fmax(d[q] - (ri[q].re * ri[q].re + ri[q].im * ri[q].im), 0.0);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const cplx<double> rj = rw[min(wave + kCholWaves * c, n - 1)];
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                // S(i, j) -= conj(r_i) r_j
                sr[c][q] = fma(-ri[q].re, rj.re, sr[c][q]);
                si[c][q] = fma(-ri[q].re, rj.im, si[c][q]);
                sr[c][q] = fma(-ri[q].im, rj.im, sr[c][q]);
                si[c][q] = fma(ri[q].im, rj.re, si[c][q]);
            }
        }
    }
}

template <typename S, typename D>
__global__ __launch_bounds__(kBlock) void convert_kernel(const cplx<S>* src, cplx<D>* dst, int64_t n,
                                                         const Ctrl* ctrl) {
    if (ctrl && ctrl->done) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = cplx<D>{(D)src[i].re, (D)src[i].im};
}

size_t gram_lds(int n) { return (size_t)((n + 15) / 16 * 16) * kGramLd * sizeof(cplx<float>); }

}  // namespace

// At most one chunk per 128 rows and 160 in all (the sum over the chunks reads
// them once more), and no more than the second slice buffer holds beside four
// n x n matrices: chunks + 4 <= m / (2 n).
int gram_chunks(int m, int n) { return std::max(1, std::min({160, (m + 127) / 128, m / (2 * n) - 4})); }

void launch_gram(const cplx<float>* A, int m, int n, int h, bool real, cplx<double>* partial, cplx<double>* G,
                 const Ctrl* ctrl, hipStream_t st) {
    const int chunks = gram_chunks(m, n), per = (m + chunks - 1) / chunks;
    const size_t lds = gram_lds(n);
    if (real)
        hipLaunchKernelGGL((gram_partial_kernel<true>), dim3(chunks, h), dim3(kBlock), lds, st, A, m, n, h, per,
                           partial, ctrl);
    else
        hipLaunchKernelGGL((gram_partial_kernel<false>), dim3(chunks, h), dim3(kBlock), lds, st, A, m, n, h, per,
                           partial, ctrl);
    const int64_t total = (int64_t)h * n * n;
    hipLaunchKernelGGL(gram_sum_kernel, dim3((unsigned)((total + 63) / 64)), dim3(kBlock), 0, st, partial, chunks,
                       total, G, ctrl);
}

void launch_chol(const cplx<double>* G, int n, int h, cplx<double>* R, const Ctrl* ctrl, hipStream_t st) {
    if (n <= 64)
        hipLaunchKernelGGL((chol_kernel<1, 8>), dim3(h), dim3(kCholThreads), 0, st, G, n, R, ctrl);
    else
        hipLaunchKernelGGL((chol_kernel<2, kMaxGramCols / kCholWaves>), dim3(h), dim3(kCholThreads), 0, st, G, n, R,
                           ctrl);
}

template <typename S, typename D>
void launch_convert(const cplx<S>* src, cplx<D>* dst, int64_t n, const Ctrl* ctrl, hipStream_t st) {
    const int64_t blocks = std::min<int64_t>((n + kBlock - 1) / kBlock, 1024);
    hipLaunchKernelGGL((convert_kernel<S, D>), dim3((unsigned)blocks), dim3(kBlock), 0, st, src, dst, n, ctrl);
}

template void launch_convert<float, double>(const cplx<float>*, cplx<double>*, int64_t, const Ctrl*, hipStream_t);
template void launch_convert<double, float>(const cplx<double>*, cplx<float>*, int64_t, const Ctrl*, hipStream_t);

}  // namespace tsvd
