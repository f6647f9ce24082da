// Start value of V for a cold FP64 Jacobi SVD.
//
// One-sided Jacobi converges slowly on columns that are far from orthogonal
// and far from graded: the Fourier slices of smooth data (singular values
// over 16 orders of magnitude) took 25-29 sweeps in FP64, because V = I
// leaves every column a mix of all of them.  A QR factorisation with column
// pivoting of the slice's conjugate transpose, A^H P = Q R, gives a unitary
// Q with A Q = P R^H: columns graded by the pivoted triangle, on which the
// same Jacobi takes 7-8 sweeps (Drmac and Veselic's preconditioner, taken
// here for V alone: R is never stored, and whatever Q's quality as a
// preconditioner, it is unitary, so the SVD that follows is as exact as
// before).
//
// One workgroup of 8 waves per slice.  X = A^H (n x m) lives in registers: a
// column belongs to a row of 16 lanes (each holds its elements lane + 16 k,
// k < R), a wave holds S columns in each of its four lane rows, so a
// 128 x 160 slice takes 160 of the 256 VGPRs a lane of a 512-thread
// workgroup has.  A step: the lane rows agree on the longest remaining column
// (LDS), its wave forms the Householder vector and puts it in LDS, and every
// lane row reflects its columns; a dot product is reduced with four DPP
// stages, and the rows of X already finished (16 at a time) drop out of the
// unrolled loops.  The reflectors are also kept in global memory, and
// Q = H_0 ... H_{n-1} is accumulated backwards, the columns of Q in
// registers, without barriers.  The steps end early once no remaining column
// is above the rounding level eps ||A||_F: the columns of A Q they would
// order are below the stopping rule's floor.  Tensors whose columns are not
// alike (columns_alike_kernel) keep V = I.
//
// Bound: vector issue of the reflections (two waves per SIMD) and, once a
// step, the owner's serial chain between two barriers.  With a column per
// wave (64 lanes, 16 waves) the reductions were half of the work: 841 us for
// 33 slices of 160 x 128 and 524 us for 75 of 128 x 96, here 447 and 268 us.
// The SVDs after it: 6.81 -> 1.86 ms (smooth video, 27 -> 7.6 sweeps) and
// 4.27 -> 1.30 ms (25 -> 7.2 sweeps).

#include "kernels.h"

namespace tsvd {

namespace {

// Squared norms under this count as 0 (the reciprocals taken of them would overflow).
constexpr double kSeedTiny = 1e-280;

constexpr int kSeedThreads = 512, kSeedWaves = kSeedThreads / 64, kSeedRows = kSeedThreads / 16;

template <int CTRL>
__device__ __forceinline__ double sdpp(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true));
}

// Sum and maximum over the 16 lanes of a row, in every lane of the row.
__device__ __forceinline__ double row_sum(double v) {
    v += sdpp<0xB1>(v);
    v += sdpp<0x4E>(v);
    v += sdpp<0x141>(v);
    v += sdpp<0x140>(v);
    return v;
}

__device__ __forceinline__ double row_max(double v) {
    v = fmax(v, sdpp<0xB1>(v));
    v = fmax(v, sdpp<0x4E>(v));
    v = fmax(v, sdpp<0x141>(v));
    v = fmax(v, sdpp<0x140>(v));
    return v;
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

__device__ __forceinline__ double seed_rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = y * (1.5 - 0.5 * x * y * y);
    return y * (1.5 - 0.5 * x * y * y);
}

__device__ __forceinline__ double seed_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = y * (2.0 - x * y);
    return y * (2.0 - x * y);
}

struct Z2 { double re, im; };

// x <- x - tau (v^H x) v over the rows lane + 16 k, k >= K0.
template <int R, int K0>
__device__ __forceinline__ void reflect(Z2 (&x)[R], const Z2 (&v)[R], double tau) {
    double wr = 0, wi = 0;
#pragma unroll
    for (int k = K0; k < R; ++k) {
        wr = fma(v[k].re, x[k].re, wr);
        wi = fma(v[k].re, x[k].im, wi);
        wr = fma(v[k].im, x[k].im, wr);
        wi = fma(-v[k].im, x[k].re, wi);
    }
    wr = tau * row_sum(wr);
    wi = tau * row_sum(wi);
#pragma unroll
    for (int k = K0; k < R; ++k) {
        x[k].re = fma(-wr, v[k].re, x[k].re);
        x[k].im = fma(-wr, v[k].im, x[k].im);
        x[k].re = fma(wi, v[k].im, x[k].re);
        x[k].im = fma(-wi, v[k].re, x[k].im);
    }
}

// Elements >= j of a column: squared norm, in every lane of the row.
template <int R, int K0>
__device__ __forceinline__ double tail_norm2(const Z2 (&x)[R], int l, int j) {
    double nn = 0.0;
#pragma unroll
    for (int k = K0; k < R; ++k)
        if (l + 16 * k >= j) nn += x[k].re * x[k].re + x[k].im * x[k].im;
    return row_sum(nn);
}

struct SeedShared {
    double best[kSeedRows];
    int idx[kSeedRows];
    double tau;
    Z2 v[128];
    double taus[128];
};

template <int R, int S>
struct SeedState {
    Z2 x[S][R];        // the lane row's columns of A^H
    double cn[S];      // remaining squared norms (elements >= step); < 0 once taken
    float cref[S];     // their value when last computed from the column, over the power of two of ||A||_F^2
};

// A remaining norm is recomputed from its column under 1e-6 of its last
// computed value.  Those are kept in FP32 over 2^e, the power of two next to
// ||A||_F^2, so that the steps are the same at every scale of the data (as they
// come they are 0 for entries under 1e-23, where no norm would be recomputed,
// and infinite over 1e19, where every one would at every step).  e and stop2
// (the rounding level of the norms) are scalar: the columns fill the vector
// registers.
// Steps j >= 16 K0; returns the steps done.
template <int R, int S, int K0>
__device__ __forceinline__ int seed_steps(SeedState<R, S>& st, SeedShared& sh, int n, double stop2, int e,
                                          cplx<double>* G) {
    const int lane = threadIdx.x & 63, l = lane & 15, row = threadIdx.x >> 4;
    const int j1 = min(16 * (K0 + 1), n);
    for (int j = 16 * K0; j < j1; ++j) {
        const int jl = j & 15;
        double best = -1.0;
        int bi = 0;
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (st.cn[i] > best) {
                best = st.cn[i];
                bi = i;
            }
        if (l == 0) {
            sh.best[row] = best;
            sh.idx[row] = bi;
        }
        __syncthreads();
        const double own = sh.best[lane & (kSeedRows - 1)];
        const double m16 = row_max(own);
        const double mx = fmax(lane_f64(m16, 0), lane_f64(m16, 16));
        if (!(mx > stop2)) return j;   // the same value in every wave; also when it is not finite
        const int ro = __builtin_ctzll(__ballot(own == mx));   // the row that owns the step
        if ((row & ~3) == (ro & ~3)) {
            // its wave forms the vector (the other three rows repeat their own,
            // which nobody reads)
            const int pick = __builtin_amdgcn_readfirstlane(sh.idx[ro]);
            const bool mine = row == ro;
            Z2 c[R];
#pragma unroll
            for (int i = 0; i < S; ++i)
                if (i == pick) {
#pragma unroll
                    for (int k = K0; k < R; ++k) c[k] = st.x[i][k];
                    if (mine) st.cn[i] = -1.0;
                }
            const double nn = tail_norm2<R, K0>(c, l, j);
            const double ar = __shfl(c[K0].re, (lane & 48) | jl), ai = __shfl(c[K0].im, (lane & 48) | jl);
            // v = x + e^{i arg(x_j)} ||x|| e_j, tau = 2 / ||v||^2 = 1 / (||x|| (||x|| + |x_j|))
            const double a2 = ar * ar + ai * ai;
            const double nx = nn * seed_rsqrt(nn), ra = seed_rsqrt(a2);
            const bool none = !(nn > kSeedTiny), real = !(a2 > kSeedTiny);   // nothing left; x_j counts as 0
            const double f = real ? 0.0 : nx * ra;
            const double tau = none ? 0.0 : seed_rcp(nn + (real ? 0.0 : nx * (a2 * ra)));
            if (l == jl) c[K0] = none ? Z2{0.0, 0.0} : real ? Z2{nx, 0.0} : Z2{fma(f, ar, ar), fma(f, ai, ai)};
            if (mine) {
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const int r = l + 16 * k;
                    const Z2 t = k < K0 || r < j ? Z2{0.0, 0.0} : c[k];
                    if (r < n) {
                        sh.v[r] = t;
                        G[(int64_t)j * n + r] = cplx<double>{t.re, t.im};
                    }
                }
                if (l == 0) {
                    sh.tau = tau;
                    sh.taus[j] = tau;
                }
            }
        }
        __syncthreads();
        const double tau = sh.tau;
        Z2 v[R];
#pragma unroll
        for (int k = K0; k < R; ++k) {
            const int r = l + 16 * k;
            v[k] = r < n ? sh.v[r] : Z2{0.0, 0.0};
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            reflect<R, K0>(st.x[i], v, tau);
            // row j leaves the remaining norm; it is recomputed from the
            // column when cancellation has eaten the difference
            const double t = st.x[i][K0].re * st.x[i][K0].re + st.x[i][K0].im * st.x[i][K0].im;
            double c = st.cn[i];
            if (c > 0.0) c = fmax(c - __shfl(t, (lane & 48) | jl), 0.0);
            if (__any(c >= 0.0 && c < 1e-6 * ldexp((double)st.cref[i], e))) {
                const double nn = tail_norm2<R, K0>(st.x[i], l, j + 1);
                if (c >= 0.0) {
                    c = nn;
                    st.cref[i] = (float)ldexp(nn, -e);
                }
            }
            st.cn[i] = c;
        }
    }
    return -1;
}

template <int R, int S, int K0 = 0>
__device__ __forceinline__ int seed_all(SeedState<R, S>& st, SeedShared& sh, int n, double stop2, int e,
                                        cplx<double>* G) {
    const int d = seed_steps<R, S, K0>(st, sh, n, stop2, e, G);
    if (d >= 0 || n <= 16 * (K0 + 1)) return d < 0 ? n : d;
    if constexpr (K0 + 1 < R) return seed_all<R, S, K0 + 1>(st, sh, n, stop2, e, G);
    return n;
}

// Backward accumulation Q <- H_j Q, j from j_end - 1 down, Q from the
// identity: lane row `row` holds columns row + 32 i, rows below a reflector's
// first element are still unit vectors.
template <int R, int QS, int K0>
__device__ __forceinline__ void seed_back(Z2 (&q)[QS][R], const SeedShared& sh, int n, int j_end,
                                          const cplx<double>* G) {
    const int l = threadIdx.x & 15, row = threadIdx.x >> 4;
    const int wrow = __builtin_amdgcn_readfirstlane(row | 3);   // the wave's highest column of a slot
    const int j0 = 16 * K0, j1 = min(j_end, 16 * (K0 + 1));
    Z2 nv[R];
    auto fetch = [&](int j) {
#pragma unroll
        for (int k = K0; k < R; ++k) {
            const int r = l + 16 * k;
            const cplx<double> t = r < n ? G[(int64_t)j * n + r] : cplx<double>{0.0, 0.0};
            nv[k] = Z2{t.re, t.im};
        }
    };
    if (j1 > j0) fetch(j1 - 1);
    for (int j = j1 - 1; j >= j0; --j) {
        Z2 v[R];
#pragma unroll
        for (int k = K0; k < R; ++k) v[k] = nv[k];
        if (j > j0) fetch(j - 1);
        const double tau = sh.taus[j];
#pragma unroll
        for (int i = 0; i < QS; ++i)
            if (wrow + kSeedRows * i >= j) reflect<R, K0>(q[i], v, tau);
    }
    if constexpr (K0 > 0) seed_back<R, QS, K0 - 1>(q, sh, n, j_end, G);
}

// *alike = 1 if a slice's neighbouring columns are alike: |cos|^2 of their angle,
// on average over up to 64 pairs that are not zero, over kAlike times the 1 / m
// of random columns.  A row of 16 lanes takes a pair.
//
// The QR pays on smooth data and on low rank (25-29 sweeps from V = I, 7-8 with
// it); independent columns, or columns orthogonal already, converge from V = I
// as soon, and its 60 to 450 us are lost.  t-SVTs that always took it, and now,
// us: 256 x 32 x 8 noise 483, 391; 160 x 100 x 20 noise 1729, 1418, with columns
// scaled over six decades 1607, 947; 128 x 160 x 64 diagonal 685, 263.  The
// whole tensor takes it when one of its slices is alike: a few slices without
// it would be the last to finish.  This launch is 7 us (33 slices of 160 x 128),
// so slices up to kAlikeEntries, whose QR is short, take it unasked.
constexpr double kAlike = 2.0;
constexpr int kAlikeThreads = 1024, kAlikeRows = kAlikeThreads / 16;
constexpr int kAlikeEntries = 32 * 32;

__global__ __launch_bounds__(kAlikeThreads) void columns_alike_kernel(const cplx<double>* A, int m, int n,
                                                                      int* alike) {
    __shared__ double cos2[kAlikeRows];
    __shared__ int pairs[kAlikeRows];
    const int l = threadIdx.x & 15, row = threadIdx.x >> 4;
    const cplx<double>* const a = A + (int64_t)blockIdx.x * n * m;
    double sum = 0.0;
    int count = 0;
    const int r = row * ((n - 2) / kAlikeRows + 1);
    if (r < n - 1) {
        const cplx<double>*const x = a + (int64_t)r * m, *const y = x + m;
        double xx = 0.0, yy = 0.0, dr = 0.0, di = 0.0;
#pragma unroll 8
        for (int i = l; i < m; i += 16) {
            const cplx<double> p = x[i], q = y[i];
            xx += p.re * p.re + p.im * p.im;
            yy += q.re * q.re + q.im * q.im;
            dr += p.re * q.re + p.im * q.im;
            di += p.re * q.im - p.im * q.re;
        }
        const double s = sqrt(row_sum(xx)) * sqrt(row_sum(yy));
        dr = row_sum(dr) / s;
        di = row_sum(di) / s;
        if (s > 0.0) {
            sum = dr * dr + di * di;
            count = 1;
        }
    }
    if (l == 0) {
        cos2[row] = sum;
        pairs[row] = count;
    }
    __syncthreads();
    if (threadIdx.x < kAlikeRows) {
        double c = cos2[threadIdx.x];
        int k = pairs[threadIdx.x];
        for (int off = kAlikeRows / 2; off > 0; off >>= 1) {
            c += __shfl_xor(c, off, 64);
            k += __shfl_xor(k, off, 64);
        }
        if (threadIdx.x == 0 && c * m > kAlike * k) *alike = 1;
    }
}

// alike: the answer of columns_alike_kernel, or null.
template <int R, int S>
__global__ __launch_bounds__(kSeedThreads) void jacobi_seed_kernel(const cplx<double>* A, cplx<double>* V,
                                                                   cplx<double>* G, int m, int n,
                                                                   const int* alike) {
    __shared__ SeedShared sh;
    __shared__ double fro[kSeedRows];
    const int l = threadIdx.x & 15, row = threadIdx.x >> 4;
    const int64_t s = blockIdx.x;
    if (alike && *alike == 0) {
        for (int i = threadIdx.x; i < n * n; i += kSeedThreads)
            V[s * n * n + i] = cplx<double>{i % n == i / n ? 1.0 : 0.0, 0.0};
        return;
    }
    const cplx<double>* a = A + s * n * m;
    cplx<double>* g = G + s * n * n;
    int done;
    {
        SeedState<R, S> st;
        double part = 0.0;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int c = row * S + i;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int r = l + 16 * k;
                const cplx<double> t = c < m && r < n ? a[(int64_t)r * m + c] : cplx<double>{0.0, 0.0};
                st.x[i][k] = Z2{t.re, -t.im};
            }
            const double nn = tail_norm2<R, 0>(st.x[i], l, 0);
            part += nn;
            st.cn[i] = c < m ? nn : -1.0;
        }
        if (l == 0) fro[row] = part;
        __syncthreads();
        double f2 = 0.0;
        for (int w = 0; w < kSeedRows; ++w) f2 += fro[w];
        const int e = __builtin_amdgcn_readfirstlane(f2 > kSeedTiny ? ilogb(f2) : 0);
#pragma unroll
        for (int i = 0; i < S; ++i) st.cref[i] = (float)ldexp(st.cn[i], -e);
        const double stop2 = lane_f64(fmax(4.93e-32 * f2, kSeedTiny), 0);   // eps^2 ||A||_F^2
        done = seed_all<R, S>(st, sh, n, stop2, e, g);
    }
    __syncthreads();   // the reflectors of every wave are in memory
    constexpr int QS = (16 * R + kSeedRows - 1) / kSeedRows;
    Z2 q[QS][R];
#pragma unroll
    for (int i = 0; i < QS; ++i)
#pragma unroll
        for (int k = 0; k < R; ++k) q[i][k] = Z2{l + 16 * k == row + kSeedRows * i ? 1.0 : 0.0, 0.0};
    seed_back<R, QS, R - 1>(q, sh, n, done, g);
    cplx<double>* const out = V + s * n * n;
#pragma unroll
    for (int i = 0; i < QS; ++i) {
        const int c = row + kSeedRows * i;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int r = l + 16 * k;
            if (c < n && r < n) out[(int64_t)c * n + r] = cplx<double>{q[i][k].re, q[i][k].im};
        }
    }
}

// Columns of A^H per lane row that the registers hold, by rows per lane
constexpr int seed_max_slots(int R) { return R <= 4 ? 8 : (R <= 6 ? 6 : 5); }

int seed_rows_per_lane(int n) { return n <= 32 ? 2 : (n <= 64 ? 4 : (n <= 96 ? 6 : 8)); }

template <int R, int S>
void launch_seed_t(const cplx<double>* A, cplx<double>* V, cplx<double>* G, int m, int n, int h, const int* alike,
                   hipStream_t st) {
    if constexpr (S < seed_max_slots(R)) {
        if (m > kSeedRows * S) return launch_seed_t<R, S + 1>(A, V, G, m, n, h, alike, st);
    }
    hipLaunchKernelGGL((jacobi_seed_kernel<R, S>), dim3(h), dim3(kSeedThreads), 0, st, A, V, G, m, n, alike);
}

}  // namespace

bool jacobi_seed_fits(int m, int n) {
    return n >= 2 && n <= 128 && m <= kSeedRows * seed_max_slots(seed_rows_per_lane(n));
}

void launch_jacobi_seed(const cplx<double>* A, cplx<double>* V, cplx<double>* G, int m, int n, int h, int* alike,
                        hipStream_t st) {
    if (m * n <= kAlikeEntries) alike = nullptr;
    if (alike) hipLaunchKernelGGL(columns_alike_kernel, dim3(h), dim3(kAlikeThreads), 0, st, A, m, n, alike);
    switch (seed_rows_per_lane(n)) {
        case 2: return launch_seed_t<2, 1>(A, V, G, m, n, h, alike, st);
        case 4: return launch_seed_t<4, 2>(A, V, G, m, n, h, alike, st);
        case 6: return launch_seed_t<6, 3>(A, V, G, m, n, h, alike, st);
        default: return launch_seed_t<8, 4>(A, V, G, m, n, h, alike, st);
    }
}

}  // namespace tsvd
