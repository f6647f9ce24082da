// Device helpers shared by the Jacobi kernels that keep column blocks in
// LDS (jacobi_persist.hip: several workgroups per slice; jacobi_slice.hip:
// one workgroup per slice).  See jacobi.hip for the rotation and the block
// round-robin ordering.
#pragma once

#include "kernels.h"

namespace tsvd {
namespace jac {

__device__ __forceinline__ int pblk_start(int b, int n, int nb) {
    return (int)(((int64_t)b * n) / nb);
}

__device__ __forceinline__ int ppos_player(int pos, int r, int nb) {
    return pos == 0 ? 0 : 1 + (pos - 1 + r) % (nb - 1);
}

// Position, in global round R (counted over the sweeps, nb - 1 a sweep), of the
// block in slot 0 of worker g of a slice; slot 1 holds the block at nb - 1
// minus it.  Between rounds every block but the one at position 0 moves one
// position down (from 1 to nb - 1), and one of the two positions of a pair is
// even and one odd (nb - 1 is odd).  Instead of two blocks per worker on fixed
// positions, the block at the even position stays with its worker, which takes
// over that block's next pair, and only the block at the odd position goes to
// another worker: half the traffic between rounds for the same pairs.  The
// slots replace their block by turns (worker 0, which keeps block 0: slot 1).
// An exchange is bound by the round trip through the coherence point and, with
// two workgroups on every CU, by its rate (69 MB a round in 14 us for 33 slices
// of 256 x 256).  Against two moving blocks: 256 x 256 x 64 FP32 RPCA 2.74 -> 2.43
// ms an iteration, 128 x 160 x 64 completion 1.15 -> 1.05 ms in FP64 and 0.387 ->
// 0.366 ms in FP32, a batch of uneven FP32 completions 346 -> 296 ms.
__device__ __forceinline__ int ppos_slot0(int g, int R) {
    return g == 0 || (R & 1) == 0 ? g : (g & 1 ? g + 1 : g - 1);
}

// DPP lane exchange within a 16-lane row.  Every lane reads a valid source
// for the controls used here; with bound_ctrl the exchange folds into the
// consuming add as a DPP source operand.
template <int CTRL>
__device__ __forceinline__ float pdpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double pdpp(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true));
}

// Sum of the two 16-lane rows 2r and 2r + 1, in every lane of both.
// v_permlane16_swap exchanges the odd rows of its first operand with the
// even rows of its second; with both operands holding v, the two registers
// then hold row 2r and row 2r + 1 of v in every lane of the row pair.  The
// instruction is issued from a register-only asm block (no memory access)
// because the compiler's builtin for it returns its first result for both
// results; the s_nop pairs cover the VALU-write / cross-lane-read wait
// states on both sides.
__device__ __forceinline__ float rowpair_sum(float v) {
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

__device__ __forceinline__ double rowpair_sum(double v) {
    unsigned al = (unsigned)__double2loint(v), bl = al;
    unsigned ah = (unsigned)__double2hiint(v), bh = ah;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\ts_nop 1"
                 : "+v"(al), "+v"(bl), "+v"(ah), "+v"(bh));
    return __hiloint2double((int)ah, (int)al) + __hiloint2double((int)bh, (int)bl);
}

// rowpair_sum of several independent values, their swaps in one block.
__device__ __forceinline__ void rowpair_sum2(float& v, float& w) {
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    unsigned c = __builtin_bit_cast(unsigned, w), d = c;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\ts_nop 1"
                 : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
    v = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
    w = __builtin_bit_cast(float, c) + __builtin_bit_cast(float, d);
}

__device__ __forceinline__ void rowpair_sum2(double& v, double& w) {
    v = rowpair_sum(v);
    w = rowpair_sum(w);
}

// Sum over the PG lanes of a pair group, in the element type; every lane of
// the group gets the same bits (each stage adds two equal-shaped partial
// sums, and addition is commutative).  16 lanes = one DPP row; 32 lanes =
// two rows.
template <int PG, typename T>
__device__ __forceinline__ T group_sum(T v) {
    v += pdpp<0xB1>(v);    // lane ^ 1
    v += pdpp<0x4E>(v);    // lane ^ 2
    v += pdpp<0x141>(v);   // other quad of the half row
    v += pdpp<0x140>(v);   // other half of the row
    if (PG == 32) v = rowpair_sum(v);
    return v;
}

// group_sum of two independent values, their exchange stages interleaved
// (each value gets exactly the additions group_sum gives it).
template <int PG, typename T>
__device__ __forceinline__ void group_sum2(T& a, T& b) {
    a += pdpp<0xB1>(a);
    b += pdpp<0xB1>(b);
    a += pdpp<0x4E>(a);
    b += pdpp<0x4E>(b);
    a += pdpp<0x141>(a);
    b += pdpp<0x141>(b);
    a += pdpp<0x140>(a);
    b += pdpp<0x140>(b);
    if (PG == 32) rowpair_sum2(a, b);
}

// 1/sqrt(x) and 1/x from the hardware estimates with Newton steps: NS = 2
// reaches FP64 accuracy, NS = 1 about 2^-44 (enough when the results are
// rounded to FP32).
template <int NS>
__device__ __forceinline__ double prsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < NS; ++i) y = y * (1.5 - 0.5 * x * y * y);
    return y;
}

__device__ __forceinline__ double prcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    return y * (2.0 - x * y);
}

// Rotation of a pair from alpha, beta, gamma (FP64): c, and s e = a + i b.
// Also returns t |gamma|, the amount that moves from ||x||^2 to ||y||^2.
struct PRot {
    double c, a, b, tg;
    bool on;
};

// The pair is rotated when |gamma|^2 > tol^2 alpha beta, and where that is not
// (much) larger, kMinGamma2; 0 in the FP32 form, whose gamma cannot come near
// it.  The sum of the two bounds costs no instruction (a tracked alpha may be
// rounded below 0: then d^2 alone is normal and a rotation by 0 is exact).  As a
// comparison of its own, against a 64-bit constant, it was 0.6% of a 128 x 160 x
// 64 FP64 completion, as the larger of both 1% of a 96 x 128 x 3 x 48 prox.
template <typename T>
__device__ __forceinline__ bool prot_needed(double al, double be, double g2, double tol) {
    if constexpr (sizeof(T) == 4) return g2 > (tol * tol) * al * be && g2 > 0.0;
    return g2 > fma((tol * tol) * al, be, kMinGamma2);
}

// The rotation through d = beta - alpha and r = sqrt(d^2 + 4 |gamma|^2)
// rather than the cotangent zeta = d / (2 |gamma|): with D = |d| + r,
// t = sgn(d) 2 |gamma| / D, c = 1 / sqrt(1 + t^2) = D / sqrt(D^2 + 4 |gamma|^2)
// = D / sqrt(2 r D), s e = t c gamma / |gamma| = sgn(d) 2 c gamma / D and
// t |gamma| = sgn(d) 2 |gamma|^2 / D (sgn(0) = +1).  Nothing cancels (|d| and
// r are both >= 0), and only two reciprocal square roots and a reciprocal
// are needed, the last two independent of each other: a shorter dependent
// chain than through zeta.
template <typename T>
__device__ __forceinline__ PRot prot_params(double al, double be, double gr, double gi, double g2) {
    constexpr int NS = sizeof(T) == 4 ? 1 : 2;
    PRot r;
    const double d = be - al;
    const double q = d * d + 4.0 * g2;
    const double rq = q * prsqrt<NS>(q);
    const double D = fabs(d) + rq;
    const double iD = prcp(D);
    r.c = D * prsqrt<NS>(2.0 * rq * D);
    const double f = (d >= 0.0 ? 2.0 : -2.0) * iD;
    r.a = f * r.c * gr;
    r.b = f * r.c * gi;
    r.tg = f * g2;
    r.on = true;
    return r;
}

template <typename T>
__device__ __forceinline__ PRot prot(double al, double be, double gr, double gi, double tol) {
    const double g2 = gr * gr + gi * gi;
    if (!prot_needed<T>(al, be, g2, tol)) return PRot{1.0, 0.0, 0.0, 0.0, false};
    return prot_params<T>(al, be, gr, gi, g2);
}

// Sums over the first ka row groups (the slice rows; the V rows below them
// take part in the rotations only), as chains of fused multiply-adds.  ka is
// a runtime value, at least kMinSliceGroups(RPT) (m >= n and RPT is at most
// the next instance above the row groups needed): the groups up to there are
// summed without a test, each one above behind a uniform branch.
__host__ __device__ constexpr int kMinSliceGroups(int rpt) { return rpt > 17 ? 9 : (rpt + 1) / 2; }

template <typename T, int RPT, int K>
__device__ __forceinline__ void dot_above(const cplx<T> (&x)[RPT], const cplx<T> (&y)[RPT], int ka, T& gr, T& gi) {
    if constexpr (K < RPT - 1) {
        if (K < ka) {
            gr = fma(x[K].re, y[K].re, gr);
            gr = fma(x[K].im, y[K].im, gr);
            gi = fma(x[K].re, y[K].im, gi);
            gi = fma(-x[K].im, y[K].re, gi);
            dot_above<T, RPT, K + 1>(x, y, ka, gr, gi);
        }
    }
}

template <typename T, int RPT>
__device__ __forceinline__ void dot_rows(const cplx<T> (&x)[RPT], const cplx<T> (&y)[RPT], int ka, T& gr, T& gi) {
    constexpr int K0 = kMinSliceGroups(RPT);
#pragma unroll
    for (int k = 0; k < K0; ++k) {
        gr = fma(x[k].re, y[k].re, gr);
        gr = fma(x[k].im, y[k].im, gr);
        gi = fma(x[k].re, y[k].im, gi);
        gi = fma(-x[k].im, y[k].re, gi);
    }
    dot_above<T, RPT, K0>(x, y, ka, gr, gi);
}

template <typename T, int RPT, int K>
__device__ __forceinline__ void norm_above(const cplx<T> (&x)[RPT], int ka, T& acc) {
    if constexpr (K < RPT - 1) {
        if (K < ka) {
            acc += x[K].re * x[K].re + x[K].im * x[K].im;
            norm_above<T, RPT, K + 1>(x, ka, acc);
        }
    }
}

template <typename T, int RPT>
__device__ __forceinline__ T norm_rows(const cplx<T> (&x)[RPT], int ka) {
    constexpr int K0 = kMinSliceGroups(RPT);
    T acc = 0;
#pragma unroll
    for (int k = 0; k < K0; ++k) acc += x[k].re * x[k].re + x[k].im * x[k].im;
    norm_above<T, RPT, K0>(x, ka, acc);
    return acc;
}

// Squared norm of the slice rows of a column held in registers (group sum
// in the element type, returned in FP64).
template <typename T, int PG, int RPT>
__device__ __forceinline__ double pnorm2(const cplx<T> (&x)[RPT], int ka) {
    const T acc = norm_rows<T, RPT>(x, ka);
    return (double)group_sum<PG>(acc);
}

// Device-coherent FP64 store and load (the Frobenius parts of a slice).
__device__ __forceinline__ void coh_store_f64(double* dst, double v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst), (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double coh_load_f64(const double* src) {
    return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(src),
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// The part of a slice's squared Frobenius norm (slice rows) held by a
// workgroup's block pair (widths w0 and w1; block 0 in registers, one column
// per pair group, block 1 in LDS): per column slot g the squared norms of the
// two blocks' columns g, added over g in order.  Every thread returns the
// same value.  The Jacobi variants add the parts of a slice's block pairs of
// round 0 in pair order, so all of them derive the same rounding floor bit
// for bit.  Slots past a block's width are not counted (they may hold an
// earlier block's column).  scratch: BW doubles of LDS.
template <typename T, int PG, int RPT, int BW>
__device__ __forceinline__ double pair_fro_part(const cplx<T> (&x)[RPT], const cplx<T>* blk1, int w0, int w1,
                                                int ldc, int ka, double* scratch) {
    const int g = threadIdx.x / PG, l = threadIdx.x - g * PG;
    cplx<T> c1[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) c1[k] = blk1[g * ldc + l + PG * k];
    const double n0 = pnorm2<T, PG, RPT>(x, ka), n1 = pnorm2<T, PG, RPT>(c1, ka);
    const double part = (g < w0 ? n0 : 0.0) + (g < w1 ? n1 : 0.0);
    if (l == 0) scratch[g] = part;
    __syncthreads();
    double sum = 0.0;
    for (int i = 0; i < BW; ++i) sum += scratch[i];
    __syncthreads();
    return sum;
}

// Orthogonalise column x (registers) against column y in LDS.  Lane l of
// the pair group holds rows l + PG k; the first ka row groups (1 <= ka < RPT)
// are slice rows, the rest V rows, padding rows are zero; only the slice rows
// take part in the test.  al and be are the squared norms of the slice rows,
// exact at the start of a round (or internal level) and tracked through it:
// on a rotation they are updated in place (al -= t|gamma|, be += t|gamma|).
// Returns 0 (not rotated), 1 (rotated) or 2 (rotated, and the rotation
// forces another sweep: rot_forces_sweep with the rounding floor floor2).
template <typename T, int PG, int RPT>
__device__ __forceinline__ unsigned ppair(cplx<T> (&x)[RPT], cplx<T>* y_lds, double& al, double& be, int ka,
                                          int l, double tol, double floor2 = 0.0) {
    cplx<T> y[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) y[k] = y_lds[l + PG * k];
    T gr = 0, gi = 0;
    dot_rows<T, RPT>(x, y, ka, gr, gi);
    group_sum2<PG>(gr, gi);
    const double dgr = (double)gr, dgi = (double)gi;
    const PRot rt = prot<T>(al, be, dgr, dgi, tol);
    if (!rt.on) return 0u;
    const unsigned code = rot_forces_sweep(al, be, dgr * dgr + dgi * dgi, tol, floor2) ? 2u : 1u;
    // y <- s e x + c y, then x <- c x - s conj(e) y in place (s e = a + i b):
    // the new y is formed and stored while the old x is still there, so the
    // loop-carried x needs no copies
    {
        const T c = (T)rt.c, a = (T)rt.a, b = (T)rt.b;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const cplx<T> yn{c * y[k].re + a * x[k].re - b * x[k].im, c * y[k].im + a * x[k].im + b * x[k].re};
            y_lds[l + PG * k] = yn;
            x[k].re = c * x[k].re - a * y[k].re - b * y[k].im;
            x[k].im = c * x[k].im - a * y[k].im + b * y[k].re;
        }
    }
    al -= rt.tg;
    be += rt.tg;
    return code;
}

// The workgroups of a slice meet: 0 if the bounded wait ran out or another
// workgroup gave up, 1 if all met and one of them voted (*vote, in LDS), 2 if
// none did.  The blocks travel with device-coherent transfers, so no L2
// write-back or invalidation is needed: every wave waits until its own stores
// are complete at the coherence point, the workgroup meets, and thread 0 counts
// the arrival (low half of the word) together with the vote (high half) and
// waits for the others.  seen: the word at the last meeting (thread 0's); none
// can arrive at the next one before all have left this one, since a sweep
// needs every workgroup's blocks.  (Votes in a flag of their own, set before
// and read after the meeting, cost two more
// round trips: 0.8% of a video completion in FP32, 0.5% in FP64.)
__device__ __forceinline__ int slice_meet(int* word, int G, const int* vote, unsigned& seen, int* err, int spin_limit) {
    __shared__ int met;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(word, vote && *vote ? 0x10001 : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int spins = 0;
        met = 0;
        for (;;) {
            const unsigned v = (unsigned)__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (((v - seen) & 0xffff) >= (unsigned)G) {
                met = (v ^ seen) >> 16 ? 1 : 2;
                seen = v;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
            if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || ++spins > spin_limit) {
                __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
    }
    __syncthreads();
    return met;
}

// Cross steps wave to wave: a wave finishes step st + 1 only after its
// successor wave (cyclically) has finished step st, whose column it reads
// next; each wave counts its finished steps in LDS (release after its LDS
// writes, acquire before its reads).  Every wave of the ring runs every step of
// a round, so the waits end; the bound only guards against a fault.  Waves
// without columns (a block of 12 columns fills six of eight waves) are not in
// the ring of the cross steps: none waits for them there, and a count that
// stayed behind is waited on again only after its wave has published steps of
// a later round, whose numbers start from the same `steps` in every wave.
__device__ __forceinline__ void ring_publish(int* cnt, int value) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(cnt, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void ring_wait(const int* cnt, int value) {
    for (int spins = 0; spins < (1 << 20); ++spins)
        if (__hip_atomic_load(cnt, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= value) return;
}

// Waves per SIMD to compile a kernel of BW pair groups of PG lanes for: as
// many workgroups as the LDS of a CU (160 KB) holds blocks, up to four waves
// (128 registers a lane, enough for the FP32 columns and the narrower FP64
// ones; wider FP64 columns fill the LDS alone).
template <typename T, int PG, int BW, int RPT>
constexpr int jacobi_waves_per_simd() {
    constexpr int lds = BW * (PG * RPT + 1) * 2 * (int)sizeof(T) + 1024;
    constexpr int per_cu = 160 * 1024 / lds, waves = per_cu * BW * PG / 256;
    return waves < 1 ? 1 : (waves > 4 ? 4 : waves);
}

// One round of the block tournament on one block pair of a slice.  Block 0
// lives in registers (pair group g holds its column g in x for as long as the
// block stays with the workgroup), block 1 in LDS, so a pair of blocks takes
// half the LDS it would with both resident there and two workgroups share a
// CU for slices up to 19 row groups in FP32 (9 in FP64).  Measured against
// both blocks in LDS, results bit for bit the same: 256 x 256 x 64 RPCA (264
// block pairs on 256 CUs) 3.76 -> 2.77 ms an iteration in FP32; video
// completion (128 x 160 x 64) 1.39 -> 1.15 ms in FP64 and 0.407 -> 0.386 ms in
// FP32, where the blocks' round trips between rounds lose the LDS hop.
//
// First round of a sweep (self_phase): the internal pairs of both blocks by
// halving -- the cross pairs of a block's two halves, then of the halves of
// each half, down to adjacent pairs: BW - 1 steps, every pair once.  The
// groups below BW / 2 work on block 0, the others on block 1; at level k a
// group keeps its column of the first half of its subproblem in x and meets
// the k columns of the second half, which sit in the LDS slots of the
// subproblem's groups.  Between levels the groups of a subproblem's second
// half exchange their column with the slot that starts their own subproblem
// (a group reads and writes one slot, so only barriers separate the levels),
// and after the last level the exchanges are undone in reverse order.
//
// Then every cross pair: at step st group g meets column g + st of block 1
// (cyclically over the wider block's columns), which group g + 1 met at step
// st - 1.
//
// Norms are exact at the start of the round (and of every level) and tracked
// through it.  Each level and the cross steps run wave to wave: a wave waits
// only for the wave whose previous step wrote the column it takes next
// (wait(count, value), the counts in wsteps never reset: steps holds the
// number every wave has passed).  Returns the rotations applied (per thread:
// every lane of a pair group counts its group's) and adds those that force
// another sweep to nbig.
template <typename T, int PG, int RPT>
__device__ __forceinline__ void swap_slot(cplx<T> (&x)[RPT], cplx<T>* slot, int l) {
    cplx<T> y[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) y[r] = slot[l + PG * r];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        slot[l + PG * r] = x[r];
        x[r] = y[r];
    }
}

template <typename T, int PG, int BW, int RPT, typename Wait>
__device__ __forceinline__ unsigned pair_round(cplx<T> (&x)[RPT], cplx<T>* blk1, int wi, int wj, bool self_phase,
                                               int ka, int ldc, double tol, double floor2, double* jnorm,
                                               int* wsteps, int& steps, unsigned& nbig, Wait&& wait) {
    const int g = threadIdx.x / PG, l = threadIdx.x - g * PG;
    const int wave = threadIdx.x >> 6;
    unsigned nrot = 0;
    if (self_phase) {
        const bool second = g >= BW / 2;
        const int gi = second ? g - BW / 2 : g;
        cplx<T>* const base = blk1 + (second ? (BW / 2) * ldc : 0);   // the block's second-half slots
        double* const jn = jnorm + (second ? BW / 2 : 0);
        const int w = second ? wj : wi;
        // block 0's upper half to LDS, block 1's lower half to registers
        if (second) swap_slot<T, PG, RPT>(x, blk1 + gi * ldc, l);
        __syncthreads();
        for (int k = BW / 2; k >= 1; k /= 2) {
            const int sp = gi / k, q = gi - sp * k;
            const int xcol = 2 * k * sp + q, ycol0 = 2 * k * sp + k;
            // a subproblem of k groups spans k / 2 consecutive waves (one if k <= 2)
            const int span = k * PG >= 128 ? k * PG / 64 : 1, wl = wave % span;
            const int wnext = wave - wl + (wl + 1) % span;
            double ax = pnorm2<T, PG, RPT>(x, ka);
            {
                cplx<T> yr[RPT];
#pragma unroll
                for (int r = 0; r < RPT; ++r) yr[r] = base[gi * ldc + l + PG * r];
                const double bq = pnorm2<T, PG, RPT>(yr, ka);
                if (l == 0) jn[gi] = bq;
            }
            __syncthreads();
            for (int st = 0; st < k; ++st) {
                if (st > 0) wait(wsteps + wnext, steps + st);
                const int yo = (q + st) & (k - 1), ys = k * sp + yo;
                if (xcol < w && ycol0 + yo < w) {
                    double be = jn[ys];
                    if (const unsigned code = ppair<T, PG, RPT>(x, base + ys * ldc, ax, be, ka, l, tol, floor2)) {
                        ++nrot;
                        nbig += code >> 1;
                        if (l == 0) jn[ys] = be;
                    }
                }
                ring_publish(wsteps + wave, steps + st + 1);
            }
            steps += k;
            __syncthreads();
            if (k > 1) {
                if (q >= k / 2) swap_slot<T, PG, RPT>(x, base + (k * sp + q - k / 2) * ldc, l);
                __syncthreads();
            }
        }
        for (int k = 2; k <= BW / 2; k *= 2) {
            const int sp = gi / k, q = gi - sp * k;
            if (q >= k / 2) swap_slot<T, PG, RPT>(x, base + (k * sp + q - k / 2) * ldc, l);
            __syncthreads();
        }
        if (second) swap_slot<T, PG, RPT>(x, blk1 + gi * ldc, l);
        __syncthreads();
    }
    // the ring closes over the columns there are, so that narrower blocks (the
    // blocks of a slice have equal widths, give or take one) take fewer steps.
    // Against BW steps always: 72 x 128 x 80 FP64 RPCA (12 columns) 555 -> 525
    // us an iteration, a batch of uneven FP32 completions 367 -> 346 ms
    const int width = __builtin_amdgcn_readfirstlane(wi > wj ? wi : wj);
    const int nw = (width * PG + 63) / 64;   // waves with columns
    const int wave_next = wave + 1 < nw ? wave + 1 : 0;
    double al = pnorm2<T, PG, RPT>(x, ka);
    {
        cplx<T> yj[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) yj[k] = blk1[g * ldc + l + PG * k];
        const double bj = pnorm2<T, PG, RPT>(yj, ka);
        if (l == 0) jnorm[g] = bj;
    }
    __syncthreads();
    if (wave < nw) {
        for (int st = 0; st < width; ++st) {
            if (st > 0) wait(wsteps + wave_next, steps + st);
            const int jc = g + st < width ? g + st : g + st - width;
            if (g < wi && jc < wj) {
                double be = jnorm[jc];
                if (const unsigned code = ppair<T, PG, RPT>(x, blk1 + jc * ldc, al, be, ka, l, tol, floor2)) {
                    ++nrot;
                    nbig += code >> 1;
                    if (l == 0) jnorm[jc] = be;
                }
            }
            ring_publish(wsteps + wave, steps + st + 1);
        }
    }
    steps += width;
    __syncthreads();
    return nrot;
}

// Stacked column of a block: slice rows 0..m-1 at 0..m-1, V rows at
// mp..mp+n-1 (mp = m rounded up to PG), zeros elsewhere; pair group c holds or
// moves column c, lane t the rows t + PG r, so a row group is either slice
// rows or V rows.
//
// Columns move through buffer resources of the slice's two matrices: an
// address per lane takes one register, and padding rows and columns past the
// block's width get an address past the end, where a load returns zeros and a
// store does nothing, so there are no branches and every load of an exchange
// is in flight at once.  COH: device-coherent transfers (sc1, what an
// agent-scope relaxed atomic uses), served at the device's coherence point
// and never from a stale L2 line of another XCD, so workgroups that exchange
// blocks through global memory inside one launch need no L2 write-back or
// invalidation around the exchange.
template <typename T>
struct SliceView {
    __amdgpu_buffer_rsrc_t A;   // m x n, column-major
    __amdgpu_buffer_rsrc_t V;   // n x n, column-major
    int m, n, nb, ka, ldc;
};

template <typename T>
__device__ __forceinline__ SliceView<T> slice_view(cplx<T>* A, cplx<T>* V, int m, int n, int nb, int ka, int ldc) {
    constexpr int kRaw = 0x00027000;   // raw buffer, 32-bit data format
    return {__builtin_amdgcn_make_buffer_rsrc(A, 0, m * n * (int)sizeof(cplx<T>), kRaw),
            __builtin_amdgcn_make_buffer_rsrc(V, 0, n * n * (int)sizeof(cplx<T>), kRaw), m, n, nb, ka, ldc};
}

template <typename T>
struct BufWord;
template <>
struct BufWord<float> {
    using type = unsigned __attribute__((ext_vector_type(2)));
    template <int AUX>
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t b, int off) {
        return __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, AUX);
    }
    template <int AUX>
    static __device__ __forceinline__ void store(type v, __amdgpu_buffer_rsrc_t b, int off) {
        __builtin_amdgcn_raw_buffer_store_b64(v, b, off, 0, AUX);
    }
};
template <>
struct BufWord<double> {
    using type = unsigned __attribute__((ext_vector_type(4)));
    template <int AUX>
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t b, int off) {
        return __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, AUX);
    }
    template <int AUX>
    static __device__ __forceinline__ void store(type v, __amdgpu_buffer_rsrc_t b, int off) {
        __builtin_amdgcn_raw_buffer_store_b128(v, b, off, 0, AUX);
    }
};

// Byte offset of row `row` (of `len`) of a column that starts at element
// `start` (-1: no column); past the end of every slice when it does not exist.
template <typename T>
__device__ __forceinline__ int elem_offset(int start, int row, int len) {
    return start >= 0 && row < len ? (start + row) * (int)sizeof(cplx<T>) : -16;
}

// The column of block blk that pair group c takes, -1 past the block's width.
template <typename T>
__device__ __forceinline__ int block_col(const SliceView<T>& s, int blk, int c) {
    const int c0 = pblk_start(blk, s.n, s.nb);
    return c < pblk_start(blk + 1, s.n, s.nb) - c0 ? c0 + c : -1;
}

// The value, of unknown origin to the compiler: keeps the row tests and
// offsets of a transfer (two per row group) from being computed once and held
// in registers through the sweeps.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

template <typename T, int PG, int RPT, bool COH>
__device__ __forceinline__ void load_col(const SliceView<T>& s, int blk, cplx<T> (&x)[RPT]) {
    const int c = threadIdx.x / PG, t = opaque(threadIdx.x - c * PG);
    const int ka = __builtin_amdgcn_readfirstlane(opaque(s.ka));
    const int col = block_col(s, blk, c);
    const int sa = col < 0 ? -1 : col * s.m, sv = col < 0 ? -1 : col * s.n;
#pragma unroll
    for (int r = 0; r < RPT; ++r)
        x[r] = __builtin_bit_cast(
            cplx<T>, r < ka ? BufWord<T>::template load<COH ? 16 : 0>(s.A, elem_offset<T>(sa, t + PG * r, s.m))
                              : BufWord<T>::template load<COH ? 16 : 0>(
                                    s.V, elem_offset<T>(sv, t + PG * (r - ka), s.n)));
}

template <typename T, int PG, int RPT, bool COH>
__device__ __forceinline__ void store_col(const SliceView<T>& s, int blk, const cplx<T> (&x)[RPT]) {
    const int c = threadIdx.x / PG, t = opaque(threadIdx.x - c * PG);
    const int ka = __builtin_amdgcn_readfirstlane(opaque(s.ka));
    const int col = block_col(s, blk, c);
    const int sa = col < 0 ? -1 : col * s.m, sv = col < 0 ? -1 : col * s.n;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const auto w = __builtin_bit_cast(typename BufWord<T>::type, x[r]);
        if (r < ka)
            BufWord<T>::template store<COH ? 16 : 0>(w, s.A, elem_offset<T>(sa, t + PG * r, s.m));
        else
            BufWord<T>::template store<COH ? 16 : 0>(w, s.V, elem_offset<T>(sv, t + PG * (r - ka), s.n));
    }
}

template <typename T, int PG, int RPT, bool COH>
__device__ __forceinline__ void store_lds(const SliceView<T>& s, int blk, const cplx<T>* lds) {
    const int c = threadIdx.x / PG, t = threadIdx.x - c * PG;
    cplx<T> y[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) y[r] = lds[c * s.ldc + t + PG * r];
    store_col<T, PG, RPT, COH>(s, blk, y);
}

// The blocks blk0 (into registers) and blk1 (into LDS), -1: keep; all loads of
// both in flight together.
template <typename T, int PG, int RPT, bool COH>
__device__ __forceinline__ void load_pair(const SliceView<T>& s, int blk0, cplx<T> (&x)[RPT], int blk1,
                                          cplx<T>* lds) {
    const int c = threadIdx.x / PG, t = threadIdx.x - c * PG;
    cplx<T> y[RPT];
    if (blk1 >= 0) load_col<T, PG, RPT, COH>(s, blk1, y);
    if (blk0 >= 0) load_col<T, PG, RPT, COH>(s, blk0, x);
    if (blk1 >= 0) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) lds[c * s.ldc + t + PG * r] = y[r];
    }
}

}  // namespace jac
}  // namespace tsvd
