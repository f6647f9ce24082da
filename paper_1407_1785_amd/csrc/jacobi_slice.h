// One-sided Jacobi SVD with one workgroup per Fourier slice, for batches of
// many problems (same rotation, block round-robin ordering and stopping
// rule as jacobi.hip and jacobi_persist.hip).
//
// A batch of uneven problems has thousands of slices, many more than the
// chip has CUs, so every slice gets a single workgroup and no workgroup
// ever waits for another.  The workgroup runs all sweeps of its slice: in
// every round of the block tournament it visits the round's nb/2 block
// pairs one after the other, each time loading the two blocks (stacked
// columns: m slice rows, then n rows of V; one into registers, one into LDS),
// orthogonalising them against each other (and, in the first round of a
// sweep, internally) and writing them back.  With nb = 2 the two blocks stay
// in registers and LDS for the whole SVD.  The slice stops after a sweep none of whose
// rotations forces another (rot_forces_sweep), or after max_sweeps.
//
// Work split as in jacobi_persist.hip: a column pair per group of PG = 32
// lanes, BW pairs per step (BW = 4, 8 or 16 columns per block: the block
// width is chosen per problem so that a block of its stacked height fits in
// LDS), rotation parameters in FP64, norms exact at the start of a round
// and tracked through it.
//
// Pairs-parallel schedule (jacobi_pairs_kernel) for slices with many
// blocks: one workgroup per block pair of a round, so a large slice is worked
// on by nb/2 workgroups at once, all sweeps in one launch (the blocks travel
// between the workgroups through global memory inside the launch).
//
// Launch: a table of problems; workgroup b serves problem p when
// wg_start[p] <= b < wg_start[p + 1], slice b - wg_start[p].  A problem
// whose ADMM has stopped (ctrl->done) is skipped, and so is one whose
// optional only_if word is zero (the single-problem driver's fallback after
// a persistent launch that gave up, which also writes the singular values);
// each slice raises ctrl->sweep_max to its sweep count.

#pragma once

#include "jacobi_common.h"

#include <algorithm>

namespace tsvd {

namespace {

using namespace jac;

// All sweeps of slice s by this workgroup.
template <typename T, int BW, int RPT>
__device__ __forceinline__ void slice_svd(const JacSliceArgs<T>& a, int s, int max_sweeps) {
    constexpr int PG = kPGs, NT = BW * PG;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int rot_any;
    __shared__ double jnorm[BW];
    const int m = a.m, n = a.n, nb = a.nb, G = nb / 2;
    const int ka = (m + PG - 1) / PG;
    const int ldc = PG * RPT + 1;   // one more than the column: a wave's groups read different LDS banks
    const SliceView<T> sv = slice_view(a.A + (int64_t)s * n * m, a.V + (int64_t)s * n * n, m, n, nb, ka, ldc);
    cplx<T>* const blk1 = reinterpret_cast<cplx<T>*>(smem);
    cplx<T> x[RPT];
    const int l = threadIdx.x % PG;
    const double tol = (double)a.tol;
    auto width = [&](int b) { return pblk_start(b + 1, n, nb) - pblk_start(b, n, nb); };

    __shared__ int wsteps[NT / 64];
    int steps = 0;
    if ((threadIdx.x & 63) == 0) wsteps[threadIdx.x >> 6] = 0;
    if (G == 1) load_pair<T, PG, RPT, false>(sv, 0, x, 1, blk1);
    // rounding floor of the stopping rule: the parts of the round-0 block
    // pairs in pair order (as the pairs-parallel and persistent kernels add them)
    double floor2 = 0.0;
    if (a.floor_scale > 0.0) {
        double fro2 = 0.0;
        for (int gp = 0; gp < G; ++gp) {
            const int p0 = ppos_player(gp, 0, nb), p1 = ppos_player(nb - 1 - gp, 0, nb);
            if (G > 1) load_pair<T, PG, RPT, false>(sv, p0, x, p1, blk1);
            __syncthreads();
            fro2 += pair_fro_part<T, PG, RPT, BW>(x, blk1, width(p0), width(p1), ldc, ka, jnorm);
        }
        floor2 = a.floor_scale * fro2;
    }

    unsigned nrot = 0;
    int sweeps = 0;
    const int msw = a.max_sweeps > 0 ? a.max_sweeps : max_sweeps;
    for (int sweep = 0; sweep < msw; ++sweep) {
        if (threadIdx.x == 0) rot_any = 0;
        unsigned nrot_sweep = 0, nbig_sweep = 0;
        for (int rd = 0; rd < nb - 1; ++rd) {
            for (int gp = 0; gp < G; ++gp) {
                const int pos0 = ppos_slot0(gp, sweep * (nb - 1) + rd);
                const int player0 = ppos_player(pos0, rd, nb), player1 = ppos_player(nb - 1 - pos0, rd, nb);
                // (the round's own barriers end every use of the blocks it leaves behind)
                if (G > 1) load_pair<T, PG, RPT, false>(sv, player0, x, player1, blk1);
                __syncthreads();
                nrot_sweep += pair_round<T, PG, BW, RPT>(x, blk1, width(player0), width(player1), rd == 0, ka, ldc,
                                                         tol, floor2, jnorm, wsteps, steps, nbig_sweep, ring_wait);
                if (G > 1) {
                    store_col<T, PG, RPT, false>(sv, player0, x);
                    store_lds<T, PG, RPT, false>(sv, player1, blk1);
                    __syncthreads();
                }
            }
        }
        if (nbig_sweep && l == 0) rot_any = 1;
        __syncthreads();
        nrot += nrot_sweep;
        sweeps = sweep + 1;
        if (!rot_any) break;
        __syncthreads();
    }
    if (G == 1) {
        store_col<T, PG, RPT, false>(sv, 0, x);
        store_lds<T, PG, RPT, false>(sv, 1, blk1);
    }
    if (threadIdx.x == 0) {
        if (a.sweeps) a.sweeps[s] = sweeps;
        if (a.ctrl) atomicMax(&a.ctrl->sweep_max, sweeps);
    }
    if (l == 0 && nrot && a.rotations) atomicAdd(a.rotations, (unsigned long long)nrot);
}

template <typename T, int BW, int RPT>
__global__ __launch_bounds__(BW * kPGs, (jacobi_waves_per_simd<T, kPGs, BW, RPT>()))
void jacobi_slice_kernel(const JacSliceArgs<T>* tab, const int* wg_start, int nprob, int max_sweeps) {
    const int p = batch_find(wg_start, nprob, (int)blockIdx.x);
    const JacSliceArgs<T>& a = tab[p];
    if (a.ctrl && a.ctrl->done) return;
    const int idx = (int)blockIdx.x - wg_start[p];
    const bool run = !a.only_if || *a.only_if != 0;
    if (!a.sigma) {
        if (run) slice_svd<T, BW, RPT>(a, idx, max_sweeps);
        return;
    }
    // The last launch of a single problem's SVD: the sweeps are over unless
    // the launch that ran them gave up, and what is left is to write the
    // singular values and clear the words for the next SVD.  `parts`
    // workgroups share a slice's columns; a slice whose sweeps are still to be
    // run is one workgroup's.
    // (A gated fallback, svt_sigma and a launch that clears the words are
    // 4.5 us each; 32 x 32 x 16 FP64 completion 148 -> 144 us an iteration,
    // larger shapes the same.)
    const int s = idx / a.parts, part = idx - s * a.parts;
    if (run) {
        if (part != 0) return;
        slice_svd<T, BW, RPT>(a, s, max_sweeps);
        __syncthreads();
    }
    constexpr int NW = BW * kPGs / 64;
    const int wave = threadIdx.x >> 6;
    const cplx<T>* const W = a.A + (int64_t)s * a.n * a.m;
    for (int j = (run ? 0 : part * NW) + wave; j < a.n; j += run ? NW : a.parts * NW)
        sigma_column(W + (int64_t)j * a.m, a.m, a.ctrl->tau, a.sigma + (int64_t)s * a.n + j,
                     a.dk + (int64_t)s * a.n + j);
    if (part == 0)
        for (int i = s * BW * kPGs + threadIdx.x; i < a.nclr; i += a.h * BW * kPGs)
            if (a.clr + i != a.only_if) a.clr[i] = 0;
}

// Pairs-parallel schedule: nb / 2 workgroups per slice, one per block pair
// of a round, all sweeps in one launch.  Workgroup roles (problem, slice,
// block pair) come in order from words[0], as in jacobi_persist.hip, so the
// workgroups of a slice wait only for workgroups that run or start as soon as
// others finish; between rounds a workgroup writes the block that moves on
// (ppos_slot0) to its home columns with device-coherent stores, sets its ready
// flag to the round that takes it next and waits for the flag of the block it
// takes next; at the end of a sweep the slice's workgroups meet (slice_meet)
// and stop together
// when no rotation of the sweep forces another.  Every wait between
// workgroups is bounded (spin_limit polls); one that gives up sets words[1],
// and every workgroup that meets it writes its resident blocks home and
// stops.  The rotations, their order and the stopping rule are those of the
// one-workgroup-per-slice kernel (pair_round per block pair and round), so
// both schedules give the same results bit for bit.
__device__ bool pairs_wait_flag(int* flag, int value, int* err, int spin_limit) {
    int spins = 0;
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < value) {
        __builtin_amdgcn_s_sleep(1);
        if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || ++spins > spin_limit) {
            __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
    }
    return true;
}

template <typename T, int BW, int RPT>
__global__ __launch_bounds__(BW * kPGs, (jacobi_waves_per_simd<T, kPGs, BW, RPT>())) void jacobi_pairs_kernel(const JacSliceArgs<T>* tab, const int* role_start,
                                                                  int nprob, int* words, int spin_limit) {
    constexpr int PG = kPGs, NT = BW * PG;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int role_s, rot_any, ok_flag;
    __shared__ double jnorm[BW];
    if (threadIdx.x == 0) role_s = __hip_atomic_fetch_add(words, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int role = __builtin_amdgcn_readfirstlane(role_s);
    const int p = batch_find(role_start, nprob, role);
    const JacSliceArgs<T>& a = tab[p];
    if (a.ctrl && a.ctrl->done) return;   // every workgroup of the problem returns
    const int m = a.m, n = a.n, nb = a.nb, G = nb / 2, h = a.h;
    const int local = role - role_start[p];
    const int s = local / G, gp = local - s * G;
    int* const counter = a.bar + s;
    int* const bf = a.bar + h + (int64_t)s * nb;
    int* const err = words + 1;
    const int ka = (m + PG - 1) / PG;
    const int ldc = PG * RPT + 1;   // one more than the column: a wave's groups read different LDS banks
    const SliceView<T> sv = slice_view(a.A + (int64_t)s * n * m, a.V + (int64_t)s * n * n, m, n, nb, ka, ldc);
    cplx<T>* const blk1 = reinterpret_cast<cplx<T>*>(smem);
    cplx<T> x[RPT];
    const int l = threadIdx.x % PG;
    const double tol = (double)a.tol;
    const int msw = a.max_sweeps > 0 ? a.max_sweeps : 30;
    auto width = [&](int b) { return pblk_start(b + 1, n, nb) - pblk_start(b, n, nb); };

    __shared__ int wsteps[NT / 64];
    int steps = 0;
    if ((threadIdx.x & 63) == 0) wsteps[threadIdx.x >> 6] = 0;
    int player0 = ppos_player(gp, 0, nb), player1 = ppos_player(nb - 1 - gp, 0, nb);
    load_pair<T, PG, RPT, true>(sv, player0, x, player1, blk1);
    __syncthreads();

    unsigned nrot = 0;
    int sweeps = 0;
    unsigned seen = 0;   // the barrier word at the last meeting (thread 0's)
    bool alive = true, home0 = true, home1 = true;
    // rounding floor of the stopping rule: every workgroup writes the part of
    // its round-0 block pair, the slice's workgroups meet once, and each adds
    // the parts in pair order (as the one-workgroup-per-slice kernel does)
    double floor2 = 0.0;
    if (a.floor_scale > 0.0) {
        __shared__ double fro_s;
        const double part =
            pair_fro_part<T, PG, RPT, BW>(x, blk1, width(player0), width(player1), ldc, ka, jnorm);
        if (threadIdx.x == 0) coh_store_f64(a.fro + (int64_t)s * G + gp, part);
        if (!slice_meet(counter, G, nullptr, seen, err, spin_limit)) {
            alive = false;   // giving up before any rotation: both blocks are still home
        } else {
            if (threadIdx.x == 0) {
                double fro2 = 0.0;
                for (int i = 0; i < G; ++i) fro2 += coh_load_f64(a.fro + (int64_t)s * G + i);
                fro_s = a.floor_scale * fro2;
            }
            __syncthreads();
            floor2 = fro_s;
        }
    }
    for (int sweep = 0; sweep < msw && alive; ++sweep) {
        if (threadIdx.x == 0) rot_any = 0;
        sweeps = sweep + 1;
        __syncthreads();
        unsigned nbig = 0;
        for (int rd = 0; rd < nb - 1; ++rd) {
            nrot += pair_round<T, PG, BW, RPT>(x, blk1, width(player0), width(player1), rd == 0, ka, ldc, tol, floor2,
                                               jnorm, wsteps, steps, nbig, ring_wait);
            const bool last = rd == nb - 2;
            if (last && nbig && l == 0) rot_any = 1;   // this workgroup needs another sweep
            // the next round's players (after the last round: round 0 of the next sweep)
            const int nr = (rd + 1) % (nb - 1);
            const int R = sweep * (nb - 1) + rd;
            const int pos0 = ppos_slot0(gp, R + 1);
            const int next0 = ppos_player(pos0, nr, nb), next1 = ppos_player(nb - 1 - pos0, nr, nb);
            if (next0 != player0) store_col<T, PG, RPT, true>(sv, player0, x);
            if (next1 != player1) store_lds<T, PG, RPT, true>(sv, player1, blk1);
            if (last) {
                if (slice_meet(counter, G, &rot_any, seen, err, spin_limit) != 1) {
                    home0 = next0 == player0;   // giving up, or converged
                    home1 = next1 == player1;
                    alive = false;
                    break;
                }
            } else {
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                if (threadIdx.x == 0) {
                    ok_flag = 1;
                    if (next0 != player0) __hip_atomic_store(bf + player0, R + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (next1 != player1) __hip_atomic_store(bf + player1, R + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((next0 != player0 && !pairs_wait_flag(bf + next0, R + 1, err, spin_limit)) ||
                        (next1 != player1 && !pairs_wait_flag(bf + next1, R + 1, err, spin_limit)))
                        ok_flag = 0;
                }
                __syncthreads();
                if (!ok_flag) {
                    home0 = next0 == player0;   // giving up
                    home1 = next1 == player1;
                    alive = false;
                    break;
                }
            }
            load_pair<T, PG, RPT, true>(sv, next0 != player0 ? next0 : -1, x, next1 != player1 ? next1 : -1, blk1);
            player0 = next0;
            player1 = next1;
            __syncthreads();
        }
    }
    __syncthreads();
    if (home0) store_col<T, PG, RPT, true>(sv, player0, x);
    if (home1) store_lds<T, PG, RPT, true>(sv, player1, blk1);
    if (threadIdx.x == 0) {
        if (gp == 0 && a.sweeps) a.sweeps[s] = sweeps;
        if (a.ctrl) atomicMax(&a.ctrl->sweep_max, sweeps);
    }
    if (l == 0 && nrot && a.rotations) atomicAdd(a.rotations, (unsigned long long)nrot);
}

}  // namespace

// PREPARE: set the LDS limit of both kernels.  SLICE: x = max_sweeps.
// PAIRS: words and x = spin_limit.
template <typename T, int BW, int RPT>
hipError_t slice_op_rpt(SliceOp op, const JacSliceArgs<T>* tab, const int* start, int nprob, int nwg, int* words, int x,
                        bool spread, hipStream_t st) {
    auto* fs = jacobi_slice_kernel<T, BW, RPT>;
    auto* fp = jacobi_pairs_kernel<T, BW, RPT>;
    const size_t own = jacobi_slice_lds(BW, RPT, sizeof(T));
    const size_t lds = op == SliceOp::PREPARE || spread ? std::max(own, kSpreadLds) : own;
    if (op == SliceOp::PREPARE) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fs),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        return hipFuncSetAttribute(reinterpret_cast<const void*>(fp), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds);
    }
    if (op == SliceOp::SLICE)
        hipLaunchKernelGGL(fs, dim3(nwg), dim3(BW * kPGs), lds, st, tab, start, nprob, x);
    else
        hipLaunchKernelGGL(fp, dim3(nwg), dim3(BW * kPGs), lds, st, tab, start, nprob, words, x);
    return hipGetLastError();
}

template <typename T, int BW, int... R>
hipError_t slice_op_seq(SliceOp op, int rpt, std::integer_sequence<int, R...>, const JacSliceArgs<T>* tab,
                        const int* start, int nprob, int nwg, int* words, int x, bool spread,
                        hipStream_t st) {
    hipError_t e = hipErrorInvalidValue;
    ((rpt == R + 2 ? (e = slice_op_rpt<T, BW, R + 2>(op, tab, start, nprob, nwg, words, x, spread, st), 0) : 0), ...);
    return e;
}

#define TSVD_SLICE_INSTANCE(T, BW)                                                                                   \
    template <>                                                                                                      \
    hipError_t slice_op<T, BW>(SliceOp op, int rpt, const JacSliceArgs<T>* tab, const int* start, int nprob, int nwg, \
                               int* words, int x, bool spread, hipStream_t st) {                                     \
        return slice_op_seq<T, BW>(op, rpt, std::make_integer_sequence<int, 19>{}, tab, start, nprob, nwg, words, x, \
                                   spread, st);                                                                      \
    }

}  // namespace tsvd
