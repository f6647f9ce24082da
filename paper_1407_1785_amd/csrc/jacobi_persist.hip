// Persistent one-sided Jacobi SVD: one launch runs every sweep
// of every Fourier slice (same method, ordering and stopping rule as the
// per-round kernels in jacobi.hip, which remain the path for shapes that do
// not fit this one).
//
// Layout.  Slice s gets G = nb/2 workgroups; a workgroup holds two BW-column
// blocks of stacked columns (m slice rows, then n rows of V), one in registers
// and one in LDS.  A round of the block tournament orthogonalises the two
// against each other; between rounds one of them stays and the other goes to
// another workgroup (ppos_slot0): the workgroup writes it back to its home
// columns in global memory, sets its ready flag, and waits for the one block it
// takes next.  The first round of every sweep also orthogonalises each block
// internally.  A slice of one
// block pair (n <= 32) shares no word with others and meets nobody: 32 x 32 x
// 16 FP64 completion 152 -> 148 us an iteration.
//
// Work split.  A column pair is handled by a group of PG = 32 lanes (two DPP
// rows), so a 512-thread workgroup (two waves per SIMD) works on BW = 16
// pairs per step; each lane holds rows lane + 32 k of its columns, the
// cross product is reduced with DPP and readlane, and the rotation
// parameters are computed per group in FP64.  Column norms are computed
// exactly at the start of every round and tracked through the rotations of
// the round (a rotation moves t |gamma| from one squared norm to the other).
//
// Synchronisation.  Blocks travel through global memory with device-
// coherent stores and loads.  Within a sweep, a workgroup that has written a
// block waits for the stores to complete and then sets the block's flag to
// the index of the round that takes it next; a workgroup waits only on the
// flag of the block it takes next.  At the end of a sweep all workgroups of
// the slice meet (slice_meet: the stopping decision needs every workgroup's
// vote).
//
// Residency.  A workgroup takes its role (slice, block pair) from a ticket
// counter when it starts, so the roles of the workgroups running at any time
// are the lowest ones not yet finished: the workgroups of a slice wait only
// for workgroups that are running or will start as soon as others finish.
// The grid holds at most one workgroup per CU, so on an otherwise idle
// device every workgroup is resident at once; under concurrent work the
// slices finish in ticket order.  Every wait between workgroups is bounded
// (PersistArgs.spin_limit polls): a wait that gives up sets bit 1 of the
// error word, and every workgroup that meets the error word at its next wait
// writes its resident blocks home and stops.  Each block is held by one workgroup at a
// time and every rotation is applied to the slice rows and the V rows
// together, so W = A V still holds for the partly rotated slices; the caller
// then finishes the SVD with the one-workgroup-per-slice kernel.
//
// Convergence: a workgroup votes for another sweep when a rotation of the
// sweep forces one (rot_forces_sweep); the vote travels with its arrival at the
// sweep's last barrier, and all workgroups of the slice stop together when
// there is none.  The rounding floor of that test needs the slice's Frobenius norm:
// each workgroup writes the part of its two starting blocks, and the
// workgroups of a slice meet once before the first sweep, after which every
// one adds the same parts in the same order.

#include "jacobi_common.h"

#include <algorithm>

namespace tsvd {

namespace {

using namespace jac;

constexpr int PBW = 16;   // columns per block = pairs per step

// Bounded wait (thread 0) until a block flag reaches `value`; false if the
// wait ran out or another workgroup gave up.
__device__ bool wait_flag(int* flag, int value, int* err, int spin_limit) {
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

// Cross steps of a round, wave to wave: wave w finishes step st + 1 only
// after reading what wave w + 1 (cyclically) wrote at step st, and nothing
// else.  Each wave counts its finished steps in LDS (release after its LDS
// writes); a wave waits for its successor's count (acquire) instead of a
// workgroup barrier, so a step costs the waves' average rather than the
// slowest pair.  Every wave of the ring runs every step of a round (giving up
// happens only between rounds; waves without columns are not in it), so a wait
// lasts at most a few steps.  One that runs far longer means a fault: the wave stops waiting
// and sets the error word to 2, which fails the call (the block data can no
// longer be trusted); it checks the error word every 1024 polls, so after
// such a fault no wait spins to its cap again.

// Polls back to back (a sleep between polls cost 0.7% of the iteration);
// 2^18 LDS polls are milliseconds, far beyond any step of a workgroup's own
// waves, and 1024 polls tens of microseconds, tens of steps.
constexpr int kLdsSpinLimit = 1 << 18;

__device__ __forceinline__ void lds_wait(const int* cnt, int value, int* err) {
    int spins = 0;
    while (__hip_atomic_load(cnt, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < value) {
        ++spins;
        if (spins > kLdsSpinLimit) {
            __hip_atomic_store(err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if ((spins & 1023) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            __hip_atomic_store(err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
    }
}

}  // namespace

template <typename T, int PG, int RPT>
__global__ __launch_bounds__(PBW * PG) void jacobi_persistent_kernel(JacArgs<T> a, PersistArgs p) {
    constexpr int NT = PBW * PG;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int rot_any;
    __shared__ int ok_flag;
    __shared__ double jnorm[PBW];
    __shared__ int wsteps[NT / 64];   // pair steps finished per wave, over the whole launch
    __shared__ int role;
    if (a.ctrl && a.ctrl->done) return;
    const int G = a.nb / 2;
    // the int words of the launch: h barrier words, the error word, the role ticket, h x nb block flags
    int* const err = p.pbar + a.h;
    if (threadIdx.x == 0) role = __hip_atomic_fetch_add(err + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // uniform across the workgroup: keep it (and what derives from it) scalar
    const int rl = __builtin_amdgcn_readfirstlane(role);
    const int s = rl / G, wg = rl - s * G;
    if (s >= a.h) return;
    const int ka = (a.m + PG - 1) / PG;   // row groups holding slice rows
    // column stride: the padded stacked column plus one element, so the pair
    // groups of a wavefront read different LDS banks
    const int ldc = PG * RPT + 1;
    const SliceView<T> sv =
        slice_view(a.A + (int64_t)s * a.n * a.m, a.V + (int64_t)s * a.n * a.n, a.m, a.n, a.nb, ka, ldc);
    cplx<T>* const blk1 = reinterpret_cast<cplx<T>*>(smem);
    cplx<T> x[RPT];
    const int l = threadIdx.x % PG;
    const double tol = (double)a.tol;
    int* counter = p.pbar + s;
    unsigned seen = 0;   // the barrier word at the last meeting (thread 0's)
    auto width = [&](int b) { return pblk_start(b + 1, a.n, a.nb) - pblk_start(b, a.n, a.nb); };
    auto wait = [&](const int* cnt, int value) { lds_wait(cnt, value, err); };

    if ((threadIdx.x & 63) == 0) wsteps[threadIdx.x >> 6] = 0;
    int steps = 0;   // pair steps finished by every wave before the current round
    int player0 = ppos_player(wg, 0, a.nb), player1 = ppos_player(a.nb - 1 - wg, 0, a.nb);
    load_pair<T, PG, RPT, true>(sv, player0, x, player1, blk1);
    if (wg == 0 && threadIdx.x == 0) a.sweeps[s] = 0;
    __syncthreads();

    unsigned nrot_total = 0;
    int swept = 0;   // sweeps started (kept by wg 0, thread 0)
    bool alive = true;
    // resident blocks still to be written home when the sweeps end: both at
    // the sweep cap; after a stop or a give-up, only those that did not move
    // (the moving ones were written before the exchange)
    bool home0 = true, home1 = true;
    double floor2 = 0.0;   // rounding floor of rot_forces_sweep
    if (p.floor_scale > 0.0) {
        const double part =
            pair_fro_part<T, PG, RPT, PBW>(x, blk1, width(player0), width(player1), ldc, ka, jnorm);
        if (G > 1) {
            if (threadIdx.x == 0) coh_store_f64(p.fro + (int64_t)s * G + wg, part);
            alive = slice_meet(counter, G, nullptr, seen, err, p.spin_limit) != 0;
        }
        if (G == 1) {
            floor2 = p.floor_scale * part;
        } else if (alive) {   // otherwise giving up before any rotation: both blocks are still home
            if (threadIdx.x == 0) {
                double fro2 = 0.0;
                for (int i = 0; i < G; ++i) fro2 += coh_load_f64(p.fro + (int64_t)s * G + i);
                jnorm[0] = p.floor_scale * fro2;
            }
            __syncthreads();
            floor2 = jnorm[0];
            __syncthreads();
        }
    }
    for (int sweep = 0; sweep < p.max_sweeps && alive; ++sweep) {
        if (threadIdx.x == 0) rot_any = 0;
        if (wg == 0 && threadIdx.x == 0) {
            a.sweeps[s] = sweep + 1;
            swept = sweep + 1;
        }
        __syncthreads();
        unsigned nrot = 0, nbig = 0;   // rotations of the sweep; those that force another sweep
        for (int rd = 0; rd < a.nb - 1; ++rd) {
            nrot += pair_round<T, PG, PBW, RPT>(x, blk1, width(player0), width(player1), rd == 0, ka, ldc, tol, floor2,
                                                jnorm, wsteps, steps, nbig, wait);
            const bool last = rd == a.nb - 2;
            if (last && nbig && l == 0) rot_any = 1;   // this workgroup needs another sweep
            // the next round's players (after the last round: round 0 of the next sweep)
            const int nr = (rd + 1) % (a.nb - 1);
            const int R = sweep * (a.nb - 1) + rd;
            const int pos0 = ppos_slot0(wg, R + 1);
            const int next0 = ppos_player(pos0, nr, a.nb), next1 = ppos_player(a.nb - 1 - pos0, nr, a.nb);
            if (next0 != player0) store_col<T, PG, RPT, true>(sv, player0, x);
            if (next1 != player1) store_lds<T, PG, RPT, true>(sv, player1, blk1);
            if (last) {
                // end of the sweep: every workgroup of the slice meets, and all learn
                // whether one needs another sweep (a slice of one block pair asks
                // its own flag: no word is shared)
                int met;
                if (G > 1) {
                    met = slice_meet(counter, G, &rot_any, seen, err, p.spin_limit);
                } else {
                    __syncthreads();
                    met = rot_any ? 1 : 2;
                    __syncthreads();
                }
                if (met != 1) {
                    home0 = next0 == player0;   // giving up, or converged
                    home1 = next1 == player1;
                    alive = false;
                    break;
                }
            } else {
                // within a sweep: publish the block written (ready for round R + 1)
                // and wait only for the block this workgroup takes next
                int* const bf = err + 2 + s * a.nb;
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                if (threadIdx.x == 0) {
                    ok_flag = 1;
                    if (next0 != player0) __hip_atomic_store(bf + player0, R + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (next1 != player1) __hip_atomic_store(bf + player1, R + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((next0 != player0 && !wait_flag(bf + next0, R + 1, err, p.spin_limit)) ||
                        (next1 != player1 && !wait_flag(bf + next1, R + 1, err, p.spin_limit)))
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
        nrot_total += nrot;
    }
    __syncthreads();
    if (home0) store_col<T, PG, RPT, true>(sv, player0, x);
    if (home1) store_lds<T, PG, RPT, true>(sv, player1, blk1);
    if (l == 0 && nrot_total) atomicAdd(a.rotations, (unsigned long long)nrot_total);
    if (a.ctrl && swept) atomicMax(&a.ctrl->sweep_max, swept);
}

// ------------------------------------------------------------------ host

namespace {

constexpr int kPG = 32;   // lanes per pair: 512-thread workgroups, two waves per SIMD

// row groups of PG per stacked column: slice rows and V rows each padded to PG
int persist_rpt(int m, int n) {
    const int need = (m + kPG - 1) / kPG + (n + kPG - 1) / kPG;
    for (int r : {2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16, 20})
        if (r >= need) return r;
    return -1;
}

size_t persist_lds(int rpt, int elem_bytes) { return (size_t)PBW * (kPG * rpt + 1) * 2 * elem_bytes; }

template <typename T, int RPT>
hipError_t launch_persist_t(const JacArgs<T>& a, const PersistArgs& p, size_t lds, hipStream_t st, int cus) {
    auto* fn = jacobi_persistent_kernel<T, kPG, RPT>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, PBW * kPG, lds);
    if (e != hipSuccess) return e;
    const int grid = a.h * (a.nb / 2);
    if ((int64_t)per_cu * cus < grid) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(PBW * kPG), lds, st, a, p);
    return hipGetLastError();
}

}  // namespace

int jacobi_persistent_blocks(int n) { return jacobi_num_blocks(n, PBW); }

bool jacobi_persistent_fits(int m, int n, int h, int elem_bytes, int cus, size_t lds_cap) {
    const int rpt = persist_rpt(m, n);
    if (rpt < 0 || n < 2) return false;
    if (persist_lds(rpt, elem_bytes) + 256 > lds_cap) return false;
    const int64_t grid = (int64_t)h * (jacobi_persistent_blocks(n) / 2);
    return grid <= (int64_t)cus;   // one workgroup per CU is always resident
}

template <typename T>
hipError_t launch_jacobi_persistent(const JacArgs<T>& a, const PersistArgs& p, int cus, hipStream_t st) {
    const int rpt = persist_rpt(a.m, a.n);
    size_t lds = persist_lds(rpt, sizeof(T));
    if (p.spread) {
        // more than half of a CU's LDS: the dispatcher cannot pair workgroups on a CU
        int cap = 0, dev = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cap, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev);
        if ((size_t)cap / 2 + 1024 <= (size_t)cap) lds = std::max(lds, (size_t)cap / 2 + 1024);
    }
    switch (rpt) {
        case 2: return launch_persist_t<T, 2>(a, p, lds, st, cus);
        case 3: return launch_persist_t<T, 3>(a, p, lds, st, cus);
        case 4: return launch_persist_t<T, 4>(a, p, lds, st, cus);
        case 5: return launch_persist_t<T, 5>(a, p, lds, st, cus);
        case 6: return launch_persist_t<T, 6>(a, p, lds, st, cus);
        case 7: return launch_persist_t<T, 7>(a, p, lds, st, cus);
        case 8: return launch_persist_t<T, 8>(a, p, lds, st, cus);
        case 9: return launch_persist_t<T, 9>(a, p, lds, st, cus);
        case 10: return launch_persist_t<T, 10>(a, p, lds, st, cus);
        case 12: return launch_persist_t<T, 12>(a, p, lds, st, cus);
        case 14: return launch_persist_t<T, 14>(a, p, lds, st, cus);
        case 16: return launch_persist_t<T, 16>(a, p, lds, st, cus);
        default: return launch_persist_t<T, 20>(a, p, lds, st, cus);
    }
}

template hipError_t launch_jacobi_persistent<double>(const JacArgs<double>&, const PersistArgs&, int,
                                                     hipStream_t);
template hipError_t launch_jacobi_persistent<float>(const JacArgs<float>&, const PersistArgs&, int,
                                                    hipStream_t);

}  // namespace tsvd
