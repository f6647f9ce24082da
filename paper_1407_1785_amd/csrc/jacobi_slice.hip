// Launches of the one-workgroup-per-slice and block-pair Jacobi kernels
// (jacobi_slice.h) by element type, block width and rows per lane.

#include "kernels.h"

namespace tsvd {

namespace {

template <typename T>
hipError_t dispatch(SliceOp op, int bw, int rpt, const JacSliceArgs<T>* tab, const int* start, int nprob, int nwg,
                    int* words, int x, bool spread, hipStream_t st) {
    if (rpt < 2 || rpt > 20) return hipErrorInvalidValue;
    switch (bw) {
        case 4: return slice_op<T, 4>(op, rpt, tab, start, nprob, nwg, words, x, spread, st);
        case 8: return slice_op<T, 8>(op, rpt, tab, start, nprob, nwg, words, x, spread, st);
        case 16: return slice_op<T, 16>(op, rpt, tab, start, nprob, nwg, words, x, spread, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

template <typename T>
hipError_t launch_jacobi_pairs(int bw, int rpt, const JacSliceArgs<T>* tab, const int* role_start, int nprob,
                               int nroles, int* words, int spin_limit, bool spread, hipStream_t st) {
    if (rpt < 2 || rpt > 20) return hipErrorInvalidValue;
    if (nroles <= 0) return hipSuccess;
    return dispatch<T>(SliceOp::PAIRS, bw, rpt, tab, role_start, nprob, nroles, words, spin_limit, spread, st);
}

template hipError_t launch_jacobi_pairs<double>(int, int, const JacSliceArgs<double>*, const int*, int, int, int*, int,
                                                bool, hipStream_t);
template hipError_t launch_jacobi_pairs<float>(int, int, const JacSliceArgs<float>*, const int*, int, int, int*, int,
                                               bool, hipStream_t);

int jacobi_slice_rpt(int m, int n) {
    const int need = (m + kPGs - 1) / kPGs + (n + kPGs - 1) / kPGs;
    return need < 2 ? 2 : need;
}

size_t jacobi_slice_lds(int bw, int rpt, int elem_bytes) { return (size_t)bw * (kPGs * rpt + 1) * 2 * elem_bytes; }

int jacobi_slice_max_rpt() { return 20; }

template <typename T>
hipError_t prepare_jacobi_slice(int bw, int rpt) {
    return dispatch<T>(SliceOp::PREPARE, bw, rpt, nullptr, nullptr, 0, 0, nullptr, 0, false, nullptr);
}

template <typename T>
hipError_t launch_jacobi_slice(int bw, int rpt, const JacSliceArgs<T>* tab, const int* wg_start, int nprob,
                               int nwg, int max_sweeps, bool spread, hipStream_t st) {
    return dispatch<T>(SliceOp::SLICE, bw, rpt, tab, wg_start, nprob, nwg, nullptr, max_sweeps, spread, st);
}

template hipError_t prepare_jacobi_slice<double>(int, int);
template hipError_t prepare_jacobi_slice<float>(int, int);
template hipError_t launch_jacobi_slice<double>(int, int, const JacSliceArgs<double>*, const int*, int, int, int, bool,
                                                hipStream_t);
template hipError_t launch_jacobi_slice<float>(int, int, const JacSliceArgs<float>*, const int*, int, int, int, bool,
                                               hipStream_t);

}  // namespace tsvd
