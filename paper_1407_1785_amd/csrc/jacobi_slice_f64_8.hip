// The one-workgroup-per-slice and block-pair Jacobi kernels, FP64, blocks of 8 columns.
#include "jacobi_slice.h"

namespace tsvd {

TSVD_SLICE_INSTANCE(double, 8)

}  // namespace tsvd
