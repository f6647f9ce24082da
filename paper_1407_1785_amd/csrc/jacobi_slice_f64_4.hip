// The one-workgroup-per-slice and block-pair Jacobi kernels, FP64, blocks of 4 columns.
#include "jacobi_slice.h"

namespace tsvd {

TSVD_SLICE_INSTANCE(double, 4)

}  // namespace tsvd
