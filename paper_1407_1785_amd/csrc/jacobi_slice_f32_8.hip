// The one-workgroup-per-slice and block-pair Jacobi kernels, FP32, blocks of 8 columns.
#include "jacobi_slice.h"

namespace tsvd {

TSVD_SLICE_INSTANCE(float, 8)

}  // namespace tsvd
