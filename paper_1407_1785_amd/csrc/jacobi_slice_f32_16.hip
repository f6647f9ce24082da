// The one-workgroup-per-slice and block-pair Jacobi kernels, FP32, blocks of 16 columns.
#include "jacobi_slice.h"

namespace tsvd {

TSVD_SLICE_INSTANCE(float, 16)

}  // namespace tsvd
