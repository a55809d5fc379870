// Many-channel block-CSR products with FP32 blocks and vectors.
#include "spmm_mfma.h"

namespace wpcd {
hipError_t launch_spmm_pk(int64_t rows, int nch, int B, const int64_t* rowptr, const int32_t* col, const float* val,
                          const float2* x, float2* y, hipStream_t s, int cb0, int cb1, const int32_t* order,
                          const PackView& pk, bool blockwise) {
  return spmm::launch(rows, nch, B, rowptr, col, val, x, y, s, cb0, cb1, order, pk, blockwise);
}
}  // namespace wpcd
