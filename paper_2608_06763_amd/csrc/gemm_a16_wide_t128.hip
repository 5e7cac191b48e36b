// Instantiations of the wide model-dtype GEMM for the x-tile height of 128
// rows (kernel in gemm_a16_wide.h).
#include "gemm_a16_wide.h"

namespace cq {

hipError_t launch_a16_wide128(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                             hipStream_t stream) {
    return a16_wide_dtypes<8>(w, x, x_dt, m, y, y_dt, stream);
}

}  // namespace cq
