// Instantiations of the wide Dynamic-A8 GEMM for the x-tile height of 128 rows
// (kernel in gemm_a8_wide.h).
#include "gemm_a8_wide.h"

namespace cq {

hipError_t launch_a8_wide128(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                            void *y, int y_dt, hipStream_t stream) {
    return a8_wide_bits<8>(w, ctab, x8, dx, m, y, y_dt, stream);
}

}  // namespace cq
