// Few-row Dynamic-A8 GEMM with split K: dispatch (kernel in gemm_a8_split.h).
#include "gemm_a8_split.h"

namespace cq {

namespace {

constexpr int kKS = 8;  // waves that split K

template <int B, int BI>
hipError_t split_group(const cq_weight &w, const int8_t *x8, const float *dx, int64_t m, void *y, int y_dt,
                       hipStream_t stream) {
    switch (w.group) {
        case 32: return a8_split_run<B, 4, BI, kKS>(w, x8, dx, m, y, y_dt, stream);
        case 64: return a8_split_run<B, 2, BI, kKS>(w, x8, dx, m, y, y_dt, stream);
        case 128: return a8_split_run<B, 1, BI, kKS>(w, x8, dx, m, y, y_dt, stream);
        case 256:
        case 512: return a8_split_run<B, 0, BI, kKS>(w, x8, dx, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

template <int BI>
hipError_t split_bits(const cq_weight &w, const int8_t *x8, const float *dx, int64_t m, void *y, int y_dt,
                      hipStream_t stream) {
    switch (w.bits) {
        case 1: return split_group<1, BI>(w, x8, dx, m, y, y_dt, stream);
        case 2: return split_group<2, BI>(w, x8, dx, m, y, y_dt, stream);
        case 3: return split_group<3, BI>(w, x8, dx, m, y, y_dt, stream);
        case 4: return split_group<4, BI>(w, x8, dx, m, y, y_dt, stream);
        case 5: return split_group<5, BI>(w, x8, dx, m, y, y_dt, stream);
        case 6: return split_group<6, BI>(w, x8, dx, m, y, y_dt, stream);
        case 7: return split_group<7, BI>(w, x8, dx, m, y, y_dt, stream);
        case 8: return split_group<8, BI>(w, x8, dx, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

}  // namespace

// 2 to 64 rows.  W3 and W4 with G >= 64 have the narrow kernel up to 32 rows
// (14336 x 4096 W4 at 32 rows with the quantizer: 22 us against 42 here).  The
// other widths and groups, against the generic GEMV and the wide kernel (us,
// with the quantizer; calls below 21 us are bound by the host): 4096 x 14336
// W8, 8 rows 86 -> 45, 32 rows 65 -> 51; 8192 x 8192 W6 G64, 8 rows 96 -> 38, 32
// rows 180 -> 42; 3072 x 3584 W5 G512, 64 rows 34 -> 20.  Above 32 rows two tiles
// form every carrier twice: 4096 x 4096 W8, 64 rows 59 -> 27, but 4096 x 14336 67
// -> 88; 14336 x 4096 W4, 64 rows 77 -> 44.
bool gemm_a8_split_preferred(const cq_weight &w, int64_t m) {
    if (m < 2 || m > 64 || !gemm_a8_wide_supported(w, m)) return false;
    if (m > 32) return w.n <= 8192;
    return !((w.bits == 3 || w.bits == 4) && w.group >= 64);
}

hipError_t launch_gemm_a8_split(const cq_weight &w, const int8_t *x8, const float *dx, int64_t m, void *y, int y_dt,
                                hipStream_t stream) {
    return m <= 16 ? split_bits<1>(w, x8, dx, m, y, y_dt, stream) : split_bits<2>(w, x8, dx, m, y, y_dt, stream);
}

}  // namespace cq
