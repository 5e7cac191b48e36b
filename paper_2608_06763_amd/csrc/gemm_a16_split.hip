// Few-row model-dtype GEMM with split K: dispatch (kernel in gemm_a16_split.h).
#include "gemm_a16_split.h"

namespace cq {

namespace {

constexpr int kKS = 8;  // waves that split K (16 measured slower: one workgroup a compute unit)

// FP32-whole weights, up to 16 rows
template <int XDT>
hipError_t whole_bits(const cq_weight &w, const void *x, int64_t m, void *y, int y_dt, hipStream_t stream) {
    switch (w.bits) {
        case 6: return a16_split_run<6, false, XDT, 1, 3, kKS>(w, x, m, y, y_dt, stream);
        case 7: return a16_split_run<7, false, XDT, 1, 3, kKS>(w, x, m, y, y_dt, stream);
        case 8: return a16_split_run<8, false, XDT, 1, 3, kKS>(w, x, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

// operands of the many-row kernels, tiles of 32 rows
template <int XDT>
hipError_t parts_bits(const cq_weight &w, const void *x, int64_t m, void *y, int y_dt, hipStream_t stream) {
    constexpr int P = XDT == 0 ? 2 : 1;
    switch (w.bits) {
        case 1: return a16_split_run<1, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 2: return a16_split_run<2, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 3: return a16_split_run<3, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 4:
            return w.group >= 128 ? a16_split_run<4, true, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream)
                                  : a16_split_run<4, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 5: return a16_split_run<5, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 6: return a16_split_run<6, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 7: return a16_split_run<7, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
        case 8: return a16_split_run<8, false, XDT, 2, P, kKS>(w, x, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

}  // namespace

// Up to 16 rows, B >= 6, against the generic GEMV, whose time grows with m
// (W8 G128, us, generic / split: 8192 x 8192 at 8 rows 80 / 37; 4096 x 4096 at
// 2, 4, 8 rows 17 / 20, 20 / 20, 25 / 20; 2048 x 2048 at 4, 16 rows 11 / 13,
// 17 / 13).
bool gemm_a16_split_whole_preferred(const cq_weight &w, int64_t m) {
    return w.bits >= 6 && m <= 16 && gemm_a16_wide_supported(w, m) && (m >= 12 || (m >= 5 && w.n * w.k >= (1 << 24)));
}

// 17 to 64 rows.  Up to 32 rows one tile of x, against the wide kernel for B >=
// 6 (W8, K = 4096, 17 rows: 73 / 23 us at N = 8192, 76 / 45 at 14336).  Two
// tiles decode every weight twice, which pays while the other kernels leave
// compute units idle (W4, K = 4096, 64 rows, 64-row tiles / split: 57 / 36 at N
// = 8192, 57 / 68 at 14336; W8, wide / split: 73 / 45 and 76 / 87).  Each wave
// should have two steps.
bool gemm_a16_split_preferred(const cq_weight &w, int64_t m) {
    return m <= 64 && w.k >= 2048 && gemm_a16_wide_supported(w, m) && (m <= 32 || w.n <= 8192);
}

hipError_t launch_gemm_a16_split(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt, bool whole,
                                 hipStream_t stream) {
    if (whole) return x_dt == 0 ? whole_bits<0>(w, x, m, y, y_dt, stream) : whole_bits<1>(w, x, m, y, y_dt, stream);
    return x_dt == 0 ? parts_bits<0>(w, x, m, y, y_dt, stream) : parts_bits<1>(w, x, m, y, y_dt, stream);
}

}  // namespace cq
