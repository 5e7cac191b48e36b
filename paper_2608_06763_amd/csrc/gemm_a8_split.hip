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

// W3 and W4 with G >= 64 have the narrow kernel up to 32 rows (14336 x 4096 W4
// at 32 rows with the quantizer: 22 us against 42 here) and above 64 rows the
// wide kernel, whose sums are those of the partials dump bit for bit.  Up to 16
// rows the other widths and groups had the generic GEMV (generic / here, us):
// 4096 x 12288 W8, 2 rows 61 / 39, 16 rows 112 / 42; 1024 x 32000 W2, 2 rows 25 /
// 15; only W1 does better there below 4 rows (4096 x 20000 G64, 2 rows 20 / 22, 6
// rows 34 / 23).
// Above 16 rows every tile of 32 x 32 forms its carriers anew, which pays while
// the larger tiles of the other kernels leave compute units idle (other / here),
// by rounds of tiles over the chip.  One: 8192 x 512 W5 G32, 256 rows 370 / 41;
// 8192 x 4096 W4, 64 rows 44 / 28; 1024 x 2048 W1, 128 rows 11 / 9.  Two: 4096 x
// 4096, 128 rows W8 58 / 48, G64 W5 110 / 42, but, 64 rows on 4096 x 8192, W4 27 /
// 31 and, K = 1024, W8 20 / 23.  Three: 4096 x 4096, 192 rows G64 W5 112 / 59, but
// G128 52 / 57 and, K = 2048, W8 G64 48 / 51.  Four: 4096 x 32000 W4 G32, 32 rows
// 143 / 65, but W8 G128 74 / 95.
bool gemm_a8_split_preferred(const cq_weight &w, int64_t m) {
    if (m < (w.bits == 1 ? 4 : 2) || !gemm_a8_wide_supported(w, m)) return false;
    const bool tiles = (w.bits == 3 || w.bits == 4) && w.group >= 64;  // has kernels of its own
    if (m <= 16) return !tiles;
    const int64_t rounds = split_rounds(w.n, m);
    if (tiles) return m > 32 && m <= 64 && rounds == 1;
    if (rounds == 1) return true;
    if (rounds == 2) return w.group <= 64 || w.k >= 2048;
    return w.k >= 4096 && (rounds == 3 ? w.group <= 64 : rounds == 4 && w.group == 32);
}

hipError_t launch_gemm_a8_split(const cq_weight &w, const int8_t *x8, const float *dx, int64_t m, void *y, int y_dt,
                                hipStream_t stream) {
    return m <= 16 ? split_bits<1>(w, x8, dx, m, y, y_dt, stream) : split_bits<2>(w, x8, dx, m, y, y_dt, stream);
}

}  // namespace cq
