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

// Up to 16 rows against the generic GEMV, whose time grows with m.  On few rows
// and few weight rows the split kernel leaves units idle (generic / here, us: W7
// G512 2048 x 1198, 3 rows 12 / 18; W2 G32 3584 x 1397, 2 rows 6 / 10; W8 G32 2048 x
// 1874, 2 rows 10 / 13).  Both times in 0.01 us: the generic kernel goes over K in
// sweeps of 2048 codes, 1024 weight rows in flight, with more registers above 8
// rows; a wave here takes an eighth of K in whole groups, in steps of 128 codes
// (dearer at G = 32 and 64, with several rescales, and beyond 128 cheaper where K
// has at most four groups and half the waves have none), in rounds of 256 tiles.
// Fitted to 11000 calls, K 1024-16384, N 512-32768: on 994 the split kernel is
// more than 3% slower than the generic one, up to 2.1 times; with this rule 166
// are, up to 1.4 times, and 210 more than 3% slower than the split kernel.  W3 and
// W4 with G = 32 never were.
static bool few_rows_faster(const cq_weight &w, int64_t m) {
    const int64_t sweeps = (w.k + 2047) / 2048, more_rows = (w.n + 1023) / 1024 - 1, high = m > 8;
    const int64_t chunk = w.group > 128 ? w.group / 128 : 1, all = (w.k + 127) / 128;
    const int64_t steps = ((all + chunk - 1) / chunk + kKS - 1) / kKS * chunk;
    const int64_t more = (w.n + 8191) / 8192 - 1;  // rounds after the first
    const bool large = w.group > 128, few = w.k <= 4 * w.group;
    auto by_group = [&](int64_t g32, int64_t g64, int64_t g128, int64_t large_few, int64_t large_many) {
        return large ? (few ? large_few : large_many) : w.group == 32 ? g32 : w.group == 64 ? g64 : g128;
    };
    if (w.bits <= 2) {
        const int64_t generic = w.bits == 1
            ? 510 + sweeps * (20 * m - 29 + 53 * high + more_rows * (22 + 4 * m + 24 * high))
            : 420 + sweeps * (24 * m + 21 + 33 * high + more_rows * (40 + 4 * m + 23 * high));
        return (w.bits == 1 ? 470 : 430) +
               steps * (by_group(138, 107, 80, 50, 80) + more * by_group(135, 80, 80, 60, 80)) < generic;
    }
    if (w.bits <= 4) return true;
    const int64_t generic = 590 + sweeps * (372 + 25 * m + 25 * high + more_rows * (143 + 6 * m + 50 * high));
    const int64_t step = w.bits == 5 ? by_group(325, 283, 270, 125, 190) : by_group(325, 283, 270, 150, 270);
    return (large ? 430 : 480) + steps * (step + more * by_group(250, 250, 250, 100, 230)) < generic;
}

// W3 and W4 with G >= 64 have the narrow kernel up to 32 rows (14336 x 4096 W4
// at 32 rows with the quantizer: 22 us against 42 here) and above 64 rows the
// wide kernel, whose sums are those of the partials dump bit for bit.  Up to 16
// rows the other widths and groups had the generic GEMV (generic / here, us):
// 4096 x 12288 W8, 2 rows 61 / 39, 16 rows 112 / 42; 1024 x 32000 W2, 2 rows 25 /
// 15; W1 does better there below 4 rows whatever N (4096 x 20000 G64, 2 rows 20 /
// 22, 6 rows 34 / 23).
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
    if (m <= 16) return !tiles && few_rows_faster(w, m);
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
