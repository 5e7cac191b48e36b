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
// 17 / 13).  On few weight rows the split kernel leaves most units idle while
// the generic one, a wave per row, is not slowed by its m: W6 11520 x 1678, 5
// rows FP16 29 / 47, BF16 12288 x 1588 33 / 43; W8 8192 x 598 FP16, 12 rows 24 /
// 38; but 8192 x 1228, 16 rows 51 / 36.  So the times of both are estimated, in
// 0.01 us: the generic kernel goes over K in sweeps of 2048 codes, with 1024
// rows in flight; a wave of the split kernel takes an eighth of K in steps of
// 128 codes (FP16 activations as two parts), in rounds of 256 tiles.  (Fitted to
// calls of 5-16 rows, K 1024-16384, N 512-32768: of 3650 on which the split kernel
// ran 280 were more than 3% slower than the generic one, up to 1.6 times; with this
// rule 7 of 4800, up to 1.07 times.)
bool gemm_a16_split_whole_preferred(const cq_weight &w, int x_dt, int64_t m) {
    if (w.bits < 6 || m < 5 || m > 16 || !gemm_a16_wide_supported(w, m)) return false;
    if (m < 12 && w.n * w.k < (1 << 24)) return false;
    const int64_t sweeps = (w.k + 2047) / 2048, waves = (w.n + 1023) / 1024;
    const int64_t generic = 440 + sweeps * (90 + 35 * m + (waves - 1) * (98 + 13 * m));
    const int64_t steps = ((w.k + 127) / 128 + kKS - 1) / kKS, rounds = split_rounds(w.n, m);
    const int64_t split = 100 + rounds * 350 + steps * ((x_dt == 0 ? 320 : 380) + (rounds - 1) * 300);
    return split < generic;
}

// More than 16 rows.  Every tile of 32 x 32 decodes its weights anew, which pays
// while the other kernels, whose tiles are larger, leave compute units idle: for
// up to three rounds of tiles over the chip (other kernel / here, us; 64-row
// tiles up to 64 rows of B <= 5, else the wide kernel).  One round: 8192 x 1024
// W3 G64, 256 rows 151 / 31; 4096 x 2048 W8, 128 rows 73 / 25.  Two: 4096 x 4096
// W4, 128 rows 63 / 38; 2048 x 8192, 64 rows 30 / 26, but W5 34 / 35 (3072 x
// 8192: 50 / 42).  Three: 4096 x 4096, 192 rows W4 64 / 54, W8 75 / 69; 4096 x
// 20000 W8, 20 rows 78 / 66; but 2048 x 4096 W3, 192 rows 35 / 39, and W5 6656 x
// 12159 G256, 47 rows 78 / 88 (8832 x 8560 G128, 51 rows 126 / 118).  Four: 4096 x
// 4096 W4, 256 rows 65 / 71.  Below K = 2048 a wave has fewer than two steps.
bool gemm_a16_split_preferred(const cq_weight &w, int64_t m) {
    if (!gemm_a16_wide_supported(w, m)) return false;
    const int64_t rounds = split_rounds(w.n, m);
    if (rounds > 3) return false;
    return w.k >= (rounds == 3 ? (w.bits == 5 && m <= 64 ? 8192 : 4096) : rounds == 2 && w.bits == 5 ? 3072 : 2048);
}

hipError_t launch_gemm_a16_split(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt, bool whole,
                                 hipStream_t stream) {
    if (whole) return x_dt == 0 ? whole_bits<0>(w, x, m, y, y_dt, stream) : whole_bits<1>(w, x, m, y, y_dt, stream);
    return x_dt == 0 ? parts_bits<0>(w, x, m, y, y_dt, stream) : parts_bits<1>(w, x, m, y, y_dt, stream);
}

}  // namespace cq
