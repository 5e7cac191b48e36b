// Wide model-dtype GEMM: support and choice of the x-tile height (kernel in
// gemm_a16_wide.h).
#include "gemm_a16_wide.h"

namespace cq {

bool gemm_a16_wide_supported(const cq_weight &w, int64_t m) {
    const int64_t lim = int64_t(1) << 31;
    return m * w.k * 2 < lim && stream_fits(w.n, w.k, w.bits, w.group) && w.n < lim - 128 && m < lim - 256;
}

// A tile costs a part that does not depend on its height (the decode of 128
// weight rows, about ten 16-row blocks' worth) and a part per 16-row block;
// the chip works on one tile per compute unit at a time (two tiles sharing a
// unit take twice as long).  Measured, K = 4096, W4 G128, us by height
// 64 / 128 / 160 / 256: N = 14336: 300 rows 173 / 131 / 86 / 109, 1024 rows
// 404 / 269 / 283 / 197; N = 4096: 512 rows 70 / 77 / 82 / 101.
int a16_wide_tile_rows(const cq_weight &w, int64_t m) {
    const int64_t tn = (w.n + a16_wide::kTN - 1) / a16_wide::kTN;
    int best = 256;
    int64_t best_cost = INT64_MAX;
    for (int rows : {256, 160, 128, 64}) {
        const int64_t tiles = (m + rows - 1) / rows * tn;
        const int64_t cost = (tiles + 255) / 256 * (rows / 16 + 10);
        if (cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
    }
    return best;
}

hipError_t launch_gemm_a16_wide(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                                int tile_rows, hipStream_t stream) {
    switch (tile_rows ? tile_rows : a16_wide_tile_rows(w, m)) {
        case 64: return launch_a16_wide64(w, x, x_dt, m, y, y_dt, stream);
        case 128: return launch_a16_wide128(w, x, x_dt, m, y, y_dt, stream);
        case 160: return launch_a16_wide160(w, x, x_dt, m, y, y_dt, stream);
        case 256: return launch_a16_wide256(w, x, x_dt, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

}  // namespace cq
