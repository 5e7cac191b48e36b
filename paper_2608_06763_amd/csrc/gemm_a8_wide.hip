// Wide Dynamic-A8 GEMM: support and choice of the x-tile height (kernel in
// gemm_a8_wide.h).
#include "gemm_a8_wide.h"

namespace cq {

bool gemm_a8_wide_supported(const cq_weight &w, int64_t m) {
    const int64_t lim = int64_t(1) << 31;
    return m * w.k < lim && stream_fits(w.n, w.k, w.bits, w.group) && w.n < lim - 128 && m < lim - 256;
}

static int max_rows(const cq_weight &w) {
    return w.group == 32 ? 64 : w.group == 128 && w.bits <= 4 ? 256 : 128;
}

// As for the model-dtype kernel: a tile costs the decode of its weight rows
// (about nine 16-row blocks' worth) and a part per 16-row block, one tile per
// compute unit at a time.  Measured, W4 G128, us at 64 / 128 / 256 rows:
// 4096 x 4096, 100 rows: 36 / 47 / 64; 8192 x 28672, 8192 rows: 5296 / 3469 /
// 2740.
int a8_wide_tile_rows(const cq_weight &w, int64_t m) {
    const int64_t tn = (w.n + a8_wide::kTN - 1) / a8_wide::kTN;
    int best = 64;
    int64_t best_cost = INT64_MAX;
    for (int rows : {256, 128, 64, 32}) {
        if (rows > max_rows(w)) continue;
        const int64_t tiles = (m + rows - 1) / rows * tn;
        const int64_t cost = (tiles + 255) / 256 * (rows / 16 + 9);
        if (cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
    }
    return best;
}

hipError_t launch_gemm_a8_wide(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                               void *y, int y_dt, hipStream_t stream) {
    switch (a8_wide_tile_rows(w, m)) {
        case 32: return launch_a8_wide32(w, ctab, x8, dx, m, y, y_dt, stream);
        case 64: return launch_a8_wide64(w, ctab, x8, dx, m, y, y_dt, stream);
        case 128: return launch_a8_wide128(w, ctab, x8, dx, m, y, y_dt, stream);
        case 256: return launch_a8_wide256(w, ctab, x8, dx, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

}  // namespace cq
