// Model-dtype many-row GEMM on gfx950 matrix cores: host dispatch over the
// tile configurations (kernel and its description in gemm_a16_mfma.h).
#include "gemm_a16_mfma.h"

namespace cq {

bool gemm_a16_mfma_supported(const cq_weight &w, int64_t m) {
    const int64_t lim = int64_t(1) << 31;
    return w.bits <= 5 && m * w.k * 2 < lim && stream_fits(w.n, w.k, w.bits, w.group) && m < lim;
}

// Up to 64 rows the 64-row weight tiles of gemm_a16_mfma.h put more workgroups
// on the chip (W4 G128, K = 4096, 64 rows: 56 us at N = 4096 and 57 at 14336
// against 63 and 64 for the 128-row tiles of gemm_a16_wide.h); above that the
// wide kernel leads (128 rows: 63 and 66 us against 98).  The heights 128 and
// 256 are the wide kernel's; every height accumulates in the same order.  More
// than 32 rows whose tiles would leave compute units idle take the split-K kernel.
hipError_t launch_gemm_a16_mfma(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                                int tile_rows, hipStream_t stream) {
    if (tile_rows == 0 && m > 32 && gemm_a16_split_preferred(w, m))
        return launch_gemm_a16_split(w, x, x_dt, m, y, y_dt, false, stream);
    const int tr = tile_rows ? tile_rows : m <= 32 ? 32 : m <= 64 ? 64 : 0;
    if (tr == 32) return launch_a16_tile32(w, x, x_dt, m, y, y_dt, false, stream);
    if (tr == 64) return launch_a16_tile64(w, x, x_dt, m, y, y_dt, false, stream);
    return launch_gemm_a16_wide(w, x, x_dt, m, y, y_dt, tr, stream);
}

// the single-rounded operand (an opt-in family) on the 256-row tile
hipError_t launch_gemm_a16_mfma_rounded(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                                        hipStream_t stream) {
    return launch_a16_tile256(w, x, x_dt, m, y, y_dt, true, stream);
}

}  // namespace cq
