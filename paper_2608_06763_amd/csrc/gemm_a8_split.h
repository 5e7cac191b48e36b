// Dynamic-A8 GEMM for few rows or few output tiles with lane-decoded carriers and
// split K, every B and G, on gfx950 int8 matrix cores.
//
// Numerics and decoders are those of gemm_a8_wide.h: exact INT32 partials of
// whole groups, rescaled in FP32.  A workgroup owns 16 BI rows of x by 32 rows
// of W; its KS waves split K into contiguous runs of whole groups and add their
// FP32 sums in LDS once at the end, in a fixed order.  Every wave brings its own
// activations straight into its own part of LDS (no barrier in the K loop).  In
// a 128-code step lane block q = l / 16 takes unit q of its weight rows; where a
// step holds several groups (G < 128) each group's matrix instructions see zero
// operands in the other groups' lane blocks.
//
// What bounds it: the decode (W8: FP64 estimates, about 10 instructions a code) and
// its latency at one or two workgroups of eight waves per compute unit: 3072 x 3584
// W5 G512, 64 rows has the VALU 21% busy, the matrix cores 1%.
// Measured with the quantizer: 8192 x 8192 W6 G64, 8 rows 38 us (96 for one wave
// per weight row), 32 rows 42 (180); 3072 x 3584 W5 G512, 64 rows 20 (34 for the
// wide kernel, 128 before it); 8192 x 512 W5 G32, 128 rows 40 (370).
#pragma once

#include "gemm_a8_wide.h"

namespace cq {

// GM as in gemm_a8_wide.h.
template <int B, int GM, int BI, int KS>
__global__ void __launch_bounds__(64 * KS) gemm_a8_split(
    const uint8_t *codes, const float *scale, const uint16_t *a16, const uint16_t *b16, int group, int n, int k,
    const int8_t *x8, const float *dx, int m, void *y, int y_dt, int tiles_m, int tiles_n) {
    using namespace a8_wide;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    using dec_t = decoder<B, false>;
    constexpr int TM = 16 * BI;
    constexpr int NX = TM / 8;        // 1 KB activation pieces (8 rows) of a step
    constexpr int NB = 2;             // activation buffers and code slots
    constexpr int kX = TM * kXRow;    // bytes of one wave's buffer
    constexpr int NG = GM == 0 ? 1 : GM;
    constexpr int kW = 2 * ((B + 3) / 4) + 2 * (B >= 3 ? 3 : 1);  // loads of a step's codes and metadata
    __shared__ __attribute__((aligned(1024))) uint8_t xs0[KS * kX];
    __shared__ __attribute__((aligned(1024))) uint8_t xs1[KS * kX];

    const int wg = xcd_tile(tiles_m * tiles_n);
    const int m0 = (wg / tiles_n) * TM;
    const int n0 = (wg % tiles_n) * 32;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    auto xbuf = [&](auto b_c) __attribute__((always_inline)) -> uint8_t * {
        if constexpr (decltype(b_c)::value % NB == 0) return xs0 + wave * kX;
        else return xs1 + wave * kX;
    };
    const int units = k >> 5, units_per_group = group >> 5;
    const int ng = units / units_per_group;
    const uint32_t row_bytes = uint32_t(k) * B / 8u;
    const auto rc = make_rsrc(codes, uint32_t(n) * row_bytes);
    const auto rs = make_rsrc(scale, uint32_t(n) * ng * 4u);
    const auto ra = make_rsrc(a16, uint32_t(n) * ng * 2u);
    const auto rb = make_rsrc(b16, uint32_t(n) * ng * 2u);

    // this wave's steps [s0, s1): whole groups
    const int nsteps = (units + 3) >> 2;
    const int chunk = GM == 0 ? group >> 7 : 1;
    const int per = ((nsteps + chunk - 1) / chunk + KS - 1) / KS * chunk;
    const int s0 = min(wave * per, nsteps), s1 = min(s0 + per, nsteps);

    // rows past the matrices repeat the last one, their outputs are not stored
    uint32_t coff[2], goff[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        const int row = min(n0 + 16 * jb + (lane & 15), n - 1);
        coff[jb] = uint32_t(row) * row_bytes;
        goff[jb] = uint32_t(row) * uint32_t(ng);
    }
    uint32_t xoff[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const int row = min(m0 + 8 * t + (lane >> 3), m - 1);
        xoff[t] = uint32_t(row) * uint32_t(k) + 16u * uint32_t((lane & 7) ^ (lane >> 3));
    }

    struct wslot {
        uint32_t cw[2][B];
        float s[2];
        uint32_t a[2], b[2];
    };
    wslot ws[NB];
    // Units past the row (a last step that K fills in part) read the row's last
    // unit; their operands are zeroed.
    auto load_w = [&](int st, wslot &o) __attribute__((always_inline)) {
        const int u = min(4 * min(st, nsteps - 1) + q, units - 1);
        const uint32_t g = uint32_t(u / units_per_group);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            load_words<B>(rc, coff[jb] + uint32_t(u) * (4u * B), o.cw[jb]);
            o.s[jb] = load_f32(rs, (goff[jb] + g) * 4u);
            if constexpr (B >= 3) {
                o.a[jb] = load_u16(ra, (goff[jb] + g) * 2u);
                o.b[jb] = load_u16(rb, (goff[jb] + g) * 2u);
            }
        }
    };
    auto load_x = [&](int st, uint8_t *buf) __attribute__((always_inline)) {
        const auto rx = step_rsrc(x8, uint32_t(m) * uint32_t(k), uint32_t(min(st, nsteps - 1)) * 128u);
#pragma unroll
        for (int t = 0; t < NX; ++t) load_lds16(rx, buf + 1024 * t, xoff[t]);
    };

    const i32x4 zero = {0, 0, 0, 0};
    f32x4 accf[BI][2];
    i32x4 part[GM == 0 ? BI : 1][2];  // INT32 partials of groups longer than a step
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            accf[i][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (GM == 0) part[GM == 0 ? i : 0][jb] = zero;
        }
    dec_t dec[2];
    int group_left = chunk;  // GM == 0: steps left of the group
    bool first = true;       // GM == 0: the step opens a group

    const uint32_t xrow = uint32_t(lane & 15) * kXRow;
    const uint32_t xchunk[2] = {16u * uint32_t((2 * q) ^ (lane & 7)), 16u * uint32_t((2 * q + 1) ^ (lane & 7))};
    // Step st reads buffer and slot P = (st - s0) % 2.  Its activations were
    // requested one step ago; the wait counts the loads issued since.
    auto do_step = [&](int st, auto p_c) __attribute__((always_inline)) {
        constexpr int P = decltype(p_c)::value;
        wait_loads<kW>();
        vmem_order();
        load_x(st + 1, xbuf(std::integral_constant<int, P + 1>{}));
        vmem_order();
        const uint8_t *buf = xbuf(p_c);
        const wslot &o = ws[P];
        const bool in = 4 * st + q < units;
        if (GM != 0 || first) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) dec[jb].build(o.a[jb], o.b[jb]);
        }
        i32x4 op[2][2];  // [half of the unit][row block]
        uint32_t tie[2][2] = {{~0u, ~0u}, {~0u, ~0u}};
        int kmin[2][2] = {{0, 0}, {0, 0}};
        uint32_t fw[2][2][window<B>::CW];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            unit_half<B, 0>(o.cw[jb], fw[0][jb]);
            unit_half<B, 1>(o.cw[jb], fw[1][jb]);
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                uint32_t out[4];
                unroll<0, 4>([&](auto t_c) __attribute__((always_inline)) {
                    dec[jb].template quad<decltype(t_c)::value>(fw[kk][jb], out, tie[kk][jb], kmin[kk][jb]);
                });
#pragma unroll
                for (int e = 0; e < 4; ++e) op[kk][jb][e] = int(out[e]);
            }
        auto call = [&](uint32_t t, int k) __attribute__((always_inline)) -> bool {
            return __any(t <= 0x200u || k == -(1 << (B - 1)));
        };
        if (dec_t::kCheck && __builtin_expect(call(min(min(tie[0][0], tie[0][1]), min(tie[1][0], tie[1][1])),
                                                   min(min(kmin[0][0], kmin[0][1]), min(kmin[1][0], kmin[1][1]))), 0)) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    if (!call(tie[kk][jb], kmin[kk][jb])) continue;
                    uint32_t out[4];
                    dec_t::fix(fw[kk][jb], o.a[jb], o.b[jb], out);
#pragma unroll
                    for (int e = 0; e < 4; ++e) op[kk][jb][e] = int(out[e]);
                }
        }
        if (B > 2 || GM != 1) {  // W1 and W2: K is a multiple of a step at G = 128
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) op[kk][jb] = in ? op[kk][jb] : zero;
        }
        // the scale of group e of the step for this lane's weight row, from a
        // lane block that holds it
        float s[NG][2];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const uint32_t sw = __float_as_uint(o.s[jb]);
            if constexpr (NG == 1) {
                s[0][jb] = o.s[jb];
            } else {
                const auto h = __builtin_amdgcn_permlane32_swap(sw, sw, false, false);
                if constexpr (NG == 2) {
                    // blocks 0, 1 hold the first group's scale, 2, 3 the second's
                    s[0][jb] = __uint_as_float(h[0]);
                    s[1][jb] = __uint_as_float(h[1]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s[e % NG][jb] = __uint_as_float(__builtin_amdgcn_permlane16_swap(h[e >> 1], h[e >> 1], false, false)[e & 1]);
                }
            }
        }
        bool last = true;
        if constexpr (GM == 0) {
            last = --group_left == 0;
            if (last) group_left = chunk;
            first = last;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            i32x4 xf[2];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                xf[kk] = *reinterpret_cast<const i32x4 *>(buf + 16 * i * kXRow + xrow + xchunk[kk]);
#pragma unroll
            for (int e = 0; e < NG; ++e)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    i32x4 p = GM == 0 ? part[GM == 0 ? i : 0][jb] : zero;
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk) {
                        i32x4 w = op[kk][jb];
                        if constexpr (NG > 1) w = q / (4 / NG) == e ? w : zero;
                        p = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[kk], w, p, 0, 0, 0);
                    }
                    if constexpr (GM == 0) {
                        part[i][jb] = p;
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) accf[i][jb][r] = __builtin_fmaf(s[e][jb], float(p[r]), accf[i][jb][r]);
                    }
                }
        }
        if (GM == 0 && last) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    i32x4 &p = part[GM == 0 ? i : 0][jb];
#pragma unroll
                    for (int r = 0; r < 4; ++r) accf[i][jb][r] = __builtin_fmaf(s[0][jb], float(p[r]), accf[i][jb][r]);
                    p = zero;
                }
        }
        vmem_order();
        load_w(st + 2, ws[P]);
        vmem_order();
    };
    if (s0 < s1) {
        load_w(s0, ws[0]);
        load_w(s0 + 1, ws[1]);
        load_x(s0, xs0 + wave * kX);
        wait_loads<0>();
        for (int st = s0;;) {
            do_step(st, std::integral_constant<int, 0>{});
            if (++st == s1) break;
            do_step(st, std::integral_constant<int, 1>{});
            if (++st == s1) break;
        }
    }
    wait_loads<0>();

    // row factors of the outputs, requested here so that no store waits for one
    // (before the K loop they took its registers: W4 G32 2560 x 5023, 62 rows 26 ->
    // 29 us)
    vmem_order();
    const auto rd = make_rsrc(dx, uint32_t(m) * 4u);
    float f[BI][4];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) f[i][r] = load_f32(rd, uint32_t(m0 + 16 * i + 4 * q + r) * 4u);
    vmem_order();
    __syncthreads();

    // the waves' sums meet in the first activation buffer, as in
    // gemm_a16_split.h
    f32x4 *red = reinterpret_cast<f32x4 *>(xs0);
    static_assert(sizeof(f32x4) * 64 * BI * 2 * (KS / 2) <= KS * kX, "sums fit");
#pragma unroll
    for (int half = KS / 2; half >= 1; half /= 2) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) red[((wave - half) * (BI * 2) + 2 * i + jb) * 64 + lane] = accf[i][jb];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) accf[i][jb] += red[(wave * (BI * 2) + 2 * i + jb) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave != 0) return;
    // lane l holds x rows 4 (l / 16) .. +3 of a block for weight row l % 16
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = m0 + 16 * i + 4 * q + r;
            if (row >= m) continue;
            const float fr = f[i][r] / 127.0f;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const int col = n0 + 16 * jb + (lane & 15);
                if (col >= n) continue;
                const int64_t at = int64_t(row) * n + col;
                const float v = accf[i][jb][r] * fr;
                if (y_dt == 0) store_out<0>(y, at, v);
                else if (y_dt == 1) store_out<1>(y, at, v);
                else store_out<2>(y, at, v);
            }
        }
}

template <int B, int GM, int BI, int KS>
static hipError_t a8_split_run(const cq_weight &w, const int8_t *x8, const float *dx, int64_t m, void *y, int y_dt,
                               hipStream_t stream) {
    const int64_t tiles_m = (m + 16 * BI - 1) / (16 * BI);
    const int64_t tiles_n = (w.n + 31) / 32;
    if (tiles_m * tiles_n > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_a8_split<B, GM, BI, KS>), dim3(unsigned(tiles_m * tiles_n)), dim3(64 * KS), 0, stream,
                       w.codes, w.scale, w.a, w.b, w.group, int(w.n), int(w.k), x8, dx, int(m), y, y_dt, int(tiles_m),
                       int(tiles_n));
    return hipGetLastError();
}

}  // namespace cq
