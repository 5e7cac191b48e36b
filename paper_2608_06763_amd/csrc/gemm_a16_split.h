// Model-dtype GEMM for few rows or few output tiles with lane-decoded weight
// operands and split K, every B and G, on gfx950 matrix cores.
//
// Tiling.  A workgroup owns 16 BI rows of x by 32 rows of W; its KS waves split
// K into contiguous runs of 128-code steps and add their FP32 sums in LDS once
// at the end, in a fixed order.  Every wave brings its own activations straight
// into its own part of LDS, so the K loop has no barrier.
//
// K order.  In a step lane block q = l / 16 takes unit q of its weight rows, 8
// codes per matrix instruction, and reads the activations in the same order: a
// lane loads its 32 codes as whole words (full cache lines per row), stays in
// one group and decodes at compile-time positions.
//
// Numerics.  PARTS is the number of BF16 operand parts of an FP32 weight
// s_g sign(k) q(|k|/M): three carry it whole (by truncation, 8 + 8 + 8 bits) for
// up to 16 rows, where the products are FP32 otherwise too; two are hi + lo as
// in the many-row kernels.  FP16 activations: with three parts every activation
// is split exactly into two BF16 numbers; otherwise the weight is one FP16
// operand, as in the many-row kernels.  Infinite activations give what FP32
// products give, with three parts: their sign times the weight's, NaN for 0.
//
// A matrix instruction cuts its sum off below (its result is low by about a
// tenth of a unit of 2^-24, measured), so a chain of them drifts: with one chain
// over all of K the relative error of FP32 outputs was 3.6e-7 at K = 8192 and
// 5.1e-7 at 16384 (W8, BF16).  With three parts only the products of the same 32 codes
// meet in one chain, the smallest first; the chains' sums are added in FP32, by
// pairs within a step, and every other step has its weights negated: 1.0e-7 and
// 1.2e-7, the FP32 GEMV 1.4e-7 at both.
//
// What bounds it: VALU issue of the decode (W8 in three parts about 12
// instructions a code: 8192 x 8192 needs 20 us of it on every SIMD) and its
// latency at two waves per SIMD (VALU 53% busy, matrix cores 6%).
// Measured: 8192 x 8192 W8 G128, 8 rows 34 us (80 for one wave per weight row); with
// one chain of matrix instructions 32, then with K in 64-code steps with 8 codes
// per lane and unit, or with 16 waves, 2 to 4 more.  4096 x 4096 W4, 48 rows 19 us (55 for 64-row tiles);
// 14336 x 4096, 64 rows 46 (184); 4096 x 4096 W4, 128 rows 38 (63 for the wide
// kernel).
#pragma once

#include "gemm_a16_wide.h"

namespace cq {

namespace a16_split {

using namespace a16_wide;

constexpr int kSRow = 256;  // LDS bytes per activation row: 128 codes of K

// codes 8C .. 8C + 7 of a unit as an aligned window
template <int B, int C>
__device__ __forceinline__ void uwindow(const uint32_t *w, uint32_t &f0, uint32_t &f1) {
    constexpr int bit = 8 * C * B, wd = bit >> 5, sh = bit & 31;
    auto word = [&](int i) __attribute__((always_inline)) { return wd + i < B ? w[wd + i] : 0u; };
    if constexpr (sh == 0) {
        f0 = word(0);
        f1 = word(1);
    } else {
        f0 = __builtin_amdgcn_alignbit(word(1), word(0), sh);
        f1 = __builtin_amdgcn_alignbit(word(2), word(1), sh);
    }
}

// an FP32 pair in three truncated BF16 parts
__device__ __forceinline__ void split3(float v0, float v1, uint32_t &a, uint32_t &b, uint32_t &c) {
    const uint32_t u0 = __float_as_uint(v0), u1 = __float_as_uint(v1);
    a = bperm(u1, u0, 0x07060302u);
    v0 -= __uint_as_float(u0 & 0xffff0000u);
    v1 -= __uint_as_float(u1 & 0xffff0000u);
    const uint32_t r0 = __float_as_uint(v0), r1 = __float_as_uint(v1);
    b = bperm(r1, r0, 0x07060302u);
    v0 -= __uint_as_float(r0 & 0xffff0000u);
    v1 -= __uint_as_float(r1 & 0xffff0000u);
    c = bperm(__float_as_uint(v1), __float_as_uint(v0), 0x07060302u);
}

// Operand words op[part][pair] of eight codes.
template <int B, int WDT, int PARTS, int C>
__device__ __forceinline__ void decode8(const decoder_t<B, WDT> &d, const uint32_t *w, uint32_t (&op)[PARTS][4]) {
    uint32_t f0, f1;
    uwindow<B, C>(w, f0, f1);
    int kmin = 0;
    if constexpr (PARTS == 3) {
        unroll<0, 4>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int P = decltype(p_c)::value;
            const int k0 = field<B, 2 * P>(f0, f1), k1 = field<B, 2 * P + 1>(f0, f1);
            kmin = min(kmin, min(k0, k1));
            split3(d.level(k0), d.level(k1), op[0][P], op[1][P], op[2][P]);
        });
    } else {
        uint32_t lo[4];
        unroll<0, 4>([&](auto p_c) __attribute__((always_inline)) {
            d.template step<decltype(p_c)::value>(f0, f1, op[0], lo, kmin);
        });
        if constexpr (PARTS == 2) {
#pragma unroll
            for (int p = 0; p < 4; ++p) op[1][p] = lo[p];
        }
    }
    // the reserved pattern (never written by the packer) decodes to zero
    if (B >= 5 && __builtin_expect(__any(kmin == -(1 << (B - 1))), 0)) {
        unroll<0, 8>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int J = decltype(j_c)::value;
            const uint32_t keep = field<B, J>(f0, f1) == -(1 << (B - 1)) ? (J & 1 ? 0x0000ffffu : 0xffff0000u) : ~0u;
#pragma unroll
            for (int p = 0; p < PARTS; ++p) op[p][J / 2] &= keep;
        });
    }
}

// eight FP16 activations as two BF16 fragments (8 + 3 bits, exact)
__device__ __forceinline__ void split_x(const u32x4 &xf, u32x4 &hi, u32x4 &lo) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float v0 = f16_to_f32(uint16_t(xf[e])), v1 = f16_to_f32(uint16_t(xf[e] >> 16));
        const uint32_t u0 = __float_as_uint(v0), u1 = __float_as_uint(v1);
        hi[e] = bperm(u1, u0, 0x07060302u);
        lo[e] = bperm(__float_as_uint(v1 - __uint_as_float(u1 & 0xffff0000u)),
                      __float_as_uint(v0 - __uint_as_float(u0 & 0xffff0000u)), 0x07060302u);
    }
}

// BF16 pairs with infinities and NaNs replaced by 0
__device__ __forceinline__ u32x4 finite_only(const u32x4 &h, const u32x4 &v) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // an exponent of all ones in h carries into the half's top bit
        const uint32_t bad = (((h[e] & 0x7f807f80u) + 0x00800080u) >> 15) & 0x00010001u;
        o[e] = v[e] & ~(bad * 0xffffu);
    }
    return o;
}

}  // namespace a16_split

// G128: G >= 128, so that the four lanes of a row share a group and form W4's
// tables together.
template <int B, bool G128, int XDT, int BI, int PARTS, int KS>
__global__ void __launch_bounds__(64 * KS, PARTS == 3 ? 4 : 1) gemm_a16_split(
    const uint8_t *codes, const float *scale, const uint16_t *a16, const uint16_t *b16, int units_per_group, int n,
    int k, const uint16_t *x, int m, void *y, int y_dt, int tiles_m, int tiles_n) {
    using namespace a16_split;
    constexpr int WDT = PARTS == 1 ? 1 : 0;  // weight operands: BF16 parts or one FP16
    constexpr int TM = 16 * BI;
    constexpr int NX = TM / 4;        // 1 KB activation pieces (4 rows) of a step
    constexpr int NB = 2;             // activation buffers and code slots
    constexpr int kX = TM * kSRow;    // bytes of one wave's buffer
    // loads of a step's codes and metadata
    constexpr int kW = 2 * ((B + 3) / 4) + 2 * (B >= 3 ? 3 : 1);
    // separate objects, so that reads of one need not wait for loads into another
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
    const int units = k >> 5;
    const int ng = units / units_per_group;
    const uint32_t row_bytes = uint32_t(k) * B / 8u;
    const auto rc = make_rsrc(codes, uint32_t(n) * row_bytes);
    const auto rs = make_rsrc(scale, uint32_t(n) * ng * 4u);
    const auto ra = make_rsrc(a16, uint32_t(n) * ng * 2u);
    const auto rb = make_rsrc(b16, uint32_t(n) * ng * 2u);

    // this wave's steps [s0, s1)
    const int nsteps = (units + 3) >> 2;
    const int per = (nsteps + KS - 1) / KS;
    const int s0 = wave * per, s1 = min(s0 + per, nsteps);

    // rows past the matrices repeat the last one, their outputs are not stored
    uint32_t coff[2], goff[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        const int row = min(n0 + 16 * jb + (lane & 15), n - 1);
        coff[jb] = uint32_t(row) * row_bytes;
        goff[jb] = uint32_t(row) * uint32_t(ng);
    }
    // activation pieces: lane l brings 16 bytes of row l / 16 of the piece to
    // position l % 16 of its LDS row, chunk (position ^ row % 8) of the step
    uint32_t xoff[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const int row = min(m0 + 4 * t + q, m - 1);
        xoff[t] = uint32_t(row) * uint32_t(k) * 2u + 16u * uint32_t((lane & 15) ^ ((4 * t + q) & 7));
    }

    struct wslot {
        uint32_t cw[2][B];
        float s[2];
        uint32_t a[2], b[2];
    };
    wslot ws[NB];
    // Units past the row (a last step K fills in part) read the row's last unit
    // and decode with zero scales; their activations are zeroed.
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
        const auto rx = step_rsrc(x, uint32_t(m) * uint32_t(k) * 2u, uint32_t(min(st, nsteps - 1)) * 256u);
#pragma unroll
        for (int t = 0; t < NX; ++t) load_lds16(rx, buf + 1024 * t, xoff[t]);
    };

    f32x4_t acc[BI][2];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[i][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const uint32_t xrow = uint32_t(lane & 15) * kSRow;
    // Step st reads buffer and slot P = (st - s0) % NB.  Its activations were
    // requested NB - 1 steps ago; the wait counts the loads issued since.
    constexpr int kAfter = (NB - 1) * kW + (NB - 2) * NX;
    bool inf = false;  // PARTS == 3: the second pass below
    auto do_step = [&](int st, auto p_c) __attribute__((always_inline)) {
        constexpr int P = decltype(p_c)::value;
        wait_loads<(kAfter < 62 ? kAfter : 62)>();
        vmem_order();
        load_x(st + NB - 1, xbuf(std::integral_constant<int, P + NB - 1>{}));
        vmem_order();
        const uint8_t *buf = xbuf(p_c);
        const wslot &o = ws[P];
        const bool in = 4 * st + q < units;
        const float sg = PARTS == 3 && (st & 1) ? -1.f : 1.f;
        decoder_t<B, WDT> d[2];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) d[jb].template build<G128, PARTS == 3>(in ? sg * o.s[jb] : 0.f, o.a[jb], o.b[jb], q);
        f32x4_t sum[2], half[2];  // PARTS == 3: chains' sums of this step
        unroll<0, 4>([&](auto c_c) __attribute__((always_inline)) {
            constexpr int C = decltype(c_c)::value;
            uint32_t op[2][PARTS][4];
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) decode8<B, WDT, PARTS, C>(d[jb], o.cw[jb], op[jb]);
#pragma unroll
            for (int i = 0; i < BI; ++i) {
                u32x4 xf = *reinterpret_cast<const u32x4 *>(buf + 16 * i * kSRow + xrow +
                                                            16u * uint32_t((4 * q + C) ^ (lane & 7)));
                if (!in) xf = u32x4{0, 0, 0, 0};
                auto mul = [&](auto p_c, int jb, const u32x4 &xv, f32x4_t c) __attribute__((always_inline)) {
                    constexpr int Q = decltype(p_c)::value;
                    return mma<WDT>(u32x4{op[jb][Q][0], op[jb][Q][1], op[jb][Q][2], op[jb][Q][3]}, xv, c);
                };
                if constexpr (PARTS == 3) {
                    u32x4 h = xf, l = xf;
                    if constexpr (XDT == 1) split_x(xf, h, l);
                    // the smallest products first
                    f32x4_t p[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
                    auto chain = [&](const u32x4 &hf, const u32x4 &lf) __attribute__((always_inline)) {
                        unroll<0, 3>([&](auto r_c) __attribute__((always_inline)) {
                            using Q = std::integral_constant<int, 2 - decltype(r_c)::value>;
                            if constexpr (XDT == 1) {
#pragma unroll
                                for (int jb = 0; jb < 2; ++jb) p[jb] = mul(Q{}, jb, lf, p[jb]);
                            }
#pragma unroll
                            for (int jb = 0; jb < 2; ++jb) p[jb] = mul(Q{}, jb, Q::value == 0 ? h : hf, p[jb]);
                        });
                    };
                    // activations that are not finite meet the first weight part
                    // only, which is 0 where the weight is
                    if (__builtin_expect(inf, 0)) chain(finite_only(h, h), XDT == 1 ? finite_only(h, l) : l);
                    else chain(h, l);
#pragma unroll
                    for (int jb = 0; jb < 2; ++jb) {
                        if constexpr (C == 0) sum[jb] = p[jb];
                        else if constexpr (C == 1) sum[jb] += p[jb];
                        else if constexpr (C == 2) half[jb] = p[jb];
                        else acc[i][jb] += sg * (sum[jb] + (half[jb] + p[jb]));
                    }
                } else {
                    unroll<0, PARTS>([&](auto p_c) __attribute__((always_inline)) {
#pragma unroll
                        for (int jb = 0; jb < 2; ++jb) acc[i][jb] = mul(p_c, jb, xf, acc[i][jb]);
                    });
                }
            }
        });
        vmem_order();
        load_w(st + NB, ws[P]);
        vmem_order();
    };
    while (s0 < s1) {
        // (opaque, so that no address of this rare loop's start is kept in a register)
        int first = s0;
        if constexpr (PARTS == 3) __asm__ volatile("" : "+s"(first));
        unroll<0, NB>([&](auto p_c) __attribute__((always_inline)) { load_w(first + decltype(p_c)::value, ws[decltype(p_c)::value]); });
        unroll<0, NB - 1>([&](auto p_c) __attribute__((always_inline)) { load_x(first + decltype(p_c)::value, xbuf(p_c)); });
        wait_loads<0>();
        for (int st = first;;) {
            do_step(st, std::integral_constant<int, 0>{});
            if (++st == s1) break;
            do_step(st, std::integral_constant<int, 1>{});
            if (++st == s1) break;
        }
        if (PARTS != 3 || inf) break;
        // An activation that is not finite leaves no finite sum in its row and
        // may have met a weight part of 0, or of another sign: only then this
        // wave goes over its steps again.
        float bad = 0.f;
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int e = 0; e < 4; ++e) bad += acc[i][jb][e] - acc[i][jb][e];
        if (__builtin_expect(!__any(!(bad == 0.f)), 1)) break;
        inf = true;
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) acc[i][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        wait_loads<0>();
    }
    wait_loads<0>();
    __syncthreads();

    // the waves' sums meet in the first activation buffer: the upper half hands
    // its sums to the lower, and so on (a fixed order)
    f32x4_t *red = reinterpret_cast<f32x4_t *>(xs0);
    static_assert(sizeof(f32x4_t) * 64 * BI * 2 * (KS / 2) <= KS * kX, "sums fit");
#pragma unroll
    for (int half = KS / 2; half >= 1; half /= 2) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) red[((wave - half) * (BI * 2) + 2 * i + jb) * 64 + lane] = acc[i][jb];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) acc[i][jb] += red[(wave * (BI * 2) + 2 * i + jb) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave != 0) return;
    // lane l holds weight rows 4 (l / 16) .. +3 of a block for x row l % 16
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int row = m0 + 16 * i + (lane & 15);
        if (row >= m) continue;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int col = n0 + 16 * jb + 4 * q + e;
                if (col >= n) continue;
                const int64_t at = int64_t(row) * n + col;
                if (y_dt == 0) store_out<0>(y, at, acc[i][jb][e]);
                else if (y_dt == 1) store_out<1>(y, at, acc[i][jb][e]);
                else store_out<2>(y, at, acc[i][jb][e]);
            }
    }
}

template <int B, bool G128, int XDT, int BI, int PARTS, int KS>
static hipError_t a16_split_run(const cq_weight &w, const void *x, int64_t m, void *y, int y_dt, hipStream_t stream) {
    const int64_t tiles_m = (m + 16 * BI - 1) / (16 * BI);
    const int64_t tiles_n = (w.n + 31) / 32;
    if (tiles_m * tiles_n > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_a16_split<B, G128, XDT, BI, PARTS, KS>), dim3(unsigned(tiles_m * tiles_n)), dim3(64 * KS), 0,
                       stream, w.codes, w.scale, w.a, w.b, w.group / 32, int(w.n), int(w.k),
                       static_cast<const uint16_t *>(x), int(m), y, y_dt, int(tiles_m), int(tiles_n));
    return hipGetLastError();
}

}  // namespace cq
