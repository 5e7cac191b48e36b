// Dynamic-A8 many-row GEMM (Sec. 5.4), every B and G, with lane-decoded weight
// carriers, on gfx950 int8 matrix cores.
//
// Numerics are eq. a8-output: INT8 activations times exact INT8 weight carriers
// (eq. carrier) accumulate into exact INT32 group partials (eq. a8-int32-bound),
// each converted to FP32 and multiplied by s_g in group order; the row factor
// d_x / 127 multiplies the FP32 sum.
//
// Tiling.  As in gemm_a16_wide.h: a workgroup of four waves owns TM = 16 BI rows
// of x by 128 rows of W; every wave owns all TM rows of x and 32 rows of W.  In
// v_mfma_i32_16x16x64_i8 lane l supplies weight row l % 16 with the K slots
// 16 (l / 16) .. +15, so each lane decodes its own operand registers, and the
// carriers never pass through LDS.  Activations go from memory straight into
// LDS, 128 codes of K per step.
//
// Carriers.  W3..W5 look theirs up in byte tables in registers (one byte
// permute per four W3 codes, two and a select for W4, four and three for W5);
// at G >= 128 every lane forms the whole table of one of four groups and hands
// its words round by row swaps when their group comes, so metadata is read once
// per four groups.  W6..W8 form every carrier from its code.  All estimates are
// FP64, accurate far below 2^-24, so the exact test runs only for a carrier
// within that of a half-integer; with FP32 estimates (margin 4e-4) a wave of
// 4096 codes met it in every step and W8 ran 2.5 times slower.
//
// What bounds it: VALU issue.  Per 128 codes of K a wave of the 256-row tile
// issues 64 MFMAs (1024 cycles) beside 256 instructions of rescale, about 120
// (W4) of decode and 70 of tables: 8192 x 28672 at 8192 rows has the VALU 71% busy,
// the matrix cores 33%, 16% of the time both, at 1.85 GHz.  Measured: 8192 x 28672, W4 G128, 8192 rows
// 2612 us (1473 TOP/s) against 3506 for decoding through LDS; 8192 x 10240 W3,
// 2048 rows 299 (405); 4096 x 14336 W8, 1024 rows 250 (2640 for the 64 x 64
// kernel); 3072 x 3584 W5 G512, 64 rows with the quantizer 34 (128).
#pragma once

#include "cq_device.h"
#include "cq_internal.h"
#include "stream_common.h"
#include "a8_carriers.h"
#include "wide_common.h"

#include <type_traits>

namespace cq {

namespace a8_wide {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kTN = 128;    // weight rows per tile
constexpr int kXRow = 128;  // LDS bytes per activation row: 128 codes of K

// A lane's sixteen codes of a 64-code block are the 16B bits at byte 2Bq
// (q = l / 16) of its 8B bytes.  It loads the aligned window of CW words that
// holds them; odd widths start in the middle of a word for odd q.
template <int B>
struct window {
    static constexpr int CW = (B + 1) / 2;
    static __device__ __forceinline__ uint32_t byte(int q) { return uint32_t(2 * B * q) & ~3u; }
    static __device__ __forceinline__ void align(const uint32_t *w, int q, uint32_t *f) {
        if constexpr (B % 2 == 0) {
#pragma unroll
            for (int i = 0; i < CW; ++i) f[i] = w[i];
        } else {
            const uint32_t cs = 16u * uint32_t(q & 1);
#pragma unroll
            for (int i = 0; i < CW; ++i) f[i] = __builtin_amdgcn_alignbit(i + 1 < CW ? w[i + 1] : 0u, w[i], cs);
        }
    }
};

template <int B, int J>
__device__ __forceinline__ int field(const uint32_t *f) {
    constexpr int bit = J * B, wd = bit >> 5, sh = bit & 31;
    if constexpr (sh + B <= 32) return __builtin_amdgcn_sbfe(int(f[wd]), sh, B);
    else return __builtin_amdgcn_sbfe(int(__builtin_amdgcn_alignbit(f[wd + 1], f[wd], sh)), 0, B);
}

// Sixteen codes of a whole 32-code unit (kk: which half) start at bit 16 kk B of
// its B words, a compile-time position for every width.
template <int B, int KK>
__device__ __forceinline__ void unit_half(const uint32_t *w, uint32_t *f) {
    constexpr int bit = 16 * KK * B, wd = bit >> 5, sh = bit & 31;
#pragma unroll
    for (int i = 0; i < window<B>::CW; ++i) {
        if constexpr (sh == 0) f[i] = w[wd + i];
        else f[i] = __builtin_amdgcn_alignbit(wd + i + 1 < B ? w[wd + i + 1] : 0u, w[wd + i], sh);
    }
}

// State of one (row, group) and the decode of sixteen codes, four at a time.
// `tie` collects the smallest distance of an estimate from a half-integer,
// `kmin` the smallest code; a step in which either calls for it forms its
// carriers again (fix).
template <int B, bool TB>
struct decoder {
    static constexpr int M = max_code(B);
    static constexpr bool kTable = B >= 3 && B <= 5;  // byte tables formed per group
    static constexpr bool kCheck = B >= 6;            // carriers formed per code
    static constexpr int NT = B == 5 ? 4 : 2;         // table words of the magnitudes
    double ca, cb, cc;
    uint32_t ta[NT], tb[NT];

    // carrier of magnitude I from (a, b) in FP64, units of 2^-24 in `tie`
    static __device__ __forceinline__ uint32_t carrier64(int i, double a, double b, double c, uint32_t &tie) {
        const double t = double(i) / M;
        const double v = __builtin_fma(127.0 * t, __builtin_fma(t, __builtin_fma(t, c, b), a), 402653184.0);
        const uint32_t r = uint32_t(__builtin_bit_cast(uint64_t, v)) + 0x00800000u;
        tie = min(tie, (r << 8) + 0x100u);
        return r >> 24;
    }
    // W3..W5: the table words r(0) .. r(M) of a shape (r(0) = 0, r(M) = 127)
    static __device__ __forceinline__ void table(uint32_t a16, uint32_t b16, uint32_t *t) {
        const float af = f16_to_f32(uint16_t(a16)), bf = f16_to_f32(uint16_t(b16));
        const double a = af, b = bf, c = 1.0 - a - b;
        uint32_t tie = ~0u;
#pragma unroll
        for (int w = 0; w < NT; ++w) t[w] = 0;
#pragma unroll
        for (int i = 1; i < M; ++i) t[i / 4] |= carrier64(i, a, b, c, tie) << (8 * (i % 4));
        if (__builtin_expect(__any(tie <= 0x200u), 0)) {
            const float cf = 1.f - af - bf, mg = carrier_margin(af, bf, cf);
#pragma unroll
            for (int w = 0; w < NT; ++w) t[w] = 0;
#pragma unroll
            for (int i = 1; i < M; ++i)
                t[i / 4] |= carrier_u8<M>(i, float(i) / float(M), af, bf, cf, mg) << (8 * (i % 4));
        }
        t[M / 4] |= 127u << (8 * (M % 4));
    }
    // from the table words (W3..W5) or a shape (FP16 bits)
    __device__ __forceinline__ void set(const uint32_t *w) {
        if constexpr (B <= 2) {
            ta[0] = B == 1 ? 0x00007f81u : 0x81007f00u;  // -127, 127 | 0, 127, 0, -127
        } else if constexpr (kTable) {
#pragma unroll
            for (int i = 0; i < NT; ++i) ta[i] = w[i];
            negate();
        } else {
            const double a = f16_to_f32(uint16_t(w[0])), b = f16_to_f32(uint16_t(w[1]));
            ca = a * (127.0 / M);
            cb = b * (127.0 / (double(M) * M));
            cc = (1.0 - a - b) * (127.0 / (double(M) * M * M));
        }
    }
    // the same, forming the table first (TB: w0, w1 are its words already)
    __device__ __forceinline__ void build(uint32_t w0, uint32_t w1) {
        uint32_t t[NT] = {w0, w1};
        if constexpr (kTable && !TB) table(w0, w1, t);
        set(t);
    }
    // the fields above the reserved pattern: W3 0 -r3 -r2 -r1, W4 0 -r7 .. -r1
    __device__ __forceinline__ void negate() {
        if constexpr (B == 3) {
            const uint32_t neg = (0x80808080u - ta[0]) ^ 0x80808080u;
            tb[0] = perm(neg, neg, 0x01020300u);
        } else if constexpr (B == 4) {
            w4_negative_table(ta[0], ta[1], tb[0], tb[1]);
        } else if constexpr (B == 5) {
            // 0 -r15 .. -r13 | -r12 .. -r9 | -r8 .. -r5 | -r4 .. -r1
            tb[0] = perm(ta[3], ta[3], 0x0102030cu);
#pragma unroll
            for (int i = 1; i < 4; ++i) tb[i] = perm(ta[4 - i], ta[3 - i], 0x01020304u);
#pragma unroll
            for (int i = 0; i < 4; ++i) tb[i] = (0x80808080u - tb[i]) ^ 0x80808080u;
        }
    }
    // 127 q(|k|/M) sign(k) + 1.5 * 2^28 in FP64: the low word is the value in
    // units of 2^-24, and its top byte, half a unit added, the rounded carrier.
    // (FP64 multiply-adds issue at the FP32 rate here.)  The estimate's error is
    // below 2^-44; a value within 2^-24 of a half-integer leaves a fraction of at
    // most one unit.
    __device__ __forceinline__ uint32_t estimate(int k, uint32_t &tie) const {
        const double kd = double(k), ak = __builtin_fabs(kd);
        const double v = __builtin_fma(kd, __builtin_fma(ak, __builtin_fma(ak, cc, cb), ca), 402653184.0);
        const uint32_t r = uint32_t(__builtin_bit_cast(uint64_t, v)) + 0x00800000u;
        tie = min(tie, (r << 8) + 0x100u);
        return r;
    }
    static __device__ __forceinline__ uint32_t pack(const uint32_t (&r)[4]) {
        return perm(perm(r[3], r[2], 0x0c0c0703u), perm(r[1], r[0], 0x0c0c0703u), 0x05040100u);
    }
    // carriers of codes 4T .. 4T + 3 (aligned window f) into out[T]
    template <int T>
    __device__ __forceinline__ void quad(const uint32_t *f, uint32_t *out, uint32_t &tie, int &kmin) const {
        if constexpr (B == 4) {
            if constexpr (T % 2 == 0) w4_word_carriers(f[T / 2], ta[0], ta[1], tb[0], tb[1], out[T], out[T + 1]);
        } else if constexpr (B <= 5) {
            constexpr int bit = 4 * B * T, wd = bit >> 5, sh = bit & 31;
            uint32_t v;
            if constexpr (sh + 4 * B <= 32) v = f[wd] >> sh;
            else v = __builtin_amdgcn_alignbit(f[wd + 1], f[wd], sh);
            constexpr uint32_t m = (1u << B) - 1u;
            const uint32_t sel = (v & m) | ((v << (8 - B)) & (m << 8)) | ((v << (16 - 2 * B)) & (m << 16)) |
                                 ((v << (24 - 3 * B)) & (m << 24));
            if constexpr (B == 5) {
                // bits 2:0 index the four 8-entry parts, bits 3 and 4 pick one
                const uint32_t idx = sel & 0x07070707u;
                const uint32_t m3 = perm(0u, 0x00008000u, sel & 0x08080808u);
                const uint32_t m4 = perm(0u, 0x00008000u, (sel >> 1) & 0x08080808u);
                const uint32_t p = (m3 & perm(ta[3], ta[2], idx)) | (~m3 & perm(ta[1], ta[0], idx));
                const uint32_t n = (m3 & perm(tb[3], tb[2], idx)) | (~m3 & perm(tb[1], tb[0], idx));
                out[T] = (m4 & n) | (~m4 & p);
            } else {
                out[T] = perm(B == 3 ? tb[0] : 0u, ta[0], sel);
            }
        } else {
            uint32_t r[4];
            unroll<0, 4>([&](auto e_c) __attribute__((always_inline)) {
                constexpr int E = decltype(e_c)::value;
                const int k = field<B, 4 * T + E>(f);
                kmin = min(kmin, k);
                r[E] = estimate(k, tie);
            });
            out[T] = pack(r);
        }
    }
    // The sixteen carriers again from the same coefficients, the exact test for
    // the few near a tie, the reserved pattern (never written by the packer) as 0.
    // An exact tie needs q = 1/2, which W7 has at t = 2/3 in one group of 7000, and
    // then in nearly every step of the group; with the exact test for all sixteen
    // codes such a step took 10 us (2048 x 1198 W7 G512, 6 rows: 45 us, now 18).
    // (The coefficients are formed anew, from opaque copies of the shape: with the
    // decoder's own, kept alive for this branch, the kernels that spill spilled more,
    // 14464 x 4852 W8 G32, 1503 rows 2270 -> 2660 us.)
    static __device__ __forceinline__ void fix(const uint32_t *f, uint32_t a16, uint32_t b16, uint32_t *out) {
        if constexpr (kCheck) {
            decoder d;
            uint32_t shape[2] = {a16, b16};
            __asm__ volatile("" : "+v"(shape[0]), "+v"(shape[1]));
            d.set(shape);
            uint32_t w[4] = {f[0], window<B>::CW > 1 ? f[1] : 0u, window<B>::CW > 2 ? f[2] : 0u,
                             window<B>::CW > 3 ? f[3] : 0u};
            uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll 1
            for (int t = 0; t < 4; ++t) {
                uint32_t v = w[0], near = 0, r[4];
                unroll<0, 4>([&](auto e_c) __attribute__((always_inline)) {
                    constexpr int E = decltype(e_c)::value;
                    int k = __builtin_amdgcn_sbfe(int(v), E * B, B);
                    if (k == -(1 << (B - 1))) k = 0;
                    uint32_t tie = ~0u;
                    r[E] = d.estimate(k, tie);
                    near |= tie <= 0x200u ? 1u << E : 0u;
                });
                uint32_t q4 = pack(r);
                if (__any(near != 0)) {
#pragma unroll 1
                    for (int e = 0; e < 4; ++e) {
                        if (__any(near & 1u)) {
                            // the double arithmetic stays inside this branch
                            uint32_t ea = shape[0], eb = shape[1];
                            __asm__ volatile("" : "+v"(ea), "+v"(eb));
                            int k = __builtin_amdgcn_sbfe(int(v), 0, B);
                            if (k == -(1 << (B - 1))) k = 0;
                            const int c = exact_carrier(k < 0 ? -k : k, M, double(f16_to_f32(uint16_t(ea))),
                                                        double(f16_to_f32(uint16_t(eb))));
                            q4 = (q4 & 0xffffff00u) | (uint32_t(k < 0 ? -c : c) & 0xffu);
                        }
                        q4 = __builtin_amdgcn_alignbit(q4, q4, 8);
                        v >>= B;
                        near >>= 1;
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    w[i] = B == 8 ? w[i + 1] : __builtin_amdgcn_alignbit(w[i + 1], w[i], 4 * B & 31);
                    o[i] = o[i + 1];
                }
                w[3] = B == 8 ? 0u : w[3] >> (4 * B & 31);
                o[3] = q4;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = o[i];
        }
    }
};

}  // namespace a8_wide

// GM: groups per 128-code step: 4 (G = 32), 2 (G = 64), 1 (G = 128), 0 for
// larger groups, whose INT32 partials live across steps.
template <int B, int GM, int BI, bool TB>
__global__ void __launch_bounds__(256, 2) gemm_a8_wide(
    const uint8_t *codes, const float *scale, const uint16_t *a16, const uint16_t *b16, int group, int n, int k,
    const int8_t *x8, const float *dx, int m, void *y, int y_dt, int tiles_m, int tiles_n, const int8_t *ctab) {
    using namespace a8_wide;
    constexpr int TM = 16 * BI;
    constexpr int NX = TM / 32;  // 1 KB activation pieces (8 rows) per wave and step
    // Groups of 128 codes or more: lane block q takes unit q of every step (any
    // order of K inside a group gives the same INT32 sums), so a lane loads its
    // 32 codes as whole words; smaller groups keep each matrix instruction inside
    // a 64-code block.
    constexpr bool kUnit = GM <= 1;
    // and metadata of four groups at a time, lane block q holding group q
    constexpr bool kBatch = kUnit;
    constexpr int CW = window<B>::CW;
    constexpr int NW = kUnit ? B : 2 * CW;  // code words of a lane per row block and step
    constexpr int NG = GM == 0 ? 1 : GM;  // groups whose tables a step needs
    constexpr bool kAB = B >= 3;          // widths with a shape
    constexpr int NB = BI <= 8 && GM != 0 ? 4 : 2;  // activation buffers
    // loads of one step's codes and metadata
    constexpr int kW = (kUnit ? 2 * ((B + 3) / 4) : 4) + (kBatch ? 0 : NG * 2 * (kAB ? (TB ? 2 : 3) : 1));
    __shared__ __attribute__((aligned(1024))) uint8_t xs0[TM * kXRow];
    __shared__ __attribute__((aligned(1024))) uint8_t xs1[TM * kXRow];
    __shared__ __attribute__((aligned(1024))) uint8_t xs2[NB == 4 ? TM * kXRow : 16];
    __shared__ __attribute__((aligned(1024))) uint8_t xs3[NB == 4 ? TM * kXRow : 16];
    auto xbuf = [&](auto b_c) __attribute__((always_inline)) -> uint8_t * {
        constexpr int P = decltype(b_c)::value % NB;
        if constexpr (P == 0) return xs0;
        else if constexpr (P == 1) return xs1;
        else if constexpr (P == 2) return xs2;
        else return xs3;
    };

    const int wg = xcd_tile(tiles_m * tiles_n);
    const int m0 = (wg / tiles_n) * TM;
    const int n0 = (wg % tiles_n) * kTN;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    const int ng = k / group;
    const uint32_t row_bytes = uint32_t(k) * B / 8u;
    const auto rc = make_rsrc(codes, uint32_t(n) * row_bytes);
    const auto rs = make_rsrc(scale, uint32_t(n) * ng * 4u);
    const auto ra = make_rsrc(a16, uint32_t(n) * ng * 2u);
    const auto rb = make_rsrc(b16, uint32_t(n) * ng * 2u);
    const auto rt = make_rsrc(ctab, TB ? uint32_t(n) * ng * (1u << (B - 1)) : 0u);

    // this lane's weight rows (block jb of the wave: row 16 jb + l % 16); rows
    // past the matrix repeat the last one, their outputs are not stored
    uint32_t coff[2], goff[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        const int row = min(n0 + 32 * wave + 16 * jb + (lane & 15), n - 1);
        coff[jb] = uint32_t(row) * row_bytes + (kUnit ? uint32_t(4 * B * q) : window<B>::byte(q));
        goff[jb] = uint32_t(row) * uint32_t(ng);
    }
    // activation pieces, swizzled as in gemm_a16_wide.h
    uint32_t xoff[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const int row = min(m0 + 8 * (4 * t + wave) + (lane >> 3), m - 1);
        xoff[t] = uint32_t(row) * uint32_t(k) + 16u * uint32_t((lane & 7) ^ (lane >> 3));
    }

    struct wslot {
        uint32_t cw[2][NW];  // [row block]
        float s[NG][2];
        uint32_t a[NG][2], b[NG][2];
    };
    wslot ws[2];
    const int nsteps = (k + 127) >> 7;

    // Codes and metadata of step st.  A last step that K fills in part reads
    // codes and activations of the rows that follow (in bounds: block indices
    // and, where a block itself can be partial, offsets are clamped); their
    // groups lie past the row's and are rescaled by zero.
    const int nblk = (k + 63) >> 6;
    const uint32_t clast = uint32_t(n) * row_bytes - 4u * CW;
    auto load_w = [&](int st, wslot &o) __attribute__((always_inline)) {
        st = __builtin_amdgcn_readfirstlane(min(st, nsteps - 1));
        if constexpr (kUnit) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) load_words_s<B>(rc, coff[jb], uint32_t(st) * (16u * B), o.cw[jb]);
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const uint32_t so = uint32_t(min(2 * st + kk, nblk - 1)) * (8u * B);
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    if constexpr (GM == 4) load_words_s<CW>(rc, min(coff[jb] + so, clast), 0u, o.cw[jb] + kk * CW);
                    else load_words_s<CW>(rc, coff[jb], so, o.cw[jb] + kk * CW);
                }
            }
        }
        if constexpr (kBatch) return;
#pragma unroll
        for (int e = 0; e < NG; ++e) {
            const uint32_t g = __builtin_amdgcn_readfirstlane(GM == 0 ? 128 * st / group : min(GM * st + e, ng - 1));
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                o.s[e][jb] = load_f32_s(rs, goff[jb] * 4u, g * 4u);
                if constexpr (kAB && TB) {
                    uint32_t t[2] = {0, 0};
                    load_words_s<B == 4 ? 2 : 1>(rt, goff[jb] << (B - 1), g << (B - 1), t);
                    o.a[e][jb] = t[0];
                    o.b[e][jb] = t[1];
                } else if constexpr (kAB) {
                    o.a[e][jb] = load_u16_s(ra, goff[jb] * 2u, g * 2u);
                    o.b[e][jb] = load_u16_s(rb, goff[jb] * 2u, g * 2u);
                }
            }
        }
    };
    // kBatch: scales and table words (or shapes) of the current four groups,
    // and the raw metadata of the next four, of this lane's block
    float bs[2], ns[2];
    using dec_t = decoder<B, TB>;
    uint32_t bt[2][dec_t::NT], nt[2][2];
    auto load_batch = [&](int period) __attribute__((always_inline)) {
        const uint32_t g = uint32_t(min(4 * period + q, ng - 1));
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const uint32_t gi = goff[jb] + g;
            ns[jb] = load_f32(rs, gi * 4u);
            if constexpr (kAB && TB) {
                nt[jb][1] = 0;
                load_words<B == 4 ? 2 : 1>(rt, gi << (B - 1), nt[jb]);
            } else if constexpr (kAB) {
                nt[jb][0] = load_u16(ra, gi * 2u);
                nt[jb][1] = load_u16(rb, gi * 2u);
            }
        }
    };
    auto take_batch = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            bs[jb] = ns[jb];
            if constexpr (dec_t::kTable && !TB) {
                dec_t::table(nt[jb][0], nt[jb][1], bt[jb]);
            } else if constexpr (kAB) {
                bt[jb][0] = nt[jb][0];
                bt[jb][1] = nt[jb][1];
            }
        }
    };
    // the word of lane block e for every lane of a row (e compile-time for
    // G = 128, whose groups are steps, else in a scalar register)
    auto from_block = [&](uint32_t w, auto e) __attribute__((always_inline)) -> uint32_t {
        if constexpr (std::is_same_v<decltype(e), int>) {
            return uint32_t(__builtin_amdgcn_ds_bpermute(4 * (16 * e + (lane & 15)), int(w)));
        } else {
            const uint32_t h = __builtin_amdgcn_permlane32_swap(w, w, false, false)[decltype(e)::value >> 1];
            return __builtin_amdgcn_permlane16_swap(h, h, false, false)[decltype(e)::value & 1];
        }
    };
    auto load_x = [&](int st, uint8_t *buf) __attribute__((always_inline)) {
        const auto rx = step_rsrc(x8, uint32_t(m) * uint32_t(k), uint32_t(min(st, nsteps - 1)) * 128u);
#pragma unroll
        for (int t = 0; t < NX; ++t) load_lds16(rx, buf + 1024 * (4 * t + wave), xoff[t]);
    };

    float accf[BI][2][4];
    i32x4 part[GM == 0 ? BI : 1][2];  // INT32 partials of groups longer than a step
    const i32x4 zero = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            if (GM == 0) part[GM == 0 ? i : 0][jb] = zero;
#pragma unroll
            for (int e = 0; e < 4; ++e) accf[i][jb][e] = 0.f;
        }

    decoder<B, TB> dec[NG][2];
    uint32_t bt_used[2][2] = {};  // kBatch: the shapes (B >= 5) behind dec, for fix
    i32x4 op[2][2][2];  // operands [step parity][64-code block][row block]
    // the group (table index) of 64-code block kk for this lane
    auto build = [&](const wslot &o, auto e_c) __attribute__((always_inline)) {
        if constexpr (kBatch) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
            {
                uint32_t w[dec_t::NT];
#pragma unroll
                for (int i = 0; i < dec_t::NT; ++i) w[i] = kAB && !(B == 3 && i) ? from_block(bt[jb][i], e_c) : 0u;
                bt_used[jb][0] = w[0];
                bt_used[jb][1] = w[1];
                dec[0][jb].set(w);
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < NG; ++e)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) dec[e][jb].build(o.a[e][jb], o.b[e][jb]);
    };
    // Operand quad T (0..15: block T / 8, row block T / 4 % 2) of a slot.  At
    // G = 32 the two halves of a block belong to two groups: lanes with q < 2
    // hold codes of the first.
    auto pick = [&](int kk, int jb) __attribute__((always_inline)) -> decoder<B, TB> {
        if constexpr (GM == 4) return q < 2 ? dec[(2 * kk) % NG][jb] : dec[(2 * kk + 1) % NG][jb];
        else return dec[GM == 2 ? kk : 0][jb];
    };
    auto shape_of = [&](const wslot &o, int kk, int jb, uint32_t &a, uint32_t &b) __attribute__((always_inline)) {
        if constexpr (kBatch) {
            a = bt_used[jb][0];
            b = bt_used[jb][1];
            return;
        }
        const int e0 = GM == 4 ? (2 * kk) % NG : GM == 2 ? kk : 0;
        a = o.a[e0][jb];
        b = o.b[e0][jb];
        if constexpr (GM == 4) {
            a = q < 2 ? a : o.a[(2 * kk + 1) % NG][jb];
            b = q < 2 ? b : o.b[(2 * kk + 1) % NG][jb];
        }
    };

    const uint32_t xrow = uint32_t(lane & 15) * kXRow;
    const uint32_t xchunk[2] = {16u * uint32_t((kUnit ? 2 * q : q) ^ (lane & 7)),
                                16u * uint32_t((kUnit ? 2 * q + 1 : 4 + q) ^ (lane & 7))};

    using E0 = std::integral_constant<int, 0>;
    if constexpr (kBatch) load_batch(0);
    load_w(0, ws[0]);
    load_w(1, ws[1]);
    unroll<0, NB - 1>([&](auto b_c) __attribute__((always_inline)) { load_x(decltype(b_c)::value, xbuf(b_c)); });

    uint32_t tie;
    int kmin;
    uint32_t fw[2][2][CW];
    auto align_slot = [&](const wslot &o) __attribute__((always_inline)) {
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            if constexpr (kUnit) {
                unit_half<B, 0>(o.cw[jb], fw[0][jb]);
                unit_half<B, 1>(o.cw[jb], fw[1][jb]);
            } else {
                window<B>::align(o.cw[jb], q, fw[0][jb]);
                window<B>::align(o.cw[jb] + CW, q, fw[1][jb]);
            }
        }
        tie = ~0u;
        kmin = 0;
    };
    auto decode_quad = [&](auto t_c, auto p_c) __attribute__((always_inline)) {
        constexpr int T = decltype(t_c)::value, P = decltype(p_c)::value;
        constexpr int kk = T >> 3, jb = (T >> 2) & 1;
        uint32_t out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = uint32_t(op[P][kk][jb][e]);
        pick(kk, jb).template quad<(T & 3)>(fw[kk][jb], out, tie, kmin);
#pragma unroll
        for (int e = 0; e < 4; ++e) op[P][kk][jb][e] = int(out[e]);
    };
    auto fix_all = [&](const wslot &o, auto p_c) __attribute__((always_inline)) {
        constexpr int P = decltype(p_c)::value;
        if (decoder<B, TB>::kCheck && __builtin_expect(__any(tie <= 0x200u || kmin == -(1 << (B - 1))), 0)) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    uint32_t a = 0, b = 0, out[4];
                    shape_of(o, kk, jb, a, b);
                    decoder<B, TB>::fix(fw[kk][jb], a, b, out);
#pragma unroll
                    for (int e = 0; e < 4; ++e) op[P][kk][jb][e] = int(out[e]);
                }
        }
    };

#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) op[0][kk][jb] = op[1][kk][jb] = zero;
    if constexpr (kBatch) {
        take_batch();
        load_batch(1);
    }
    build(ws[0], E0{});
    align_slot(ws[0]);
    unroll<0, 16>([&](auto t_c) __attribute__((always_inline)) { decode_quad(t_c, std::integral_constant<int, 0>{}); });
    fix_all(ws[0], std::integral_constant<int, 0>{});
    wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");

    // Step st (activation buffer X = st % NB, operands and slot P = st % 2): its
    // matrix work while step st + 1 (slot 1 - P) is decoded.  Step st + NB - 1's
    // activations and step st + 2's codes are requested first; the wait at the
    // end counts the loads issued after step st + 1's activations, as in
    // gemm_a16_wide.h.
    constexpr int kMeta = 2 * (kAB ? (TB ? 2 : 3) : 1);  // loads of load_batch
    constexpr int kAfter = NB == 2 ? kW : 3 * kW + 2 * NX;
    // GM == 0: steps left of the group, its index and scales
    int group_left = group >> 7, group_at = 0;
    float gs[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) gs[jb] = GM == 0 ? __uint_as_float(from_block(__float_as_uint(bs[jb]), 0)) : 0.f;
    auto do_step = [&](int st, auto x_c) __attribute__((always_inline)) {
        constexpr int Y = decltype(x_c)::value, X = Y % NB, P = Y & 1;
        float s[NG][2];
#pragma unroll
        for (int e = 0; e < NG; ++e)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                if constexpr (GM == 0) s[e][jb] = gs[jb];
                else if constexpr (kBatch) s[e][jb] = __uint_as_float(from_block(__float_as_uint(bs[jb]), x_c));
                else s[e][jb] = GM * st + e < ng ? ws[P].s[e][jb] : 0.f;
            }
        vmem_order();
        load_x(st + NB - 1, xbuf(std::integral_constant<int, Y + NB - 1>{}));
        vmem_order();
        load_w(st + 2, ws[P]);
        vmem_order();
        // the next step opens four new groups: their tables, and the request
        // for the four after them
        bool last = false;  // GM == 0: this step ends its group
        if constexpr (GM == 0) {
            last = --group_left == 0;
            if (last) {
                group_left = group >> 7;
                ++group_at;
                if ((group_at & 3) == 0) {
                    take_batch();
                    load_batch((group_at >> 2) + 1);
                }
                build(ws[1 - P], group_at & 3);
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) gs[jb] = __uint_as_float(from_block(__float_as_uint(bs[jb]), group_at & 3));
            }
            vmem_order();
        } else {
            if constexpr (kBatch && Y == 3) {
                take_batch();
                load_batch(((st + 1) >> 2) + 1);
                vmem_order();
            }
            build(ws[1 - P], std::integral_constant<int, (Y + 1) % 4>{});
        }
        align_slot(ws[1 - P]);
        const uint8_t *buf = xbuf(x_c);
        i32x4 p[2][NG][2];
        auto rescale = [&](const i32x4 (&t)[NG][2], int i) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < NG; ++e)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        accf[i][jb][r] = __builtin_fmaf(s[e][jb], float(t[e][jb][r]), accf[i][jb][r]);
        };
        unroll<0, BI>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int I = decltype(i_c)::value;
            i32x4 xf[2];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                xf[kk] = *reinterpret_cast<const i32x4 *>(buf + 16 * I * kXRow + xrow + xchunk[kk]);
            if constexpr (GM == 0) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int jb = 0; jb < 2; ++jb)
                        part[I][jb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[kk], op[P][kk][jb], part[I][jb], 0, 0, 0);
            } else {
                // the groups' partials of row block I; those of block I - 1
                // are rescaled meanwhile
#pragma unroll
                for (int e = 0; e < NG; ++e)
#pragma unroll
                    for (int jb = 0; jb < 2; ++jb) {
                        if constexpr (GM == 1) {
                            const i32x4 t = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[0], op[P][0][jb], zero, 0, 0, 0);
                            p[I & 1][e][jb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[1], op[P][1][jb], t, 0, 0, 0);
                        } else {
                            i32x4 w = op[P][GM == 2 ? e : e / 2][jb];
                            if constexpr (GM == 4) w = (q < 2) == (e % 2 == 0) ? w : zero;
                            p[I & 1][e][jb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[GM == 2 ? e : e / 2], w, zero, 0, 0, 0);
                        }
                    }
                if constexpr (I > 0) rescale(p[(I - 1) & 1], I - 1);
                if constexpr (I == BI - 1) rescale(p[I & 1], I);
            }
            unroll<(16 * I) / BI, (16 * (I + 1)) / BI>([&](auto t_c) __attribute__((always_inline)) {
                decode_quad(t_c, std::integral_constant<int, 1 - P>{});
            });
        });
        pin(op[1 - P]);
        // activation fragments two row blocks ahead of the matrix work
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, GM == 4 ? 8 : 4, 0);
            if (i + 2 < BI) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        if (GM == 0 && last) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    i32x4 &p = part[GM == 0 ? i : 0][jb];
#pragma unroll
                    for (int e = 0; e < 4; ++e) accf[i][jb][e] = __builtin_fmaf(s[0][jb], float(p[e]), accf[i][jb][e]);
                    p = zero;
                }
        }
        fix_all(ws[1 - P], std::integral_constant<int, 1 - P>{});
        constexpr int kWait = kAfter + (GM == 1 && NB == 2 && Y == 3 ? kMeta : 0);
        wait_loads<(kWait < 62 ? kWait : 62)>();
        __builtin_amdgcn_s_barrier();
        __asm__ volatile("" ::: "memory");
    };
    for (int st = 0;;) {
        do_step(st, std::integral_constant<int, 0>{});
        if (++st == nsteps) break;
        do_step(st, std::integral_constant<int, 1>{});
        if (++st == nsteps) break;
        if constexpr (NB == 4 || GM == 1) {
            do_step(st, std::integral_constant<int, 2>{});
            if (++st == nsteps) break;
            do_step(st, std::integral_constant<int, 3>{});
            if (++st == nsteps) break;
        }
    }
    wait_loads<0>();

    // lane l holds x rows 4 (l / 16) .. +3 of a block for weight row l % 16.  All
    // row factors are requested before the first store: y may alias dx for the
    // compiler, and one load per row between the stores took 0.5 us each (W4
    // G128, 1024 x 5000, 1200 rows: 50 us)
    const auto rd = make_rsrc(dx, uint32_t(m) * 4u);
    float f[BI][4];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[i][e] = load_f32(rd, uint32_t(m0 + 16 * i + 4 * q + e) * 4u);
    vmem_order();
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = m0 + 16 * i + 4 * q + e;
            if (row >= m) continue;
            const float fr = f[i][e] / 127.0f;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const int col = n0 + 32 * wave + 16 * jb + (lane & 15);
                if (col >= n) continue;
                const int64_t at = int64_t(row) * n + col;
                const float v = accf[i][jb][e] * fr;
                if (y_dt == 0) store_out<0>(y, at, v);
                else if (y_dt == 1) store_out<1>(y, at, v);
                else store_out<2>(y, at, v);
            }
        }
}

// Tallest tile without register spills: 256 rows for the byte tables of W1..W4
// at G = 128, 128 where carriers are formed per code, tables are larger, or a
// step holds several groups or long partials, 64 at G = 32.
template <int B, int GM>
constexpr int a8_wide_max_bi = GM == 4 ? 4 : GM == 1 && B <= 4 ? 16 : 8;

template <int B, int GM, int BI, bool TB>
static hipError_t a8_wide_run(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                              void *y, int y_dt, hipStream_t stream) {
    const int64_t tiles_m = (m + 16 * BI - 1) / (16 * BI);
    const int64_t tiles_n = (w.n + a8_wide::kTN - 1) / a8_wide::kTN;
    if (tiles_m * tiles_n > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_a8_wide<B, GM, BI, TB>), dim3(unsigned(tiles_m * tiles_n)), dim3(256), 0, stream, w.codes,
                       w.scale, w.a, w.b, w.group, int(w.n), int(w.k), x8, dx, int(m), y, y_dt, int(tiles_m),
                       int(tiles_n), ctab);
    return hipGetLastError();
}

template <int B, int BI, bool TB>
static hipError_t a8_wide_group(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                                void *y, int y_dt, hipStream_t stream) {
    switch (w.group) {
        case 32:
            if constexpr (BI <= a8_wide_max_bi<B, 4> && !TB)
                return a8_wide_run<B, 4, BI, TB>(w, ctab, x8, dx, m, y, y_dt, stream);
            break;
        case 64:
            if constexpr (BI <= a8_wide_max_bi<B, 2>)
                return a8_wide_run<B, 2, BI, TB>(w, ctab, x8, dx, m, y, y_dt, stream);
            break;
        case 128:
            if constexpr (BI <= a8_wide_max_bi<B, 1>)
                return a8_wide_run<B, 1, BI, TB>(w, ctab, x8, dx, m, y, y_dt, stream);
            break;
        case 256:
        case 512:
            if constexpr (BI <= a8_wide_max_bi<B, 0>)
                return a8_wide_run<B, 0, BI, TB>(w, ctab, x8, dx, m, y, y_dt, stream);
            break;
    }
    return hipErrorNotSupported;
}

// One x-tile height each, in files of their own.  ctab (W3 and W4, G >= 64):
// load-time carrier tables to read instead of the shapes.
template <int BI>
static hipError_t a8_wide_bits(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                               void *y, int y_dt, hipStream_t stream) {
    if (ctab) {
        if (w.bits == 3) return a8_wide_group<3, BI, true>(w, ctab, x8, dx, m, y, y_dt, stream);
        if (w.bits == 4) return a8_wide_group<4, BI, true>(w, ctab, x8, dx, m, y, y_dt, stream);
        return hipErrorNotSupported;
    }
    switch (w.bits) {
        case 1: return a8_wide_group<1, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 2: return a8_wide_group<2, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 3: return a8_wide_group<3, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 4: return a8_wide_group<4, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 5: return a8_wide_group<5, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 6: return a8_wide_group<6, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 7: return a8_wide_group<7, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
        case 8: return a8_wide_group<8, BI, false>(w, ctab, x8, dx, m, y, y_dt, stream);
    }
    return hipErrorNotSupported;
}

hipError_t launch_a8_wide32(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                            void *y, int y_dt, hipStream_t stream);
hipError_t launch_a8_wide64(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                            void *y, int y_dt, hipStream_t stream);
hipError_t launch_a8_wide128(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                            void *y, int y_dt, hipStream_t stream);
hipError_t launch_a8_wide256(const cq_weight &w, const int8_t *ctab, const int8_t *x8, const float *dx, int64_t m,
                            void *y, int y_dt, hipStream_t stream);

}  // namespace cq
