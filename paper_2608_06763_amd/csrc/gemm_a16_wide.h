// Model-dtype many-row GEMM (Sec. 5.3, dense tactic), every B and G, with
// lane-decoded weight operands, on gfx950 matrix cores.
//
// Numerics are those of gemm_a16_mfma.h: with BF16 activations every FP32
// weight s_g sign(k) q(|k|/M) is carried as hi + lo BF16 parts (two MFMAs into
// one FP32 accumulator), with FP16 activations as one FP16 operand.
//
// Tiling.  A workgroup of four waves owns TM = 16 BI rows of x by 128 rows of
// W; every wave owns all TM rows of x and 32 rows of W.  In
// v_mfma_f32_16x16x32 lane l supplies weight row l % 16 with the K slots
// 8 (l / 16) .. +7, so each lane decodes its own operand registers: the
// decoded weights never pass through LDS, and no wave decodes a code that
// another wave of the workgroup decodes.  Activations go from memory straight
// into LDS (64 codes of K per step, two buffers, one barrier per step) and are
// read once per wave for four MFMAs (two blocks of weight rows, hi and lo).
//
// Why this split.  A kernel that stages decoded hi and lo tiles in LDS spends
// more LDS time on them (fragment reads, writes and level lookups, about 1300
// of 1024 MFMA cycles per 32 codes at 64 x 64 per wave) than matrix time.  Here
// the LDS carries only activations: 512 + 128 cycles per 1024 MFMA cycles.
//
// What bounds it.  Per 32 codes a wave issues 64 MFMAs (1024 cycles) and about 90
// (W4) to 180 (W6..W8) decode instructions of 4 cycles.  With two tiles to a
// compute unit (two waves per SIMD) that is mostly the matrix cores: W4 at 8192 x
// 10240, 2048 rows keeps them 54% busy, the VALU 33%, 12% of the time both.  A grid
// of at most one tile per unit has one wave per SIMD, whose load latency and
// barriers nothing hides: 4096 x 14336 W6, 512 rows 36% and 31%, 5120 x 13824 W3
// FP16, 300 rows (two activation buffers) 16% and 18%.  Measured at 8192 x 10240, W4 G128, 2048 rows
// (343 GFLOP): 571 us (602 TFLOP/s, twice that in MFMAs) against 791 for the
// LDS-staged kernel; 438 without the decode, 384 without loads too, 359 for the
// MFMAs alone.  4096 x 14336, W6 G128, 512 rows: 125 us against 651 for the
// 64 x 64 kernel.  5120 x 13824, W3 G64, FP16, 300 rows: 108 us against 126.
// The 8192 x 10240 grid is 640 tiles for 256 compute units (2.5 rounds).
#pragma once

#include "cq_device.h"
#include "cq_internal.h"
#include "stream_common.h"
#include "wide_common.h"

#include <type_traits>

namespace cq {

namespace a16_wide {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTN = 128;   // weight rows per tile
constexpr int kXRow = 128; // LDS bytes per activation row: 64 codes of K

template <int XDT>
__device__ __forceinline__ f32x4_t mma(const u32x4 &a, const u32x4 &b, f32x4_t c) {
    if constexpr (XDT == 0)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                       c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b),
                                                      c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16(float v0, float v1) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{v0, v1}, bf16x2_t));
}

__device__ __forceinline__ uint32_t pack_f16(float v0, float v1) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{v0, v1}, f16x2_t));
}

__device__ __forceinline__ uint32_t bperm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// hi and lo operand words of two FP32 weights (hi = RNE(v), lo = RNE(v - hi));
// FP16 operands have no lo part.
template <int XDT>
__device__ __forceinline__ void split2(float v0, float v1, uint32_t &hi, uint32_t &lo) {
    if constexpr (XDT == 0) {
        hi = pack_bf16(v0, v1);
        lo = pack_bf16(v0 - __uint_as_float(hi << 16), v1 - __uint_as_float(hi & 0xffff0000u));
    } else {
        hi = pack_f16(v0, v1);
        lo = 0;
    }
}

// A lane's eight codes of a unit are the 8B bits at bit 8Bq (q = l / 16).  It
// loads the aligned window of CW words that holds them and shifts it down.
template <int B>
struct window {
    static constexpr int CW = (B == 1 || B == 4) ? 1 : (B == 7 ? 3 : 2);
    static __device__ __forceinline__ uint32_t byte(int q) {
        return min(uint32_t(B * q) & ~3u, uint32_t(4 * B - 4 * CW));
    }
    static __device__ __forceinline__ void align(const uint32_t *w, int q, uint32_t &f0, uint32_t &f1) {
        const uint32_t cs = uint32_t(8 * B * q) - 8u * byte(q);
        f1 = 0;
        if constexpr (B == 4) {
            f0 = w[0];
        } else if constexpr (B == 1) {
            f0 = w[0] >> cs;
        } else if constexpr (B == 8) {
            f0 = w[0];
            f1 = w[1];
        } else if constexpr (B == 7) {
            const bool up = cs >= 32u;
            const uint32_t a = up ? w[1] : w[0], b = up ? w[2] : w[1], c = up ? 0u : w[2];
            f0 = __builtin_amdgcn_alignbit(b, a, cs & 31u);
            f1 = __builtin_amdgcn_alignbit(c, b, cs & 31u);
        } else {
            const uint64_t v = ((uint64_t(w[1]) << 32) | w[0]) >> cs;
            f0 = uint32_t(v);
            f1 = uint32_t(v >> 32);
        }
    }
};

// Signed field j (compile-time) of the aligned window; the reserved pattern
// stays -2^(B-1).
template <int B, int J>
__device__ __forceinline__ int field(uint32_t f0, uint32_t f1) {
    constexpr int bit = J * B;
    if constexpr (bit + B <= 32) return __builtin_amdgcn_sbfe(int(f0), bit, B);
    else if constexpr (bit >= 32) return __builtin_amdgcn_sbfe(int(f1), bit - 32, B);
    else return __builtin_amdgcn_sbfe(int(__builtin_amdgcn_alignbit(f1, f0, bit)), 0, B);
}

// ---- B >= 5: every weight from the curve in registers

template <int B, int XDT>
struct curve_decoder {
    float s, a, b, c;

    // ONCE: for weights carried whole
    template <bool SHARE = true, bool ONCE = false>
    __device__ __forceinline__ void build(float sv, uint32_t a16, uint32_t b16, int q) {
        const float av = f16_to_f32(uint16_t(a16)), bv = f16_to_f32(uint16_t(b16));
        const float cv = 1.f - av - bv;
        s = sv;
        if constexpr (B == 5) {
            a = av;
            b = bv;
            c = cv;
        } else {
            // s and the powers of 1/M folded into the coefficients.  With one
            // rounding for each (ONCE) a formed weight is within 0.7 units of 2^-24
            // (rms), 0.8 for a correctly rounded k/M in the Horner form; with one
            // for every factor 1.0 to 1.2, which operands of hi + lo (2^-18) or FP16
            // do not show and which costs less (4096 x 14336 W6, 512 rows: 1%)
            constexpr int M = max_code(B);
            if constexpr (ONCE) {
                a = folded<M>(sv, av);
                b = folded<M * M>(sv, bv);
                c = folded<M * M * M>(sv, cv);
            } else {
                constexpr float m = float(M);
                a = sv * av * (1.f / m);
                b = sv * bv * (1.f / (m * m));
                c = sv * cv * (1.f / (m * m * m));
            }
        }
    }
    // s v / D with one rounding (up to a remainder of 2^-46): the quotient's
    // remainder is exact, D having at most 21 bits
    template <int D>
    static __device__ __forceinline__ float folded(float sv, float v) {
        constexpr float rd = 1.f / float(D);
        const float h = v * rd;
        const float l = __builtin_fmaf(-h, float(D), v) * rd;
        return __builtin_fmaf(sv, h, sv * l);
    }
    __device__ __forceinline__ float level(int k) const {
        const float kf = float(k);
        if constexpr (B == 5) {
            // bit for bit the s * signed_level of the other many-row kernels:
            // k / M correctly rounded by one multiply and one fused multiply-add
            constexpr float M = float(max_code(B));
            constexpr float rh = 1.0f / M;
            constexpr float rl = float(1.0 / double(M) - double(rh));
            const float t = __builtin_fmaf(kf, rh, kf * rl);
            const float ta = __builtin_fabsf(t);
            return s * (t * __builtin_fmaf(ta, __builtin_fmaf(ta, c, b), a));
        } else {
            const float ka = __builtin_fabsf(kf);
            return kf * __builtin_fmaf(ka, __builtin_fmaf(ka, c, b), a);
        }
    }
    // operand words of the lane's eight codes, two codes at a time; kmin keeps
    // the smallest code seen
    template <int P>
    __device__ __forceinline__ void step(uint32_t f0, uint32_t f1, uint32_t *hi, uint32_t *lo, int &kmin) const {
        const int k0 = field<B, 2 * P>(f0, f1), k1 = field<B, 2 * P + 1>(f0, f1);
        kmin = min(kmin, min(k0, k1));
        split2<XDT>(level(k0), level(k1), hi[P], lo[P]);
    }
    // the reserved pattern (never written by the packer) decodes to zero
    static __device__ __forceinline__ void fix(uint32_t f0, uint32_t f1, uint32_t *hi, uint32_t *lo) {
        unroll<0, 8>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int J = decltype(j_c)::value;
            const uint32_t keep = field<B, J>(f0, f1) == -(1 << (B - 1)) ? (J & 1 ? 0x0000ffffu : 0xffff0000u) : ~0u;
            hi[J / 2] &= keep;
            lo[J / 2] &= keep;
        });
    }
};

// ---- B <= 4: byte-permute tables in registers.  Plane p of an operand pair
// (hi low byte, hi high byte, lo low byte, lo high byte) holds one byte per
// level: of the fields 0 .. 2^B - 1 (B <= 3) or of the magnitudes 0 .. 7 (W4,
// the sign being applied to the high bytes).

template <int B, int XDT>
struct table_decoder {
    static constexpr int NP = XDT == 0 ? 4 : 2;
    static constexpr int NW = B >= 3 ? 2 : 1;
    uint32_t ta[NP][NW];

    // SHARE: the four lanes of a row (q = 0..3) form the tables of one group
    // together; without it every lane forms its own
    template <bool SHARE = true, bool ONCE = false>
    __device__ __forceinline__ void build(float s, uint32_t a16, uint32_t b16, int q) {
        if constexpr (B <= 2) {
            uint32_t h, l;
            split2<XDT>(s, -s, h, l);  // low half +s, high half -s
            // W1: [-s, +s]; W2: [0, +s, 0, -s]
            constexpr uint32_t sel_lo = B == 1 ? 0x0c0c0002u : 0x020c000cu;
            constexpr uint32_t sel_hi = B == 1 ? 0x0c0c0103u : 0x030c010cu;
            ta[0][0] = bperm(0u, h, sel_lo);
            ta[1][0] = bperm(0u, h, sel_hi);
            if constexpr (NP == 4) {
                ta[2][0] = bperm(0u, l, sel_lo);
                ta[3][0] = bperm(0u, l, sel_hi);
            }
        } else {
            constexpr int M = max_code(B);
            const float a = f16_to_f32(uint16_t(a16)), b = f16_to_f32(uint16_t(b16));
            const float c = 1.f - a - b;
            auto lev = [&](float t) __attribute__((always_inline)) {
                return s * (t * __builtin_fmaf(t, __builtin_fmaf(t, c, b), a));
            };
            if constexpr (B == 3) {
                uint32_t h0, l0, h1, l1;  // levels (0, 1), (2, 3)
                split2<XDT>(0.f, lev(1.f / 3.f), h0, l0);
                split2<XDT>(lev(2.f / 3.f), lev(1.f), h1, l1);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const uint32_t w0 = p < 2 ? h0 : l0, w1 = p < 2 ? h1 : l1;
                    const uint32_t t = bperm(w1, w0, p & 1 ? 0x07050301u : 0x06040200u);  // levels 0..3
                    ta[p][0] = t;
                    ta[p][1] = bperm(t, t, 0x0102030cu) ^ (p & 1 ? 0x80808000u : 0u);  // 0, -3, -2, -1
                }
            } else {
                if constexpr (!SHARE) {
                    uint32_t h[4], l[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        split2<XDT>(lev(float(2 * i) / float(M)), lev(float(2 * i + 1) / float(M)), h[i], l[i]);
                    planes(h, 0);
                    if constexpr (NP == 4) planes(l, 2);
                    return;
                }
                // the lanes l % 16 + 16 q of a row evaluate magnitudes 2q, 2q + 1
                // and share them by row swaps
                const float t0 = float(2 * q) / float(M), t1 = float(2 * q + 1) / float(M);
                uint32_t h, l;
                split2<XDT>(lev(t0), lev(t1), h, l);
                gather(h, 0);
                if constexpr (NP == 4) gather(l, 2);
            }
        }
    }
    // planes p, p + 1 from the words (level 2q | level 2q + 1 << 16) of the
    // four lanes of a row
    __device__ __forceinline__ void gather(uint32_t w, int p) {
        const auto s32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);  // lanes 0..31, lanes 32..63
        const auto s0 = __builtin_amdgcn_permlane16_swap(s32[0], s32[0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(s32[1], s32[1], false, false);
        const uint32_t v[4] = {s0[0], s0[1], s1[0], s1[1]};
        planes(v, p);
    }
    __device__ __forceinline__ void planes(const uint32_t *v, int p) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t sel = e ? 0x07050301u : 0x06040200u;
            ta[p + e][0] = bperm(v[1], v[0], sel);
            ta[p + e][NW - 1] = bperm(v[3], v[2], sel);
        }
    }
    // operand words of the lane's eight codes, four codes at a time
    template <int P>
    __device__ __forceinline__ void step(uint32_t f0, uint32_t f1, uint32_t *hi, uint32_t *lo, int &) const {
        if constexpr (P % 2 == 0) {
            constexpr int Q = P / 2;
            uint32_t idx, sign = 0;
            if constexpr (B == 4) {
                // magnitudes of the eight fields: 16 - f for f = 9 .. 15 and 0
                // for the reserved 8
                const uint32_t neg = (f0 >> 3) & 0x11111111u;
                const uint32_t mag = (((f0 & 0x77777777u) ^ (neg | (neg << 1) | (neg << 2))) + neg) & 0x77777777u;
                constexpr uint32_t sel = Q ? 0x07030602u : 0x05010400u;
                idx = bperm((mag >> 4) & 0x0f0f0f0fu, mag & 0x0f0f0f0fu, sel);
                sign = bperm(f0 & 0x80808080u, (f0 & 0x08080808u) << 4, sel);
            } else {
                constexpr uint32_t m = (1u << B) - 1u;
                const uint32_t v = f0 >> (4 * B * Q);
                idx = (v & m) | ((v << (8 - B)) & (m << 8)) | ((v << (16 - 2 * B)) & (m << 16)) |
                      ((v << (24 - 3 * B)) & (m << 24));
            }
            uint32_t pl[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                pl[p] = bperm(ta[p][NW - 1], ta[p][0], idx);
                if (B == 4 && p % 2 == 1) pl[p] ^= sign;
            }
            hi[2 * Q] = bperm(pl[1], pl[0], 0x05010400u);
            hi[2 * Q + 1] = bperm(pl[1], pl[0], 0x07030602u);
            if constexpr (NP == 4) {
                lo[2 * Q] = bperm(pl[3], pl[2], 0x05010400u);
                lo[2 * Q + 1] = bperm(pl[3], pl[2], 0x07030602u);
            }
        }
    }
    static __device__ __forceinline__ void fix(uint32_t, uint32_t, uint32_t *, uint32_t *) {}
};

template <int B, int XDT>
using decoder_t = std::conditional_t<(B <= 4), table_decoder<B, XDT>, curve_decoder<B, XDT>>;

}  // namespace a16_wide

// SPG: steps per group, 0 for G = 32 (a step then spans two groups), 1 and 2 for
// G = 64 and 128, whose group starts are compile-time positions of the unrolled
// loop, 4 for larger groups (a uniform branch).
template <int B, int SPG, int XDT, int YDT, int BI>
__global__ void __launch_bounds__(256, 2) gemm_a16_wide(
    const uint8_t *codes, const float *scale, const uint16_t *a16, const uint16_t *b16, int units_per_group, int n,
    int k, const uint16_t *x, int m, void *y, int tiles_m, int tiles_n) {
    using namespace a16_wide;
    constexpr bool SPLIT = XDT == 0;
    constexpr int TM = 16 * BI;
    constexpr int NX = TM / 32;  // 1 KB activation pieces (8 rows) per wave and step
    constexpr int CW = window<B>::CW;
    static_assert(BI % 2 == 0, "whole pieces per wave");
    // NB activation buffers and code slots: a step's loads are requested NB - 1
    // (activations) and NB (codes) steps ahead
    constexpr int NB = BI <= 8 ? 4 : 2;
    // separate objects, so that reads of one need not wait for loads into another
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
    const int units = k >> 5;
    const int ng = units / units_per_group;
    const uint32_t row_bytes = uint32_t(k) * B / 8u;
    const auto rc = make_rsrc(codes, uint32_t(n) * row_bytes);
    const auto rs = make_rsrc(scale, uint32_t(n) * ng * 4u);
    const auto ra = make_rsrc(a16, uint32_t(n) * ng * 2u);
    const auto rb = make_rsrc(b16, uint32_t(n) * ng * 2u);

    // this lane's weight rows (block jb of the wave: row 16 jb + l % 16);
    // rows past the matrix repeat the last one, their outputs are not stored
    uint32_t coff[2], goff[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        const int row = min(n0 + 32 * wave + 16 * jb + (lane & 15), n - 1);
        coff[jb] = uint32_t(row) * row_bytes + window<B>::byte(q);
        goff[jb] = uint32_t(row) * uint32_t(ng);
    }
    // Activation pieces: piece t of the wave holds 8 rows; lane l brings the
    // 16 bytes of row l / 8 that belong at position l % 8 of its LDS row:
    // position p holds chunk p ^ (row % 8), so that the 16 rows of a fragment
    // read lie in different banks.  Rows past the matrix repeat the last one
    // (their outputs are not stored).
    uint32_t xoff[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const int row = min(m0 + 8 * (4 * t + wave) + (lane >> 3), m - 1);
        xoff[t] = uint32_t(row) * uint32_t(k) * 2u + 16u * uint32_t((lane & 7) ^ (lane >> 3));
    }

    struct wslot {
        uint32_t cw[2][2][CW];  // [block][unit of the step]
    };
    wslot ws[NB];
    // metadata of the next group whose tables are built; G = 32: of the next four
    // groups, lane block q holding group q, and of the current four.  (With one
    // group at a time the lines of 128 rows' metadata left the L1 between the loads
    // of one and the next: W3, 9216 x 15652 FP16, 104 rows 265 us, now 148.)
    float ms[2], cs[2];
    uint32_t ma[2], mb[2], cab[2];
    const int nsteps = (units + 1) >> 1;

    // codes of step st (units past the last repeat it)
    auto load_w = [&](int st, wslot &o) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int u = min(2 * st + kk, units - 1);
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) load_words_s<CW>(rc, coff[jb], uint32_t(u) * (4u * B), o.cw[jb][kk]);
        }
    };
    auto load_meta = [&](int group) __attribute__((always_inline)) {
        if constexpr (SPG == 0) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const uint32_t gi = goff[jb] + uint32_t(min(4 * group + q, ng - 1));
                ms[jb] = load_f32(rs, gi * 4u);
                if constexpr (B >= 3) {
                    ma[jb] = load_u16(ra, gi * 2u);
                    mb[jb] = load_u16(rb, gi * 2u);
                }
            }
            return;
        }
        const uint32_t g = __builtin_amdgcn_readfirstlane(min(group, ng - 1));
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            ms[jb] = load_f32_s(rs, goff[jb] * 4u, g * 4u);
            if constexpr (B >= 3) {
                ma[jb] = load_u16_s(ra, goff[jb] * 2u, g * 2u);
                mb[jb] = load_u16_s(rb, goff[jb] * 2u, g * 2u);
            }
        }
    };
    auto load_x = [&](int st, uint8_t *buf) __attribute__((always_inline)) {
        const auto rx = step_rsrc(x, uint32_t(m) * uint32_t(k) * 2u, uint32_t(min(st, nsteps - 1)) * 128u);
#pragma unroll
        for (int t = 0; t < NX; ++t) load_lds16(rx, buf + 1024 * (4 * t + wave), xoff[t]);
    };

    f32x4_t acc[BI][2];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[i][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    decoder_t<B, XDT> dec[2];
    uint32_t hi[2][2][4], lo[2][2][4];  // operands [phase parity][block]

    // tables or coefficients of the next group, and the request for the one after;
    // G = 32: of group E of the current four, and where E is 0 the next four become
    // current
    int next_group = 0;
    auto build = [&](auto e_c) __attribute__((always_inline)) {
        constexpr int E = decltype(e_c)::value;
        if constexpr (SPG == 0) {
            if constexpr (E == 0) {
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    cs[jb] = ms[jb];
                    if constexpr (B >= 3) cab[jb] = ma[jb] | (mb[jb] << 16);
                }
                load_meta(++next_group);
            }
            auto from_block = [&](uint32_t w) __attribute__((always_inline)) -> uint32_t {
                const uint32_t h = __builtin_amdgcn_permlane32_swap(w, w, false, false)[E >> 1];
                return __builtin_amdgcn_permlane16_swap(h, h, false, false)[E & 1];
            };
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const uint32_t ab = B >= 3 ? from_block(cab[jb]) : 0u;
                dec[jb].build(__uint_as_float(from_block(__float_as_uint(cs[jb]))), ab & 0xffffu, ab >> 16, q);
            }
            return;
        }
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) dec[jb].build(ms[jb], ma[jb], mb[jb], q);
        load_meta(++next_group);
    };

    // fragment of x rows 16 i .. +15, unit kk of the step
    const uint32_t xrow = uint32_t(lane & 15) * kXRow;
    const uint32_t xchunk[2] = {16u * uint32_t(q ^ (lane & 7)), 16u * uint32_t((4 + q) ^ (lane & 7))};

    // matrix work of unit KK of the step in `buf` on operand set KK, while the
    // next unit's codes (words cw) are decoded into the other set
    auto phase = [&](const uint8_t *buf, const wslot &o, auto kk_c) __attribute__((always_inline)) {
        constexpr int KK = decltype(kk_c)::value;
        uint32_t f0[2], f1[2];
        int kmin = 0;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) window<B>::align(o.cw[jb][1 - KK], q, f0[jb], f1[jb]);
        unroll<0, BI>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int I = decltype(i_c)::value;
            const u32x4 xf = *reinterpret_cast<const u32x4 *>(buf + 16 * I * kXRow + xrow + xchunk[KK]);
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
                acc[I][jb] = mma<XDT>(u32x4{hi[KK][jb][0], hi[KK][jb][1], hi[KK][jb][2], hi[KK][jb][3]}, xf, acc[I][jb]);
            if constexpr (SPLIT) {
#pragma unroll
                for (int jb = 0; jb < 2; ++jb)
                    acc[I][jb] = mma<XDT>(u32x4{lo[KK][jb][0], lo[KK][jb][1], lo[KK][jb][2], lo[KK][jb][3]}, xf, acc[I][jb]);
            }
            // the eight pairs of codes of the two blocks, spread over the rows
            unroll<(8 * I) / BI, (8 * (I + 1)) / BI>([&](auto p_c) __attribute__((always_inline)) {
                constexpr int P = decltype(p_c)::value;
                constexpr int jb = P >> 2;
                dec[jb].template step<(P & 3)>(f0[jb], f1[jb], hi[1 - KK][jb], lo[1 - KK][jb], kmin);
            });
        });
        // the decode belongs to this phase: without a use here the compiler
        // sinks it below the matrix work
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                __asm__ volatile("" : "+v"(hi[1 - KK][jb][e]));
                if constexpr (SPLIT) __asm__ volatile("" : "+v"(lo[1 - KK][jb][e]));
            }
        // activation fragments four reads ahead of the matrix work
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, SPLIT ? 4 : 2, 0);
            if (i + 4 < BI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (B >= 5 && __builtin_expect(__any(kmin == -(1 << (B - 1))), 0)) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) dec[jb].fix(f0[jb], f1[jb], hi[1 - KK][jb], lo[1 - KK][jb]);
        }
    };

    load_meta(0);
    unroll<0, NB>([&](auto b_c) __attribute__((always_inline)) { load_w(decltype(b_c)::value, ws[decltype(b_c)::value]); });
    unroll<0, NB - 1>([&](auto b_c) __attribute__((always_inline)) { load_x(decltype(b_c)::value, xbuf(b_c)); });
    build(std::integral_constant<int, 0>{});
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        uint32_t f0, f1;
        int kmin = 0;
        window<B>::align(ws[0].cw[jb][0], q, f0, f1);
        unroll<0, 4>([&](auto p_c) __attribute__((always_inline)) {
            dec[jb].template step<decltype(p_c)::value>(f0, f1, hi[0][jb], lo[0][jb], kmin);
        });
        dec[jb].fix(f0, f1, hi[0][jb], lo[0][jb]);
    }
    wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");

    // Step st (buffer and slot P = st % NB): unit 2 st while unit 2 st + 1 is
    // decoded, then unit 2 st + 1 while the first unit of step st + 1 is
    // decoded.  The activations of step st + NB - 1 and, once slot P is used
    // up, the codes of step st + NB are requested meanwhile.  The barrier at
    // the end must find this wave's activations of step st + 1 in LDS; loads
    // complete in issue order, so it waits until no more loads are in flight
    // than were issued after them (kAfter; the metadata requests, which come
    // now and then, are counted where they are known to be recent, and
    // otherwise only make the wait longer).  The codes thus stay in flight
    // across barriers.
    int group_left = units_per_group >> 1;  // steps left of the group
    constexpr int kMeta = 2 * (B >= 3 ? 3 : 1);
    constexpr int kAfter = NB == 2 ? 4 : 3 * 4 + 2 * NX;
    auto do_step = [&](int st, auto p_c) __attribute__((always_inline)) {
        constexpr int P = decltype(p_c)::value;
        if constexpr (SPG == 0) build(std::integral_constant<int, (2 * P + 1) % 4>{});
        vmem_order();
        load_x(st + NB - 1, xbuf(std::integral_constant<int, P + NB - 1>{}));
        vmem_order();
        phase(xbuf(p_c), ws[P], std::integral_constant<int, 0>{});
        vmem_order();
        load_w(st + NB, ws[P]);
        vmem_order();
        bool start = SPG == 1 || (SPG != 4 && P % 2 == 1);  // a request for metadata follows
        if constexpr (SPG == 4) {
            start = --group_left == 0;
            if (start) group_left = units_per_group >> 1;
        }
        if (start || SPG == 0) build(std::integral_constant<int, (2 * P + 2) % 4>{});
        vmem_order();
        phase(xbuf(p_c), ws[(P + 1) % NB], std::integral_constant<int, 1>{});
        if (NB == 2 && start) wait_loads<kAfter + kMeta>();
        else wait_loads<kAfter>();
        __builtin_amdgcn_s_barrier();
        __asm__ volatile("" ::: "memory");
    };
    const int full = units >> 1;  // steps of two units; a lone last unit follows
    if (full > 0) {
        // every exit leaves the loop at once, so that the waits the compiler
        // places at its head see one order of loads
        for (int st = 0;;) {
            do_step(st, std::integral_constant<int, 0>{});
            if (++st == full) break;
            do_step(st, std::integral_constant<int, 1>{});
            if (++st == full) break;
            if constexpr (NB == 4) {
                do_step(st, std::integral_constant<int, 2>{});
                if (++st == full) break;
                do_step(st, std::integral_constant<int, 3>{});
                if (++st == full) break;
            }
        }
    }
    if (units & 1) {
        const uint8_t *last = (full & 1) ? xs1 : xs0;
        if (NB == 4 && (full & 2)) last = (full & 1) ? xs3 : xs2;
        phase(last, ws[0], std::integral_constant<int, 0>{});
    }
    wait_loads<0>();

    // lane l holds weight rows 4 (l / 16) .. +3 of a block for x row l % 16.  One
    // store of four outputs at the alignment of one: with four stores of one where
    // N is no multiple of 4, calls of short K lost more than the K loop gained
    // (1024 x 6249 W1 FP16, 3501 rows: 81 us, now 62)
    typedef f32x4_t f32x4_e __attribute__((aligned(4)));
    typedef u32x2 u32x2_e __attribute__((aligned(2)));
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int row = m0 + 16 * i + (lane & 15);
        if (row >= m) continue;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int col = n0 + 32 * wave + 16 * jb + 4 * q;
            const int64_t at = int64_t(row) * n + col;
            if (col + 4 <= n) {
                if constexpr (YDT == 2) {
                    *reinterpret_cast<f32x4_e *>(static_cast<float *>(y) + at) = acc[i][jb];
                } else {
                    const f32x4_t v = acc[i][jb];
                    const u32x2 o = YDT == 0 ? u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])}
                                             : u32x2{pack_f16(v[0], v[1]), pack_f16(v[2], v[3])};
                    *reinterpret_cast<u32x2_e *>(static_cast<uint16_t *>(y) + at) = o;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < n) store_out<YDT>(y, at + e, acc[i][jb][e]);
            }
        }
    }
}

template <int B, int SPG, int XDT, int YDT, int BI>
static hipError_t a16_wide_run(const cq_weight &w, const void *x, int64_t m, void *y, hipStream_t stream) {
    const int64_t tiles_m = (m + 16 * BI - 1) / (16 * BI);
    const int64_t tiles_n = (w.n + a16_wide::kTN - 1) / a16_wide::kTN;
    if (tiles_m * tiles_n > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_a16_wide<B, SPG, XDT, YDT, BI>), dim3(unsigned(tiles_m * tiles_n)), dim3(256), 0, stream,
                       w.codes, w.scale, w.a, w.b, w.group / 32, int(w.n), int(w.k), static_cast<const uint16_t *>(x),
                       int(m), y, int(tiles_m), int(tiles_n));
    return hipGetLastError();
}

template <int B, int XDT, int YDT, int BI>
static hipError_t a16_wide_launch(const cq_weight &w, const void *x, int64_t m, void *y, hipStream_t stream) {
    switch (w.group) {
        case 32: return a16_wide_run<B, 0, XDT, YDT, BI>(w, x, m, y, stream);
        case 64: return a16_wide_run<B, 1, XDT, YDT, BI>(w, x, m, y, stream);
        case 128: return a16_wide_run<B, 2, XDT, YDT, BI>(w, x, m, y, stream);
        case 256:
        case 512: return a16_wide_run<B, 4, XDT, YDT, BI>(w, x, m, y, stream);
    }
    return hipErrorNotSupported;
}

template <int XDT, int YDT, int BI>
static hipError_t a16_wide_bits(const cq_weight &w, const void *x, int64_t m, void *y, hipStream_t stream) {
    switch (w.bits) {
        case 1: return a16_wide_launch<1, XDT, YDT, BI>(w, x, m, y, stream);
        case 2: return a16_wide_launch<2, XDT, YDT, BI>(w, x, m, y, stream);
        case 3: return a16_wide_launch<3, XDT, YDT, BI>(w, x, m, y, stream);
        case 4: return a16_wide_launch<4, XDT, YDT, BI>(w, x, m, y, stream);
        case 5: return a16_wide_launch<5, XDT, YDT, BI>(w, x, m, y, stream);
        case 6: return a16_wide_launch<6, XDT, YDT, BI>(w, x, m, y, stream);
        case 7: return a16_wide_launch<7, XDT, YDT, BI>(w, x, m, y, stream);
        case 8: return a16_wide_launch<8, XDT, YDT, BI>(w, x, m, y, stream);
    }
    return hipErrorNotSupported;
}

template <int BI>
static hipError_t a16_wide_dtypes(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                                  hipStream_t stream) {
    if (x_dt == 0) {
        if (y_dt == 0) return a16_wide_bits<0, 0, BI>(w, x, m, y, stream);
        return a16_wide_bits<0, 2, BI>(w, x, m, y, stream);
    }
    if (y_dt == 1) return a16_wide_bits<1, 1, BI>(w, x, m, y, stream);
    return a16_wide_bits<1, 2, BI>(w, x, m, y, stream);
}

// One x-tile height each, in files of their own.
hipError_t launch_a16_wide64(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                             hipStream_t stream);
hipError_t launch_a16_wide128(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                              hipStream_t stream);
hipError_t launch_a16_wide160(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                              hipStream_t stream);
hipError_t launch_a16_wide256(const cq_weight &w, const void *x, int x_dt, int64_t m, void *y, int y_dt,
                              hipStream_t stream);

}  // namespace cq
