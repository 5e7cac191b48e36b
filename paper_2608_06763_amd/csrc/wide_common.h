// Building blocks of the wide lane-decoded GEMMs (gfx950): loads straight into
// LDS, their order and their waits, and the tile order over the XCDs.
#pragma once

#include "cq_device.h"
#include "stream_common.h"

#include <type_traits>

namespace cq {

// f(integral_constant<P>) for P = P0 .. PN - 1, in order
template <int P0, int PN, typename F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (P0 < PN) {
        f(std::integral_constant<int, P0>{});
        unroll<P0 + 1, PN>(f);
    }
}

// Every lane brings 16 bytes from its byte offset voff to LDS bytes
// dst + 16 lane .. +15 (dst wave-uniform), without passing through registers.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, uint8_t *dst, uint32_t voff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, voff, 0, 0, 0);
}

// Resource of the `bytes` at `base` from byte `off` on (wave-uniform): the range
// check then covers a step's whole offset, and a last step that reads past the
// tensor stays inside it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t step_rsrc(const void *base, uint32_t bytes, uint32_t off) {
    off = __builtin_amdgcn_readfirstlane(off);
    return make_rsrc(static_cast<const uint8_t *>(base) + off, bytes - off);
}

// Keep loads in program order across this point, for the compiler (the kernel's
// pointers carry no __restrict__, so that a load cannot be moved over the empty
// asm) and for its scheduler.
__device__ __forceinline__ void vmem_order() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0x78f);
}

// Wait until at most N vector-memory loads are in flight and every LDS read
// has returned.
template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N >= 0 && N < 64, "counter range");
    __asm__ volatile("" ::: "memory");
    // vmcnt in bits 3:0 and 15:14, expcnt (no wait) 6:4, lgkmcnt 11:8
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x70);
    __asm__ volatile("" ::: "memory");
}

// Tile index of this workgroup: those of one XCD (blockIdx modulo 8) take
// consecutive tiles, which walk the weight tiles of one activation tile.
__device__ __forceinline__ int xcd_tile(int nwg) {
    const int xcd = int(blockIdx.x) & 7, per = nwg >> 3, rem = nwg & 7;
    return xcd * per + min(xcd, rem) + (int(blockIdx.x) >> 3);
}

// Rounds over the chip's 256 compute units that the 32 x 32 tiles of the split-K
// kernels take.
inline int64_t split_rounds(int64_t n, int64_t m) {
    return ((m + 31) / 32 * ((n + 31) / 32) + 255) / 256;
}

// A use of the operand registers at this point: without one the compiler sinks
// their computation below the matrix work it is meant to run beside.
template <typename V>
__device__ __forceinline__ void pin(V (&op)[2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t w = uint32_t(op[a][b][e]);
                __asm__ volatile("" : "+v"(w));
                op[a][b][e] = int(w);
            }
}

}  // namespace cq
