// Boxes, curve order and digit ranks: what the kernels that pick local maxima (fps_local.hip,
// fps_block.hip) and the sorts (spatial.hip) share.
#pragma once
#include "fps_device.h"

namespace ffps {

// Workgroup barrier for LDS data alone: stores to memory stay in flight (a barrier of the
// language would wait for them, which is the latency of the exchange once more).
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// LDS that lanes of one wave pass on to one another is read and written in order: only the compiler has to be held.
__device__ __forceinline__ void wave_lds_order() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// Distances to boxes use the operations of sqdist in its order.  Rounding is monotonic, so the
// result is never above the distance, as the kernels compute it, to any point of the box.
struct Box { float lx, ly, lz, hx, hy, hz; };
__device__ __forceinline__ float gap(float lo, float hi, float p) {
    return fmaxf(fmaxf(__fsub_rn(lo, p), __fsub_rn(p, hi)), 0.f);
}
__device__ __forceinline__ float box_dist(const Box &b, float x, float y, float z) {
    const float dx = gap(b.lx, b.hx, x), dy = gap(b.ly, b.hy, y), dz = gap(b.lz, b.hz, z);
    return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
}
__device__ __forceinline__ Box no_box() {
    const float f = __builtin_inff();
    return Box{f, f, f, -f, -f, -f};
}
__device__ __forceinline__ Box box_or(const Box &a, const Box &b) {
    return Box{fminf(a.lx, b.lx), fminf(a.ly, b.ly), fminf(a.lz, b.lz), fmaxf(a.hx, b.hx), fmaxf(a.hy, b.hy), fmaxf(a.hz, b.hz)};
}
__device__ __forceinline__ Box box_shfl_xor(const Box &a, int o) {
    return Box{__shfl_xor(a.lx, o), __shfl_xor(a.ly, o), __shfl_xor(a.lz, o), __shfl_xor(a.hx, o), __shfl_xor(a.hy, o), __shfl_xor(a.hz, o)};
}

__device__ __forceinline__ float box_box(const Box &a, const Box &b) {
    const float dx = fmaxf(fmaxf(__fsub_rn(a.lx, b.hx), __fsub_rn(b.lx, a.hx)), 0.f);
    const float dy = fmaxf(fmaxf(__fsub_rn(a.ly, b.hy), __fsub_rn(b.ly, a.hy)), 0.f);
    const float dz = fmaxf(fmaxf(__fsub_rn(a.lz, b.hz), __fsub_rn(b.lz, a.hz)), 0.f);
    return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
}

// Code of 3 * BITS bits of a cell of a (2^BITS)^3 grid along the Hilbert curve (Skilling's transpose form).
template <int BITS>
__device__ __forceinline__ uint32_t hilbert_code(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t X[3] = {x, y, z};
#pragma unroll
    for (uint32_t q = 1u << (BITS - 1); q > 1; q >>= 1) {
        const uint32_t p = q - 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (X[i] & q) {
                X[0] ^= p;
            } else {
                const uint32_t t = (X[0] ^ X[i]) & p;
                X[0] ^= t;
                X[i] ^= t;
            }
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t t = 0;
#pragma unroll
    for (uint32_t q = 1u << (BITS - 1); q > 1; q >>= 1)
        if (X[2] & q) t ^= q - 1;
    uint32_t r = 0;
#pragma unroll
    for (int k = BITS - 1; k >= 0; --k) {
#pragma unroll
        for (int i = 0; i < 3; ++i) r = (r << 1) | (((X[i] ^ t) >> k) & 1u);
    }
    return r;
}

// Lanes of the wave whose digit equals this lane's (among the lanes of `valid`).
template <int BITS>
__device__ __forceinline__ uint64_t same_digit(uint32_t d, uint64_t valid) {
    uint64_t m = valid;
#pragma unroll
    for (int k = 0; k < BITS; ++k) {
        const bool on = (d >> k) & 1u;
        const uint64_t s = __builtin_amdgcn_ballot_w64(on);
        m &= on ? s : ~s;
    }
    return m;
}
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

}  // namespace ffps
