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

__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Bits 0 to 9 to every third place.
__device__ __forceinline__ uint32_t every_third(uint32_t x) {
    x = (x | x << 16) & 0x030000ffu;
    x = (x | x << 8) & 0x0300f00fu;
    x = (x | x << 4) & 0x030c30c3u;
    return (x | x << 2) & 0x09249249u;
}

// Code of 3 * BITS bits of a cell of a (2^BITS)^3 grid along the Hilbert curve (Skilling's transpose form,
// without branches: about 17 instructions per bit).
template <int BITS>
__device__ __forceinline__ uint32_t hilbert_code(uint32_t x, uint32_t y, uint32_t z) {
    static_assert(BITS <= 10, "");
#pragma unroll
    for (int k = BITS - 1; k > 0; --k) {
        const uint32_t p = (1u << k) - 1u;
        // bit set: flip the bits of x below it; otherwise exchange them with those of the axis
        x ^= p & (uint32_t)__builtin_amdgcn_sbfe((int)x, k, 1);
        const uint32_t my = (uint32_t)__builtin_amdgcn_sbfe((int)y, k, 1);
        const uint32_t ty = (x ^ y) & p & ~my;
        x ^= ty | (p & my);
        y ^= ty;
        const uint32_t mz = (uint32_t)__builtin_amdgcn_sbfe((int)z, k, 1);
        const uint32_t tz = (x ^ z) & p & ~mz;
        x ^= tz | (p & mz);
        z ^= tz;
    }
    y ^= x;
    z ^= y;
    uint32_t t = z >> 1;  // parity of the bits above
    t ^= t >> 1;
    t ^= t >> 2;
    t ^= t >> 4;
    t ^= t >> 8;
    return every_third(x ^ t) << 2 | every_third(y ^ t) << 1 | every_third(z ^ t);
}

// ---- the order of a cloud that does not fill its bounding box ----
// Most clouds are ordered by the cells of a grid over their bounding box.  One with points or tails
// far away, or of a few parts far apart, would leave most of its points to a few cells and their
// order to chance: with one stray point at 300 times the extent of 200,000, to 50,000 samples, rounds went from
// 188 to 1093 and every unit applied every pick (12.9 ms instead of 0.93).  There the coordinates are
// linear within most of the cloud and logarithmic outside, codes have many bits, and the codes of some
// points, sorted, are splitters: a point's key is the splitter below its code and its place on the
// way to the next.  Keys ascend with the codes and are spent where the points are.  (Keys like that for
// every cloud cost ordinary ones 1 to 5 us and a few rounds.)
struct Frame {
    float low[3];  // least coordinates, squashed, so that an axis without extent lies on a face of the grid
    float scale;   // 1 / extent
    float mid[3];  // middle of most of the cloud
    float inv;     // 1 / its width
};
constexpr int kFramePoints = 64;  // points that are looked at, one per lane
constexpr int kFrameCells = 16;   // cells of the longest side of the box, per axis ...
// ... and how many of them these points fill, on the best axis, where a grid will do.  Cubes, rooms, planes and
// surfaces fill 14 to 16; with 9 here instead, normally distributed points and some LiDAR frames still had the
// grid: 300,000 points to 16,384 took 1642 and 1554 us, 1061 and 918 with 13.
constexpr int kFrameFilled = 13;

// Whether a grid over the box (lowest corner, longest side) will do, decided by 64 points, one per lane.
__device__ __forceinline__ bool fills_box(float x, float y, float z, const float (&low)[3], float side) {
    const float per = side > 0.f ? (float)kFrameCells / side : 0.f;
    auto bit = [&](float v, int k) { return 1u << (uint32_t)fmaxf(0.f, fminf((float)(kFrameCells - 1), (v - low[k]) * per)); };
    auto rows_or = [](uint32_t v) {  // over rows of 16 lanes
        v |= dpp_or_zero<kDppRowShr1>(v);
        v |= dpp_or_zero<kDppRowShr2>(v);
        v |= dpp_or_zero<kDppRowShr4>(v);
        return v | dpp_or_zero<kDppRowShr8>(v);
    };
    const uint32_t xy = rows_or(bit(x, 0) | bit(y, 1) << kFrameCells), zz = rows_or(bit(z, 2));
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int l = 15; l < kWave; l += 16) {
        a |= (uint32_t)readlane_i((int)xy, l);
        b |= (uint32_t)readlane_i((int)zz, l);
    }
    const int n = max(max(__builtin_popcount(a & 0xffffu), __builtin_popcount(a >> 16)), __builtin_popcount(b));
    return n >= kFrameFilled || !(side > 0.f);
}

__device__ __forceinline__ float squash(float t) {
    const float a = fabsf(t);
    return copysignf(a <= 1.f ? a : 1.f + __builtin_amdgcn_logf(a), t);
}
template <int BITS>
__device__ __forceinline__ uint32_t code_of(const Frame &f, float x, float y, float z) {
    const float top = (float)((1 << BITS) - 1), scale = f.scale * (float)(1 << BITS);
    auto cell = [&](float v, int k) { return (uint32_t)fmaxf(0.f, fminf(top, (squash((v - f.mid[k]) * f.inv) - f.low[k]) * scale)); };
    return hilbert_code<BITS>(cell(x, 0), cell(y, 1), cell(z, 2));
}

// Point number j of 2^LOG points spread over N, one at a hashed place of each of 2^LOG stretches: a plain
// stride could follow the order in which a sensor lists its points.
template <int LOG>
__device__ __forceinline__ int sample_index(int j, int N) {
    const uint32_t h = ((uint32_t)j * 2654435761u) >> 16;
    return (int)((((uint64_t)((uint32_t)j << 16 | h)) * (uint64_t)(uint32_t)N) >> (16 + LOG));
}

// One value per lane in ascending order of the lanes: a bitonic sort whose steps within rows of 16 are DPP moves.
__device__ __forceinline__ uint32_t wave_sort(uint32_t v, int lane) {
    auto step = [&](uint32_t o, int lower) { v = lane & lower ? umax(v, o) : umin(v, o); };
#define FFPS_DPP(ctrl, x) (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(x), ctrl, 0xf, 0xf, true)
    auto by1 = [&]() { step(FFPS_DPP(0xB1, v), 1); };                  // quad_perm 1,0,3,2
    auto by2 = [&]() { step(FFPS_DPP(0x4E, v), 2); by1(); };           // quad_perm 2,3,0,1
    auto by4 = [&]() { const uint32_t q = FFPS_DPP(0x1B, v); step(FFPS_DPP(0x141, q), 4); by2(); };  // both of the mirrors below
    auto by8 = [&]() { step(FFPS_DPP(0x128, v), 8); by4(); };          // row_ror 8
    by1();
    step(FFPS_DPP(0x1B, v), 2); by1();                                 // quad_perm 3,2,1,0
    step(FFPS_DPP(0x141, v), 4); by2();                                // row_half_mirror
    step(FFPS_DPP(0x140, v), 8); by4();                                // row_mirror
    step((uint32_t)__shfl_xor((int)v, 31), 16); by8();
    step((uint32_t)__shfl_xor((int)v, 63), 32);
    step((uint32_t)__shfl_xor((int)v, 16), 16); by8();
#undef FFPS_DPP
    return v;
}

// Floats as unsigned integers of the same order, and back.
__device__ __forceinline__ uint32_t ordered(float v) { return f2u(v) >> 31 ? ~f2u(v) : f2u(v) | 0x80000000u; }
__device__ __forceinline__ float unordered(uint32_t k) { return u2f(k >> 31 ? k & 0x7fffffffu : ~k); }

// Least and largest of 64 values, one per lane, and the range of most of the distinct ones (points that
// share one place, the way sensors and padding mark what is missing, count once).
struct Spread { float least, most, lo, hi; };
__device__ __forceinline__ Spread spread_of(float value, int lane) {
    const uint32_t v = wave_sort(ordered(value), lane);
    auto at = [&](int l) { return unordered((uint32_t)readlane_i((int)v, l)); };
    const uint64_t firsts = __builtin_amdgcn_ballot_w64(v != (uint32_t)__shfl_up((int)v, 1)) | 1ull;
    const int n = __builtin_popcountll(firsts), rank = lanes_below(firsts);
    const bool first = (firsts >> lane) & 1u;
    return Spread{at(0), at(63), at(first_lane(first && rank == n * 3 / 16)), at(first_lane(first && rank == n * 13 / 16))};
}
__device__ __forceinline__ Frame frame_of(const Spread (&s)[3]) {
    Frame f;
    const float w = fmaxf(fmaxf(s[0].hi - s[0].lo, s[1].hi - s[1].lo), s[2].hi - s[2].lo);
    f.inv = w > 0.f ? 1.f / w : 1.f;
    float extent = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        f.mid[k] = 0.5f * s[k].lo + 0.5f * s[k].hi;
        f.low[k] = squash((s[k].least - f.mid[k]) * f.inv);
        extent = fmaxf(extent, squash((s[k].most - f.mid[k]) * f.inv) - f.low[k]);
    }
    f.scale = extent > 0.f ? 1.f / extent : 1.f;
    return f;
}

// Last of 2^LOG ascending splitters that is not above a code (the first one is 0).
template <int LOG>
__device__ __forceinline__ uint32_t splitter_of(const uint32_t *sp, uint32_t code) {
    uint32_t b = 0;
#pragma unroll
    for (uint32_t o = 1u << (LOG - 1); o > 0; o >>= 1) b += sp[b + o] <= code ? o : 0u;
    return b;
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

}  // namespace ffps
