// k_fps_block: exact FPS (Sec. 3.1, Eq. 1) of a cloud held by one workgroup, by local maxima
// (the rule, and why picks may be made and applied out of order, stands in fps_local.hip).
//
// What bounds a cloud this small is the number of instructions of a round (with two waves on a
// SIMD an instruction costs about eight cycles): nine tenths of its 3300 cycles with 1024 points, five sixths of 4900 with
// 4096, where the waves wait for the one that has most picks to apply (seven tenths in LiDAR stretches).  k_fps_wgm takes 20 to 30 picks a round but
// needs about 12,000 cycles for it: pairwise masks of 64 candidates, one wave that settles them,
// and every pick applied to every point.  Here a round has eleven picks and takes 1.3 us (1024 points):
//   - The points are put along a space-filling curve (two stable radix passes in LDS, by cells of a
//     grid over the cloud or, where that would not do, by splitters: fps_space.h); a UNIT
//     is a row of 16 lanes with P points each, 32 units in eight waves, so that everything a
//     unit does is done for the four units of a wave by the same instructions and a
//     reduction is four DPP steps.  (64 units in sixteen waves make 0.7 times the rounds, but
//     the pairwise tests are four times as many.)
//   - Every unit puts its two best points and a bound of the values of all others into LDS; a lane tests
//     the unit's candidate against two units, a row against all of them.  (With the value of the second
//     alone, 57 rounds in place of 48 for 1024 points to 512, 126 in place of 100 for 4096 to 1024, each 12 to 17 %
//     shorter: 76 us against 73, 239 against 214.  With one point per lane it is still that way: the second
//     made no fewer rounds of 300 and 512 points, and 2 % of the time.)
//   - Every unit has a slot for its pick (value 0: none), so a round needs two barriers.
//     Picks near the unit's box are applied, two at a time.  All waves see all slots, so each counts
//     the picks for itself (an atomic in LDS, and looking at half of the units only where the boxes
//     of the others are near, which one of a wave's lanes always was: 75 us in place of 73).
//   - Once there are as many picks as samples, a round counts the picks above the largest
//     value that is left; when these are enough it is the last.
// Measured against k_fps_wgm, one cloud of planes and clusters (before the second points): 1024 points to 512 in 70 us
// (54 rounds), 119 there; 4096 to 1024 in 230 us (119 rounds), 364 there; 4608 to 2304 in 400 us (198 rounds), 646 there.
#include "fps_exchange.h"
#include "fps_block.h"
#include "fps_space.h"

namespace ffps {

namespace {

constexpr int kBlockWaves = 8;
constexpr int kBlockThreads = kBlockWaves * kWave;
constexpr int kBlockUnits = kBlockThreads / 16;
constexpr int kDigits = 64;   // six of the twelve bits of a key: of a 16^3 grid, or splitters and places between two
constexpr int kCodeBits = 8;  // per axis, of the codes that have splitters
constexpr int kSplitBits = 6, kSplitters = 1 << kSplitBits;
static_assert(kSplitters == kDigits && kSplitters == kWave && kFramePoints == kWave, "a splitter per lane");
static_assert(kDigits * kBlockWaves == kBlockThreads, "one counter per thread");
constexpr int kBins = 4 * kBlockThreads;  // of pick values, in the final sort
constexpr uint32_t kBinMax = 64;          // picks of a bin that are compared with one another

__host__ __device__ constexpr size_t pow2_above(int n) { return n <= 1 ? 1 : 2 * pow2_above((n + 1) / 2); }

// unsigned maximum over each row of 16 lanes, in all of them
__device__ __forceinline__ uint32_t row_max_all(uint32_t v) {
    v = umax(v, dpp_or_zero<0xB1>(v));   // quad_perm 1,0,3,2
    v = umax(v, dpp_or_zero<0x4E>(v));   // quad_perm 2,3,0,1
    v = umax(v, dpp_or_zero<0x141>(v));  // row_half_mirror
    v = umax(v, dpp_or_zero<0x140>(v));  // row_mirror
    return v;
}
// this row's sixteen bits of a wave's mask
__device__ __forceinline__ uint32_t row_bits(uint64_t m, int lane) {
    const uint32_t half = lane & 32 ? (uint32_t)(m >> 32) : (uint32_t)m;
    return (half >> (lane & 16)) & 0xffffu;
}
__device__ __forceinline__ uint64_t key_of(const u32x4 &rec) { return ((uint64_t)rec.y << 32) | rec.x; }

// Waves per SIMD the registers have to leave room for.  With two points per lane six (three clouds on a CU): 80 registers,
// five of them spilled outside the rounds.  With 86 a CU holds two clouds, and 600 of 1000 points to 300 took 115 us, 101 now.
constexpr int waves_per_simd(int P) { return P == 2 ? 6 : 2; }

// Clouds of a launch beyond which a CU holds several workgroups: FAR below.
constexpr int kOnePerCu = 256;

// FAR: a wave passes over the half of the units that is not around it where the boxes are too far apart for every lane.  With
// one workgroup on a CU that is slower (the test comes before the loads: 1 to 3 % of 1024 and 4096 points); with several,
// instructions count, and LiDAR stretches and clusters have such halves: 512 clouds of 3000 to 700 303 and 178 us without, 281 and
// 167 with it, cubes and rooms the same.
template <int P, bool FAR>
__global__ __launch_bounds__(kBlockThreads, waves_per_simd(P)) void k_fps_block(BlockArgs a) {
    constexpr int kCap = kBlockThreads * P;
    constexpr bool kTwo = P > 1;  // units report their second points
    constexpr bool kTwoOfTies = P <= 3;  // also where values are equal (see report)
    // coordinates by index and the order, later the keys of the picks
    __shared__ __attribute__((aligned(16))) float sx[4 * kCap];
    uint32_t *order = reinterpret_cast<uint32_t *>(sx + 3 * kCap);
    __shared__ uint32_t bins[kBins];  // first the digits' counters, one set per wave
    uint32_t(*cnt)[kDigits] = reinterpret_cast<uint32_t(*)[kDigits]>(bins);
    __shared__ float wbox[kBlockWaves][6];
    __shared__ Spread part[3];
    __shared__ float per_code[kSplitters];
    __shared__ uint32_t split[kSplitters];
    __shared__ uint32_t wsum[kBlockWaves], wtop[kBlockWaves];
    __shared__ __attribute__((aligned(16))) u32x4 recA[kBlockUnits];  // {~index, value, second value, x}
    __shared__ __attribute__((aligned(8))) u32x2 recB[kBlockUnits];   // {y, z}
    __shared__ __attribute__((aligned(16))) u32x4 recC[kBlockUnits];  // {x, y, z} of the second, a bound of all others
    __shared__ __attribute__((aligned(16))) u32x4 pick_of[kBlockUnits + 1];  // {x, y, z, value}, the last one never a pick
    __shared__ Box ubox[kBlockUnits];
    __shared__ uint32_t s_above[2];  // picks above what is left
    static_assert(sizeof(sx) >= pow2_above(kCap) * sizeof(uint64_t), "keys take the coordinates' place");
    uint64_t *keys = reinterpret_cast<uint64_t *>(sx);

    const int cloud = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = a.N, want = a.M - 1;
    const float *xyz = a.xyz + (size_t)cloud * a.cloud_points * 3;
    const int32_t *sel = a.sel ? a.sel + cloud * a.sel_stride : nullptr;
    const int start = a.start_dev ? a.start_dev[cloud] : a.start;

    if (a.clear && tid < kStatusWords) a.status[tid] = 0;

    // ---- the points along the curve ----
    const int w0 = wave * kWave * P + lane;  // this lane's points in the caller's order: w0 + 64 r
    uint32_t code[P];
    {
        float rx[P], ry[P], rz[P];
        float lo[3], hi[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) { lo[k] = __builtin_inff(); hi[k] = -__builtin_inff(); }
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int i = w0 + r * kWave;
            rx[r] = ry[r] = rz[r] = 0.f;
            if (i < N) {
                const float *p = xyz + 3 * (size_t)(sel ? sel[i] : i);
                rx[r] = p[0]; ry[r] = p[1]; rz[r] = p[2];
            }
        }
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int i = w0 + r * kWave;
            if (i < N) {
                sx[i] = rx[r]; sx[kCap + i] = ry[r]; sx[2 * kCap + i] = rz[r];
                lo[0] = fminf(lo[0], rx[r]); hi[0] = fmaxf(hi[0], rx[r]);
                lo[1] = fminf(lo[1], ry[r]); hi[1] = fmaxf(hi[1], ry[r]);
                lo[2] = fminf(lo[2], rz[r]); hi[2] = fmaxf(hi[2], rz[r]);
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                lo[k] = fminf(lo[k], __shfl_xor(lo[k], o));
                hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], o));
            }
            if (lane == 0) { wbox[wave][k] = lo[k]; wbox[wave][3 + k] = hi[k]; }
        }
        cnt[wave][lane] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k)
            for (int v = 0; v < kBlockWaves; ++v) {
                lo[k] = fminf(lo[k], wbox[v][k]);
                hi[k] = fmaxf(hi[k], wbox[v][3 + k]);
            }
        const float side = fmaxf(fmaxf(hi[0] - lo[0], hi[1] - lo[1]), hi[2] - lo[2]);
        const float scale = side > 0.f ? 16.f / side : 0.f;
        const int sample = sample_index<kSplitBits>(lane, N);
        if (fills_box(sx[sample], sx[kCap + sample], sx[2 * kCap + sample], lo, side)) {
            auto cell = [&](float v, float l) { return (uint32_t)fmaxf(0.f, fminf(15.f, (v - l) * scale)); };
#pragma unroll
            for (int r = 0; r < P; ++r) code[r] = hilbert_code<4>(cell(rx[r], lo[0]), cell(ry[r], lo[1]), cell(rz[r], lo[2]));
        } else {
            if (wave < 3) {
                const Spread s = spread_of(sx[wave * kCap + sample], lane);
                if (lane == 0) part[wave] = s;
            }
            __syncthreads();
            const Spread parts[3] = {part[0], part[1], part[2]};
            const Frame f = frame_of(parts);
            if (wave == 0) {
                const uint32_t c = code_of<kCodeBits>(f, sx[sample], sx[kCap + sample], sx[2 * kCap + sample]);
                const uint32_t key = wave_sort(c << kSplitBits | (uint32_t)lane, lane);
                const uint32_t mine = lane ? key >> kSplitBits : 0u, up = (uint32_t)__shfl_down((int)(key >> kSplitBits), 1);
                split[lane] = mine;
                per_code[lane] = (float)kDigits / (float)((lane < 63 ? up : 1u << (3 * kCodeBits)) - mine);
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < P; ++r) {
                const uint32_t c = code_of<kCodeBits>(f, rx[r], ry[r], rz[r]);
                const uint32_t s = splitter_of<kSplitBits>(split, c);
                code[r] = s * kDigits + umin(kDigits - 1, (uint32_t)((float)(c - split[s]) * per_code[s]));
            }
        }
    }
    // Stable pass over six bits: elements keep the order of waves, rows and lanes.
    auto sort_pass = [&](const uint32_t (&el)[P], int shift) {
        uint32_t at[P];
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const bool ok = w0 + r * kWave < N;
            const uint32_t d = (el[r] >> shift) & (kDigits - 1);
            const uint64_t m = same_digit<6>(d, __builtin_amdgcn_ballot_w64(ok));
            at[r] = cnt[wave][d];
            const int below = lanes_below(m);
            wave_lds_order();
            if (ok && below == 0) cnt[wave][d] = at[r] + (uint32_t)__builtin_popcountll(m);
            wave_lds_order();
            at[r] += (uint32_t)below;
        }
        __syncthreads();
        // places: by digit, then by wave
        const uint32_t c = cnt[tid & 7][tid >> 3];
        uint32_t s = c;
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t v = __shfl_up(s, o);
            s += lane >= o ? v : 0u;
        }
        if (lane == 63) wsum[wave] = s;
        __syncthreads();
        uint32_t before = 0;
        for (int v = 0; v < kBlockWaves; ++v) before += v < wave ? wsum[v] : 0u;
        cnt[tid & 7][tid >> 3] = before + s - c;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < P; ++r)
            if (w0 + r * kWave < N) order[cnt[wave][(el[r] >> shift) & (kDigits - 1)] + at[r]] = el[r];
        __syncthreads();
    };
    {
        uint32_t el[P];  // code above, index below
#pragma unroll
        for (int r = 0; r < P; ++r) el[r] = (code[r] << 16) | (uint32_t)(w0 + r * kWave);
        sort_pass(el, 16);
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int i = w0 + r * kWave;
            el[r] = i < N ? order[i] : 0u;
        }
        cnt[wave][lane] = 0;
        sort_pass(el, 22);
    }

    // ---- the unit's points ----
    const int unit = tid >> 4, l16 = lane & 15;
    const int p0 = unit * N / kBlockUnits, p1 = (unit + 1) * N / kBlockUnits;
    float x[P], y[P], z[P], m[P];
    uint32_t id[P];
    Box box = no_box();
    {
        const float qx = sx[start], qy = sx[kCap + start], qz = sx[2 * kCap + start];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int at = p0 + j * 16 + l16;
            const bool ok = at < p1;
            const uint32_t i = ok ? order[at] & 0xffffu : 0u;
            x[j] = sx[i]; y[j] = sx[kCap + i]; z[j] = sx[2 * kCap + i];
            id[j] = ok ? i : kNoIndex;
            m[j] = ok ? min_dist(__builtin_inff(), sqdist(x[j], y[j], z[j], qx, qy, qz)) : 0.f;
            if (ok) box = box_or(box, Box{x[j], y[j], z[j], x[j], y[j], z[j]});
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) box = box_or(box, box_shfl_xor(box, o));
    }
    if (l16 == 0) ubox[unit] = box;
    if (tid < 2) s_above[tid] = 0;
    if (tid == 0) pick_of[kBlockUnits] = u32x4{0u, 0u, 0u, 0u};
    uint32_t pvb = 0;  // the row's largest value
    // Best point of each row, into its record.
    auto report = [&]() {
        float t1 = m[0], t2 = 0.f;
#pragma unroll
        for (int j = 1; j < P; ++j) {
            t2 = __builtin_amdgcn_fmed3f(t1, t2, m[j]);
            t1 = u2f(umax(f2u(t1), f2u(m[j])));
        }
        const uint32_t top = row_max_all(f2u(t1));
        bool win = f2u(t1) == top;
        float bx = x[0], by = y[0], bz = z[0];
        uint32_t bi = id[0];
        const bool tied = __builtin_popcountll(__builtin_amdgcn_ballot_w64(win)) != 4 ||
                          (P > 1 && __builtin_amdgcn_ballot_w64(f2u(t2) == top) != 0);
        if (!tied) {
#pragma unroll
            for (int j = 1; j < P; ++j) {
                const bool e = f2u(m[j]) == top;
                bx = e ? x[j] : bx; by = e ? y[j] : by; bz = e ? z[j] : bz;
                bi = e ? id[j] : bi;
            }
        } else {
            // equal values in a row: the lowest index
            bi = 0xffffffffu;
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const bool e = f2u(m[j]) == top && id[j] < bi;
                bx = e ? x[j] : bx; by = e ? y[j] : by; bz = e ? z[j] : bz;
                bi = e ? id[j] : bi;
            }
            const uint32_t low = ~row_max_all(~bi);
            // lanes without a point share an index: the first of the row
            const uint32_t same = row_bits(__builtin_amdgcn_ballot_w64(bi == low), lane);
            win = l16 == __builtin_ctz(same | 0x10000u);
        }
        const uint32_t rest = f2u(win ? t2 : t1), second = row_max_all(rest);
        if constexpr (kTwo) {
            if (!kTwoOfTies && tied) {
                // The others may be as large as the second, wherever that lies.  In lattices the second points release 3 picks of
                // a hundred, elsewhere 20 to 40: without looking for them 3000 points to 1500 take 819 us, with 855, 4096 to 1024 554 and 570.
                // (With two or three points per lane it is the other way round: 1500 to 700 328 without, 318 with.)
                if (l16 == 0) recC[unit] = u32x4{f2u(__builtin_inff()), f2u(__builtin_inff()), f2u(__builtin_inff()), second};
            } else {
                // Of equal seconds any will do: the third value is the same then.  So it is taken to be where a lane
                // holds the two best: its own third value is not known.
                const bool win2 = l16 == __builtin_ctz(row_bits(__builtin_amdgcn_ballot_w64(rest == second), lane) | 0x10000u);
                const uint32_t third = row_max_all(win2 ? f2u(t2) : rest);
                float cx = x[0], cy = y[0], cz = z[0];
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    const bool e = f2u(m[j]) == second;
                    cx = e ? x[j] : cx; cy = e ? y[j] : cy; cz = e ? z[j] : cz;
                }
                if (win2) recC[unit] = u32x4{f2u(cx), f2u(cy), f2u(cz), third};
            }
        }
        pvb = top;
        if (win) {
            recA[unit] = u32x4{~bi, top, second, f2u(bx)};
            recB[unit] = u32x2{f2u(by), f2u(bz)};
        }
    };
    __syncthreads();  // boxes; the coordinates are done with
    // A lane looks after two units, of the half of the curve around its wave and of the other half.
    const int base = (wave * 4 + kBlockUnits - 6) & (kBlockUnits - 1);
    const int u0 = (base + l16) & (kBlockUnits - 1), u1 = u0 ^ 16;
    const Box b0 = ubox[u0], b1 = ubox[u1];
    const uint32_t g1 = f2u(box_box(box, b1));  // not above the distance of any two of their points
    report();

    // ---- rounds ----
    uint64_t *mine = keys + p0;  // a unit lists its picks where its points are
    const int n_mine = p1 - p0;
    int n_list = 0, np = 0;
    uint32_t round = 0;
    bool bad = false;
    for (;;) {
        ++round;
        const uint32_t par = round & 1;
        wg_barrier();  // records
        const bool far = !FAR || __builtin_amdgcn_ballot_w64(g1 < pvb) != 0;  // a unit of the other half may matter
        const u32x4 rA = recA[unit], a0 = recA[u0], d0 = recC[u0];
        const u32x2 rB = recB[unit], c0 = recB[u0];
        const float pv = u2f(pvb), px = u2f(rA.w), py = u2f(rB.x), pz = u2f(rB.y);
        const uint64_t kp = key_of(rA);
        auto holds = [&](const u32x4 &A, const u32x2 &B, const u32x4 &C, const Box &b) {
            const bool first = sqdist(u2f(A.w), u2f(B.x), u2f(B.y), px, py, pz) < pv, near = box_dist(b, px, py, pz) < pv;
            if constexpr (kTwo)
                return (key_of(A) > kp) & (first | ((A.z >= pvb) & (sqdist(u2f(C.x), u2f(C.y), u2f(C.z), px, py, pz) < pv)) |
                                           ((C.w >= pvb) & near));
            else
                return (key_of(A) > kp) & (first | ((A.z >= pvb) & near));
        };
        bool held;
        if (far) {
            const u32x4 a1 = recA[u1], d1 = recC[u1];
            const u32x2 c1 = recB[u1];
            held = holds(a0, c0, d0, b0) | holds(a1, c1, d1, b1);
        } else {
            held = holds(a0, c0, d0, b0);
        }
        const bool pick = (pvb != 0u) & (n_list < n_mine) & (row_bits(__builtin_amdgcn_ballot_w64(held), lane) == 0u);
        if (l16 == 0) {
            pick_of[unit] = u32x4{f2u(px), f2u(py), f2u(pz), pick ? pvb : 0u};
            if (pick) mine[n_list] = kp;
        }
        const bool counting = np >= want;
        if (counting) {
            // picks (of the rounds before) above everything that is left
            const uint32_t left = row_max_all(umax(recA[l16].y, recA[l16 + 16].y));
            uint32_t n = 0;
            for (int k = l16; k < n_list; k += 16) n += (uint32_t)(mine[k] >> 32) > left ? 1u : 0u;
            uint32_t t = 0;
            for (int b = 0; b < 5; ++b) t += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((n >> b) & 1u)) << b;
            if (lane == 0 && t) atomicAdd(&s_above[par], t);
        }
        n_list += pick ? 1 : 0;
        wg_barrier();  // picks
        const u32x4 q0 = pick_of[u0], q1 = pick_of[u1];
        // a row looks at all units
        const int made = __builtin_popcount((uint32_t)__builtin_amdgcn_ballot_w64(q0.w != 0u) & 0xffffu) +
                         __builtin_popcount((uint32_t)__builtin_amdgcn_ballot_w64(q1.w != 0u) & 0xffffu);
        if (counting && s_above[par] >= (uint32_t)want) {
            n_list -= pick ? 1 : 0;  // the picks of this round are not needed
            break;
        }
        if (made == 0) {
            // no value is left, or (coordinates that are not finite) a point was picked twice
            bad = pvb != 0u;
            break;
        }
        np += made;
        if (tid == 0) s_above[par ^ 1] = 0;
        // ---- apply what reaches the unit's box ----
        auto reaches = [&](const u32x4 &q) {
            return box_dist(box, u2f(q.x), u2f(q.y), u2f(q.z)) < u2f(umin(pvb, q.w));
        };
        uint32_t hits = row_bits(__builtin_amdgcn_ballot_w64(reaches(q0)), lane);
        if (far) hits |= row_bits(__builtin_amdgcn_ballot_w64(reaches(q1)), lane) << 16;
        if (__builtin_amdgcn_ballot_w64(hits != 0) == 0) continue;
        do {
            const int h0 = hits ? (base + __builtin_ctz(hits)) & (kBlockUnits - 1) : kBlockUnits;
            hits &= hits - 1;
            const int h1 = hits ? (base + __builtin_ctz(hits)) & (kBlockUnits - 1) : kBlockUnits;
            hits &= hits - 1;
            const u32x4 e = pick_of[h0], f = pick_of[h1];
#pragma unroll
            for (int j = 0; j < P; ++j) {
                float d = sqdist(x[j], y[j], z[j], u2f(e.x), u2f(e.y), u2f(e.z));
                float g = sqdist(x[j], y[j], z[j], u2f(f.x), u2f(f.y), u2f(f.z));
                d = d < u2f(e.w) ? d : __builtin_inff();
                g = g < u2f(f.w) ? g : __builtin_inff();
                m[j] = min3_dist(m[j], d, g);
            }
        } while (__builtin_amdgcn_ballot_w64(hits != 0) != 0);
        report();
    }

    // ---- the picks in their order ----
    // Into bins over the range of their values, largest first; a pick's place is that of its bin
    // plus the picks of the bin before it.  (The bitonic sort below, for many picks of nearly one
    // value, takes 14 us of a cloud of 1024 points by itself.)
    __syncthreads();
    uint64_t *binned = keys + kCap;
    uint32_t vlo = 0xffffffffu, vhi = 0u;
    for (int k = l16; k < n_list; k += 16) {
        const uint32_t v = (uint32_t)(mine[k] >> 32);
        vlo = umin(vlo, v);
        vhi = umax(vhi, v);
    }
    vlo = wave_min_u32(vlo);
    vhi = wave_max_u32(vhi);
    if (lane == 0) { wsum[wave] = vlo; wtop[wave] = vhi; }
    for (int k = tid; k < kBins; k += kBlockThreads) bins[k] = 0u;
    __syncthreads();
    for (int v = 0; v < kBlockWaves; ++v) { vlo = umin(vlo, wsum[v]); vhi = umax(vhi, wtop[v]); }
    const float per = (float)(kBins - 1) / (float)(vhi - vlo + 1u);
    auto bin_of = [&](uint64_t key) { return min(kBins - 1, (int)((float)(vhi - (uint32_t)(key >> 32)) * per)); };
    uint32_t place[P];
#pragma unroll
    for (int r = 0; r < P; ++r) {
        const int k = l16 + r * 16;
        place[r] = k < n_list ? atomicAdd(&bins[bin_of(mine[k])], 1u) : 0u;
    }
    __syncthreads();
    uint32_t c[4], sum = 0, most = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) { c[k] = bins[4 * tid + k]; sum += c[k]; most = umax(most, c[k]); }
    uint32_t incl = sum;
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o);
        incl += lane >= o ? v : 0u;
    }
    most = wave_max_u32(most);
    if (lane == 63) { wsum[wave] = incl; wtop[wave] = most; }
    __syncthreads();
    uint32_t at0 = incl - sum;
    for (int v = 0; v < kBlockWaves; ++v) { at0 += v < wave ? wsum[v] : 0u; most = umax(most, wtop[v]); }
#pragma unroll
    for (int k = 0; k < 4; ++k) { bins[4 * tid + k] = at0; at0 += c[k]; }
    __syncthreads();
    int32_t *idx = a.idx + cloud * a.idx_stride;
    float *md = a.md ? a.md + cloud * a.md_stride : nullptr;
    if (tid == 0) {
        idx[0] = sel ? sel[start] : start;
        if (md) md[0] = __builtin_inff();
        __hip_atomic_fetch_max(a.status + 1, (int)round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (bad && l16 == 0) note_inconsistent(a.status, (int)round);
    auto put = [&](int i, uint64_t key) {
        if (i >= want) return;
        const int at = (int)~(uint32_t)key;
        idx[1 + i] = sel ? sel[at] : at;
        if (md) md[1 + i] = u2f((uint32_t)(key >> 32));
    };
    for (int i = np + tid; i < want; i += kBlockThreads) put(i, 0xffffffffull);  // every value is 0: point 0 again
#pragma unroll
    for (int r = 0; r < P; ++r) {
        const int k = l16 + r * 16;
        if (k < n_list) {
            const uint64_t key = mine[k];
            binned[bins[bin_of(key)] + place[r]] = key;
        }
    }
    __syncthreads();
    if (most <= kBinMax) {
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int k = tid + r * kBlockThreads;
            if (k < np) {
                const uint64_t key = binned[k];
                const int b = bin_of(key);
                const int e0 = (int)bins[b], e1 = b + 1 < kBins ? (int)bins[b + 1] : np;
                int i = e0;
                for (int e = e0; e < e1; ++e) i += binned[e] > key ? 1 : 0;
                put(i, key);
            }
        }
        return;
    }
    for (int i = tid; i < np; i += kBlockThreads) keys[i] = binned[i];
    __syncthreads();
    int size = 2;
    while (size < np) size <<= 1;
    for (int i = np + tid; i < size; i += kBlockThreads) keys[i] = 0ull;
    __syncthreads();
    for (int k = 2; k <= size; k <<= 1) {
        for (int o = k >> 1; o > 0; o >>= 1) {
            for (int i = tid; i < size / 2; i += kBlockThreads) {
                const int p = 2 * i - (i & (o - 1)), q = p + o;
                const uint64_t u = keys[p], v = keys[q];
                const bool up = (p & k) != 0;  // ascending half
                if ((u < v) != up) { keys[p] = v; keys[q] = u; }
            }
            // up to a distance of 64 a wave stays within 128 keys of its own
            if (o > kWave || (o == 1 && k >= 2 * kWave)) wg_barrier();
            else wave_lds_order();
        }
    }
    __syncthreads();
    for (int i = tid; i < np; i += kBlockThreads) put(i, keys[i]);
}

template <int P>
hipError_t launch_t(const BlockArgs &a, int B, hipStream_t s) {
    // more points per lane fill a CU's LDS; fewer gain nothing (one) or spill (two: 768 clouds of 700 3 % slower)
    constexpr bool kSeveral = P >= 3 && P <= 8;
    if (kSeveral && B > kOnePerCu)
        k_fps_block<P, kSeveral><<<dim3(B), dim3(kBlockThreads), 0, s>>>(a);
    else
        k_fps_block<P, false><<<dim3(B), dim3(kBlockThreads), 0, s>>>(a);
    return hipGetLastError();
}

// Points per lane.
#define FFPS_BLOCK_ROWS(X) X(1) X(2) X(3) X(4) X(6) X(8) X(9) X(12) X(16)

}  // namespace

int block_capacity() { return kBlockThreads * 16; }

hipError_t launch_fps_block(const BlockArgs &a, int B, hipStream_t s) {
    if (a.N < kBlockUnits) return hipErrorInvalidValue;
    const int rows = (a.N + kBlockThreads - 1) / kBlockThreads;
#define X(R) if (rows <= (R)) return launch_t<R>(a, B, s);
    FFPS_BLOCK_ROWS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace ffps
