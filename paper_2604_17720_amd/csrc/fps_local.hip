// k_fps_local: exact FPS (Sec. 3.1, Eq. 1) of clouds spread over many CUs by LOCAL MAXIMA.
//
// Write v(p) for the running minimum squared distance of p and let "p before q" mean
// that p precedes q in the order (value descending, index ascending).  A point p whose
// open ball { q : d(p, q) < v(p) } holds no point before p is certain to be picked, with
// exactly the value v(p): picks outside the ball cannot lower p, and a point of the
// ball would have to come before p to be picked first.  All such points of a cloud can be
// picked at once, however far apart their values are.  A pick q only ever matters to
// points with d(p, q) < v(q): a point before q is not nearer to it than v(q), and whatever
// falls behind q later has a smaller value than that distance.  So picks may be applied in any
// order, at any time and more than once, and judging by values that are out of date is
// merely cautious (values never grow).  The samples are the picks sorted by (value descending,
// index ascending), which is the order in which the greedy loop makes them.
//
// Where the time of the loop in fps_grid.hip goes into rounds of about a hundred picks each
// (462 for 50,000 of 200,000 points) and into applying every pick to every point, here a
// round makes as many picks as there are separate maxima (348 on average, 169 rounds)
// and a pick is applied where it can matter: about 130 distances per point, not 50,000.
// What is left is the latency of a round, which is what everything below is about.
//
//   - Points are sorted along a space-filling curve first (spatial.hip); a UNIT, one
//     wave, holds a stretch of it in registers (up to 40 rows of 64 points), eight units
//     make a workgroup.  From 12 rows on registers are spilled: 6 there, 32 at 16 rows, 52 at 24,
//     149 at 32 and 228 at 40 (compiled with the build's flags).  With the boxes in LDS, records gathered two
//     slots at a time and the rows kept in their order (few_rows), all beyond 16 rows, a round of
//     five million points takes 10 us, 21 without.
//   - Per round a unit publishes its best point (value, index, coordinates), the value of
//     its second best, and whether the candidate it published the round before was picked:
//     32 bytes.  Every lane reads the records of up to four units, eight lanes for a
//     workgroup, those of neighbouring workgroups in different waves.
//   - A workgroup needs the records of another only while the distance of their points is
//     below the larger of their largest values.  Both sides see the same records and drop
//     each other in the same round, so late rounds exchange with a few neighbours and
//     neighbourhoods far apart may be many rounds apart.
//   - A candidate is a pick when no unit holds a point before it in its ball: a unit does
//     not if its best comes later, if its box lies outside, or if its second best is too
//     small and its best lies outside.
//   - A workgroup stops when as many picks as samples have values in bins above that
//     of its largest value: nothing it holds can belong to the samples any more.  Picks
//     beyond the samples are left out by the final sort (spatial.hip): 18 % more than the 50,000 of a
//     room, 45 % more than 5001 of 45,678, 37 % more than 16,384 of a LiDAR frame.
//
// Measured, exact FPS of a room of 200,000 points to 50,000 samples, sorts included:
// 0.82 ms against 4.44 ms with k_fps_grid; 45,678 points to 5,001: 0.42 against 0.84 ms;
// five million to 1024: 1.2 ms against 4.7 ms with k_fps_stream.
//
// Every wait is bounded as in fps_exchange.h.  A point that is picked twice (coordinates that are not
// finite) ends the workgroup with the status of inconsistent results; those that wait for it look at the
// status now and then and leave, too.
#include "fps_exchange.h"
#include "fps_local.h"
#include "fps_space.h"

namespace ffps {

namespace {

constexpr int kWaves = 8;  // units of a workgroup, two waves per SIMD
constexpr int kThreads = kWaves * kWave;
// A 16-byte chunk is three words and the exclusive or of them with a constant of its kind and
// the round: cleared memory stands for no round, and a chunk two rounds old (the buffer
// alternates) is told from a new one.
constexpr uint32_t kTagA = 0x9E3779B1u, kTagB = 0x85EBCA6Bu, kTagBox = 0x5F356495u;
constexpr uint32_t kTagWindow = 1u << 20;  // "this round or a later one"
constexpr int kPollsPerLook = 1024;        // at records that are missing, between two looks at the status

__device__ __forceinline__ uint32_t chunk_round(const u32x4 &c, uint32_t which) { return c.x ^ c.y ^ c.z ^ c.w ^ which; }

struct LocalArgs {
    const float *xyz;     // [clouds][N][3] as the caller has them, for the first sample
    const u32x4 *pts;     // [clouds][N] along the curve: {x, y, z, index}
    int N, M, start;
    const int *start_dev;
    int G;                // workgroups per cloud
    char *exchange;       // per cloud 8 planes of 16 bytes per unit, cleared
    u32x4 *picks;         // [clouds][N]: a unit lists its picks where its points are: {value, index, round, -}
    int *npicks;          // [clouds][units]
    uint32_t *hist;       // [clouds][kLocalWords], cleared: picks per bin, picks per unit so far
    int *status;
    int spin_limit;
};

// unsigned maximum over eight consecutive lanes, in each of them
__device__ __forceinline__ uint32_t eight_max_all(uint32_t v) {
    v = umax(v, dpp_or_zero<0xB1>(v));   // quad_perm 1,0,3,2
    v = umax(v, dpp_or_zero<0x4E>(v));   // quad_perm 2,3,0,1
    v = umax(v, dpp_or_zero<0x141>(v));  // row_half_mirror
    return v;
}

__device__ __forceinline__ Box box_shfl(const Box &a, int l) {
    return Box{__shfl(a.lx, l), __shfl(a.ly, l), __shfl(a.lz, l), __shfl(a.hx, l), __shfl(a.hy, l), __shfl(a.hz, l)};
}
// Records of this lane's slots: 16 bytes at `base` + off and 16 at `base2` + off, read past the caches
// that are not shared by the whole device.
template <int NS>
__device__ __forceinline__ void load_pairs(const char *base, const char *base2, const uint32_t (&off)[4], u32x4 (&ra)[4], u32x4 (&rb)[4]) {
    if constexpr (NS == 1) {
        asm volatile("global_load_dwordx4 %0, %2, %3 sc1\n\tglobal_load_dwordx4 %1, %2, %4 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(ra[0]), "=&v"(rb[0]) : "v"(off[0]), "s"(base), "s"(base2) : "memory");
    } else if constexpr (NS == 2) {
        asm volatile("global_load_dwordx4 %0, %4, %6 sc1\n\tglobal_load_dwordx4 %1, %4, %7 sc1\n\t"
                     "global_load_dwordx4 %2, %5, %6 sc1\n\tglobal_load_dwordx4 %3, %5, %7 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(ra[0]), "=&v"(rb[0]), "=&v"(ra[1]), "=&v"(rb[1])
                     : "v"(off[0]), "v"(off[1]), "s"(base), "s"(base2) : "memory");
    } else {
        static_assert(NS == 4, "");
        asm volatile("global_load_dwordx4 %0, %8, %12 sc1\n\tglobal_load_dwordx4 %1, %8, %13 sc1\n\t"
                     "global_load_dwordx4 %2, %9, %12 sc1\n\tglobal_load_dwordx4 %3, %9, %13 sc1\n\t"
                     "global_load_dwordx4 %4, %10, %12 sc1\n\tglobal_load_dwordx4 %5, %10, %13 sc1\n\t"
                     "global_load_dwordx4 %6, %11, %12 sc1\n\tglobal_load_dwordx4 %7, %11, %13 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(ra[0]), "=&v"(rb[0]), "=&v"(ra[1]), "=&v"(rb[1]), "=&v"(ra[2]), "=&v"(rb[2]), "=&v"(ra[3]), "=&v"(rb[3])
                     : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "s"(base2) : "memory");
    }
}

// Where a lane has many points, every few rows the compiler may not mix with those before them: its
// own order would hold the results of dozens of rows at once and spill the points.
template <int P>
__device__ __forceinline__ void few_rows(int j) {
    if (P > 16 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
}

// the best point of a unit and the value that follows it, the same in all lanes of the unit
struct Best {
    float v, sec, x, y, z;
    uint32_t i;
};

// Point indices of a lane: in registers, or read again where a lane has many points (only the
// index of a unit's best point is ever needed).
constexpr int kRegIndexRows = 16;
template <int P>
struct Indices {
    static constexpr bool kKept = P <= kRegIndexRows;
    uint32_t r[kKept ? P : 1];
    const u32x4 *pts;  // first point of the unit
    int n, lane;       // points of the unit
    __device__ __forceinline__ void set(int j, uint32_t v) { if constexpr (kKept) r[j] = v; }
    __device__ __forceinline__ uint32_t at(int j) const {
        if constexpr (kKept) return r[j];
        const int i = j * kWave + lane;
        return i < n ? reinterpret_cast<const uint32_t *>(pts + i)[3] : kNoIndex;
    }
    __device__ __forceinline__ uint32_t of(int j, int l) const {  // wave-uniform row and lane
        const int i = j * kWave + l;
        return i < n ? reinterpret_cast<const uint32_t *>(pts + i)[3] : kNoIndex;
    }
};

// A workgroup's points as two boxes: the sixteen boxes (two per unit, lane l mod 8 holding
// those of unit l) in order, cut where two neighbours are farthest apart.
__device__ __forceinline__ void two_boxes(const Box &A, const Box &B, int lane, Box &w1, Box &w2) {
    const int l = lane & 7;
    const Box nx = box_shfl(A, (lane & 56) + ((l + 1) & 7));
    const float g0 = box_box(A, B), g1 = l < 7 ? box_box(B, nx) : 0.f;
    const float g = fmaxf(g0, g1);
    const float top = u2f(eight_max_all(f2u(g)));
    int pos = 7;  // no gap at all: halves
    if (top > 0.f) {
        uint32_t c = g == top ? (uint32_t)(g0 == top ? 2 * l : 2 * l + 1) : 63u;
        c = 63u - eight_max_all(63u - c);
        pos = (int)c;
    }
    w1 = box_or(2 * l <= pos ? A : no_box(), 2 * l + 1 <= pos ? B : no_box());
    w2 = box_or(2 * l > pos ? A : no_box(), 2 * l + 1 > pos ? B : no_box());
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
        w1 = box_or(w1, box_shfl_xor(w1, o));
        w2 = box_or(w2, box_shfl_xor(w2, o));
    }
}

template <int P>
__device__ __forceinline__ Best unit_best(const float (&x)[P], const float (&y)[P], const float (&z)[P], const float (&m)[P],
                                          const Indices<P> &id, int lane) {
    Best b;
    float t1 = m[0], t2 = 0.f;
#pragma unroll
    for (int j = 1; j < P; ++j) {
        t2 = __builtin_amdgcn_fmed3f(t1, t2, m[j]);
        t1 = fmaxf(t1, m[j]);
        few_rows<P>(j);
    }
    const uint32_t T1 = wave_max_u32(f2u(t1));
    uint64_t own = __builtin_amdgcn_ballot_w64(f2u(t1) == T1);
    b.v = u2f(T1);
    int jr = 0;
#pragma unroll
    for (int j = P - 1; j > 0; --j) jr = f2u(m[j]) == T1 ? j : jr;
    if constexpr (P > 1) jr = f2u(m[0]) == T1 ? 0 : jr;
    if (__builtin_popcountll(own) != 1 || (P > 1 && __builtin_amdgcn_ballot_w64(f2u(t2) == T1) != 0)) {
        // equal values: the lowest index
        uint32_t mi = 0xffffffffu;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const uint32_t i = id.at(j);
            const bool e = f2u(m[j]) == T1 && i < mi;
            mi = e ? i : mi;
            jr = e ? j : jr;
            few_rows<P>(j);
        }
        const uint32_t lo = wave_min_u32(mi);
        own = __builtin_amdgcn_ballot_w64(mi == lo);
    }
    const int wl = (int)__builtin_ctzll(own);
    b.sec = u2f(wave_max_u32(lane == wl ? f2u(t2) : f2u(t1)));
    if constexpr (P > 4) {
        const int row = readlane_i(jr, wl);
        pick_xyz<P>(x, y, z, row, wl, b.x, b.y, b.z);
        if constexpr (Indices<P>::kKept) {
            uint32_t bi = 0;
#pragma unroll
            for (int j = 0; j < P; ++j)
                if (row == j) bi = (uint32_t)readlane_i((int)id.at(j), wl);
            b.i = bi;
        } else {
            b.i = id.of(row, wl);
        }
    } else {
        float bx = x[0], by = y[0], bz = z[0];
        uint32_t bi = id.at(0);
#pragma unroll
        for (int j = 1; j < P; ++j) {
            bx = jr == j ? x[j] : bx; by = jr == j ? y[j] : by; bz = jr == j ? z[j] : bz;
            bi = jr == j ? id.at(j) : bi;
        }
        b.x = readlane_f(bx, wl); b.y = readlane_f(by, wl); b.z = readlane_f(bz, wl);
        b.i = (uint32_t)readlane_i((int)bi, wl);
    }
    return b;
}

// Rows up to which the records of four slots are gathered at once; beyond, the registers that
// takes are dearer than a second wait (at 24 to 40 rows; 12 and 16 rows, which spill a few, were not tried).
constexpr int kGatherRows = 16;

template <int P>
__global__ __launch_bounds__(kThreads, 2) void k_fps_local(LocalArgs a) {
    constexpr int kSlots = 4;
    constexpr int kList = kSlots * kThreads;
    __shared__ __attribute__((aligned(16))) u32x4 plist[kList];     // new picks that may matter here
    __shared__ __attribute__((aligned(16))) u32x4 rlist[kList][2];  // units that may hold a candidate back
    __shared__ Box sbox[kList];                                     // boxes of all units
    __shared__ u32x4 candA[kWaves], candB[kWaves];
    __shared__ Box ubox[kWaves], boxA[kWaves], boxB[kWaves];  // a unit's two boxes and their union
    __shared__ Box wboxes[2];                                 // the workgroup's two boxes
    __shared__ uint32_t s_n[2], s_sum[2], s_bad, s_twice, s_wv[2];

    const int G = a.G, U = G * kWaves;
    const int cloud = blockIdx.x / G, w = blockIdx.x - cloud * G;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = w * kWaves + wave;
    const u32x4 *pts = a.pts + (size_t)cloud * a.N;
    char *ex = a.exchange + (size_t)cloud * 8 * U * 16;
    const size_t plane = (size_t)U * 16;  // boxes: planes 0 to 3; records: planes 4, 5 (even rounds) and 6, 7
    uint32_t *hist = a.hist + (size_t)cloud * kLocalWords, *count = hist + kLocalBins;
    const int start = a.start_dev ? a.start_dev[cloud] : a.start;

    // ---- points of this unit ----
    const int p0 = (int)((long)unit * a.N / U), p1 = (int)((long)(unit + 1) * a.N / U);
    u32x4 *picks = a.picks + (size_t)cloud * a.N + p0;
    int np = 0;  // picks of this unit in its list
    float x[P], y[P], z[P], m[P];
    Indices<P> id;
    id.pts = pts + p0;
    id.n = p1 - p0;
    id.lane = lane;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        const int i = p0 + j * kWave + lane;
        const bool ok = i < p1;
        u32x4 p = {0u, 0u, 0u, kNoIndex};
        if (ok) p = pts[i];
        x[j] = u2f(p.x); y[j] = u2f(p.y); z[j] = u2f(p.z);
        id.set(j, p.w);
        m[j] = ok ? __builtin_inff() : 0.f;
        few_rows<P>(j);
    }
    // The unit's points in their order as two boxes, cut at the widest step: the order jumps
    // now and then, and one box around both ends of a jump would be met by most picks.
    Box ba = no_box(), bb = no_box();
    {
        float g = 0.f;
        int at = p0 + (p1 - p0) / 2;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = p0 + j * kWave + lane;
            float nx = __shfl(x[j], (lane + 1) & 63), ny = __shfl(y[j], (lane + 1) & 63), nz = __shfl(z[j], (lane + 1) & 63);
            if (j + 1 < P) {
                const float fx = readlane_f(x[j + 1 < P ? j + 1 : j], 0), fy = readlane_f(y[j + 1 < P ? j + 1 : j], 0), fz = readlane_f(z[j + 1 < P ? j + 1 : j], 0);
                nx = lane == 63 ? fx : nx; ny = lane == 63 ? fy : ny; nz = lane == 63 ? fz : nz;
            }
            const float d = i + 1 < p1 ? sqdist(x[j], y[j], z[j], nx, ny, nz) : 0.f;
            at = d > g ? i : at;
            g = fmaxf(g, d);
            few_rows<P>(j);
        }
        const uint32_t top = wave_max_u32(f2u(g));
        at = readlane_i(at, first_lane(f2u(g) == top));
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = p0 + j * kWave + lane;
            const Box o = {x[j], y[j], z[j], x[j], y[j], z[j]};
            if (i < p1 && i <= at) ba = box_or(ba, o);
            if (i < p1 && i > at) bb = box_or(bb, o);
            few_rows<P>(j);
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            ba = box_or(ba, box_shfl_xor(ba, o));
            bb = box_or(bb, box_shfl_xor(bb, o));
        }
    }
    auto apply = [&](float qx, float qy, float qz, float qv) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const float d = sqdist(x[j], y[j], z[j], qx, qy, qz);
            m[j] = min_dist(m[j], d < qv ? d : __builtin_inff());
            few_rows<P>(j);
        }
    };
    {
        const float *q = a.xyz + ((size_t)cloud * a.N + start) * 3;
        apply(q[0], q[1], q[2], __builtin_inff());
    }
    Best best = unit_best<P>(x, y, z, m, id, lane);
    auto publish = [&](uint32_t round, bool picked, bool stopped) {
        if (lane == 0) {
            char *buf = ex + plane * (4 + 2 * (round & 1)) + (size_t)unit * 16;
            u32x4 A, B;
            A.x = f2u(best.v) | (stopped ? 0x80000000u : 0u);
            A.y = best.i | (picked ? 0x80000000u : 0u);
            A.z = f2u(best.sec);
            A.w = A.x ^ A.y ^ A.z ^ kTagA ^ round;
            B.x = f2u(best.x); B.y = f2u(best.y); B.z = f2u(best.z);
            B.w = B.x ^ B.y ^ B.z ^ kTagB ^ round;
            store_chunk(buf, A);
            store_chunk(buf + plane, B);
            candA[wave] = u32x4{f2u(best.v), best.i, f2u(best.sec), 0u};
            candB[wave] = B;
        }
    };
    if (lane == 0) {
        auto put = [&](int k, float c0, float c1, float c2) {
            u32x4 A = {f2u(c0), f2u(c1), f2u(c2), 0u};
            A.w = A.x ^ A.y ^ A.z ^ kTagBox ^ (uint32_t)(k + 1);
            store_chunk(ex + plane * k + (size_t)unit * 16, A);
        };
        put(0, ba.lx, ba.ly, ba.lz); put(1, ba.hx, ba.hy, ba.hz);
        put(2, bb.lx, bb.ly, bb.lz); put(3, bb.hx, bb.hy, bb.hz);
        boxA[wave] = ba;
        boxB[wave] = bb;
        ubox[wave] = box_or(ba, bb);
    }
    publish(1, false, false);
    if (tid < 2) s_n[tid] = s_sum[tid] = s_wv[tid] = 0;
    if (tid == 0) s_bad = s_twice = 0;

    // ---- slots: the units this lane keeps track of, eight lanes per workgroup ----
    float wd[kSlots], ud[kSlots];   // distance of its workgroup's box, and of its own, from this workgroup's box
    float gv[kSlots];               // largest value of its workgroup (found twice where registers are short)
    float sv[kSlots], ss[kSlots], sx[kSlots], sy[kSlots], sz[kSlots];
    uint32_t si[kSlots], off[kSlots];
    uint32_t fl[kSlots];            // 1: wanted, 2: waited for, 4: stopped, 8: this workgroup's own
    int cur = U > 2 * kThreads ? 4 : U > kThreads ? 2 : 1;  // slots in use by this wave
    bool bad = false;
    __syncthreads();
    Box w1, w2;  // the workgroup's points
    two_boxes(boxA[lane & 7], boxB[lane & 7], lane, w1, w2);
    if (tid == 0) { wboxes[0] = w1; wboxes[1] = w2; }
    // many points in registers: the boxes are read again where they are needed
    constexpr bool kBoxesInLds = P > kGatherRows;
    auto unit_dist = [&](float qx, float qy, float qz) {
        if constexpr (kBoxesInLds) return fminf(box_dist(boxA[wave], qx, qy, qz), box_dist(boxB[wave], qx, qy, qz));
        else return fminf(box_dist(ba, qx, qy, qz), box_dist(bb, qx, qy, qz));
    };
    auto group_dist = [&](float qx, float qy, float qz) {
        if constexpr (kBoxesInLds) return fminf(box_dist(wboxes[0], qx, qy, qz), box_dist(wboxes[1], qx, qy, qz));
        else return fminf(box_dist(w1, qx, qy, qz), box_dist(w2, qx, qy, qz));
    };
    auto find_units = [&](auto tag, auto first) {
        constexpr int NS = decltype(tag)::value, Q0 = decltype(first)::value;
        u32x4 ra[4], rb[4], rc[4], rd[4];
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            // workgroup q * 64 + (lane / 8) * 8 + wave: neighbours along the order go to different waves
            const int g = (Q0 + q) * 64 + (lane >> 3) * 8 + wave;
            const bool ok = g < G;
            o[q] = off[Q0 + q] = (uint32_t)(ok ? g * 8 + (lane & 7) : unit) * 16;
            fl[Q0 + q] = (ok ? 3u : 0u) | (g == w ? 8u : 0u);
        }
        for (int spin = 0;; ++spin) {
            load_pairs<NS>(ex, ex + plane, o, ra, rb);
            load_pairs<NS>(ex + 2 * plane, ex + 3 * plane, o, rc, rd);
            bool all = true;
#pragma unroll
            for (int q = 0; q < NS; ++q)
                all = all && chunk_round(ra[q], kTagBox) == 1u && chunk_round(rb[q], kTagBox) == 2u &&
                      chunk_round(rc[q], kTagBox) == 3u && chunk_round(rd[q], kTagBox) == 4u;
            if (__builtin_amdgcn_ballot_w64(!all) == 0) break;
            if (spin >= a.spin_limit) { bad = true; break; }
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const Box A = {u2f(ra[q].x), u2f(ra[q].y), u2f(ra[q].z), u2f(rb[q].x), u2f(rb[q].y), u2f(rb[q].z)};
            const Box B = {u2f(rc[q].x), u2f(rc[q].y), u2f(rc[q].z), u2f(rd[q].x), u2f(rd[q].y), u2f(rd[q].z)};
            const int s = Q0 + q;
            if (fl[s] & 1u) sbox[off[s] >> 4] = box_or(A, B);
            ud[s] = fminf(fminf(box_box(w1, A), box_box(w1, B)), fminf(box_box(w2, A), box_box(w2, B)));
            Box o1, o2;
            two_boxes(A, B, lane, o1, o2);
            wd[s] = fminf(fminf(box_box(w1, o1), box_box(w1, o2)), fminf(box_box(w2, o1), box_box(w2, o2)));
            sv[s] = ss[s] = 0.f; sx[s] = sy[s] = sz[s] = 0.f; si[s] = kNoIndex;
        }
    };
    constexpr std::integral_constant<int, 0> s0;
    constexpr std::integral_constant<int, 1> s1;
    constexpr std::integral_constant<int, 2> s2;
    constexpr std::integral_constant<int, 3> s3;
    if constexpr (kBoxesInLds) {
        find_units(s1, s0); find_units(s1, s1); find_units(s1, s2); find_units(s1, s3);
    } else {
        find_units(std::integral_constant<int, 4>{}, s0);
    }
    uint32_t maxbin = 0;
    float wv = __builtin_inff();  // largest value of this workgroup's points
    bool logged = true;           // the unit's last pick is in the list
    float lv = 0.f;
    uint32_t li = 0;
    uint32_t round = 1;
    bool enough = false;    // as many picks as samples, not counting which
    uint32_t open = 0;      // bit c: candidate c is not held back by a unit of this workgroup
    float thr = 0.f;        // the smallest value among those
    // Gathers the records of this round and adds to the two lists.
    auto gather = [&](auto tag, auto first) {
        constexpr int NS = decltype(tag)::value, Q0 = decltype(first)::value;
        u32x4 ra[4], rb[4];
        const uint32_t par = round & 1;
        {
            const char *buf = ex + plane * (4 + 2 * par);
            uint32_t o[4];
#pragma unroll
            for (int q = 0; q < NS; ++q) o[q] = (fl[Q0 + q] & 6u) == 2u ? off[Q0 + q] : (uint32_t)unit * 16;
            auto missing = [&](int q) {
                const uint32_t da = chunk_round(ra[q], kTagA) - round, db = chunk_round(rb[q], kTagB) - round;
                const bool ok = (fl[Q0 + q] & 1u) ? (da | db) == 0u : da < kTagWindow;
                return !ok && (fl[Q0 + q] & 6u) == 2u;
            };
            load_pairs<NS>(buf, buf + plane, o, ra, rb);
            for (int spin = 0;; ++spin) {
                bool any = false;
                bool ms[NS];
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    ms[q] = missing(q);
                    any = any || ms[q];
                }
                if (__builtin_amdgcn_ballot_w64(any) == 0) break;
                if (spin >= a.spin_limit || ((spin & (kPollsPerLook - 1)) == kPollsPerLook - 1 &&
                                             __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    bad = true;
                    break;
                }
                // only what is missing is read again: polling everything would be in the way of
                // those who are waited for
                u32x4 ta[4], tb[4];
#pragma unroll
                for (int q = 0; q < NS; ++q) o[q] = ms[q] ? off[Q0 + q] : (uint32_t)unit * 16;
                load_pairs<NS>(buf, buf + plane, o, ta, tb);
#pragma unroll
                for (int q = 0; q < NS; ++q)
                    if (ms[q]) { ra[q] = ta[q]; rb[q] = tb[q]; }
            }
        }
        bool pk[NS], rel[NS];
        uint64_t pm[NS], rm[NS];
        u32x4 pe[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const bool use = (fl[Q0 + q] & 5u) == 1u;
            pe[q] = u32x4{f2u(sx[Q0 + q]), f2u(sy[Q0 + q]), f2u(sz[Q0 + q]), f2u(sv[Q0 + q])};
            pk[q] = use && (ra[q].y & 0x80000000u) && group_dist(sx[Q0 + q], sy[Q0 + q], sz[Q0 + q]) < fminf(wv, sv[Q0 + q]);
            if (use) {
                fl[Q0 + q] |= (ra[q].x >> 31) << 2;
                sv[Q0 + q] = u2f(ra[q].x & 0x7fffffffu);
                si[Q0 + q] = ra[q].y & 0x7fffffffu;
                ss[Q0 + q] = u2f(ra[q].z);
                sx[Q0 + q] = u2f(rb[q].x); sy[Q0 + q] = u2f(rb[q].y); sz[Q0 + q] = u2f(rb[q].z);
            }
            rel[q] = (fl[Q0 + q] & 9u) == 1u && ud[Q0 + q] < wv && sv[Q0 + q] >= thr;
            pm[q] = __builtin_amdgcn_ballot_w64(pk[q]);
            rm[q] = __builtin_amdgcn_ballot_w64(rel[q]);
        }
        int np_w = 0, nr_w = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q) { np_w += __builtin_popcountll(pm[q]); nr_w += __builtin_popcountll(rm[q]); }
        if (np_w + nr_w) {
            uint32_t old = 0;
            if (lane == 0) old = atomicAdd(&s_n[par], (uint32_t)(np_w | (nr_w << 16)));
            old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
            int pbase = (int)(old & 0xffffu), rbase = (int)(old >> 16);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                if (pk[q]) plist[pbase + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(pm[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm[q], 0u))] = pe[q];
                if (rel[q]) {
                    const int at = rbase + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(rm[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)rm[q], 0u));
                    rlist[at][0] = u32x4{f2u(sv[Q0 + q]), si[Q0 + q], f2u(ss[Q0 + q]), f2u(sx[Q0 + q])};
                    rlist[at][1] = u32x4{f2u(sy[Q0 + q]), f2u(sz[Q0 + q]), off[Q0 + q] >> 4, 0u};
                }
                pbase += __builtin_popcountll(pm[q]);
                rbase += __builtin_popcountll(rm[q]);
            }
        }
        if (round == 1) {
            uint32_t mx = 0;
#pragma unroll
            for (int q = 0; q < NS; ++q) mx = umax(mx, f2u(sv[Q0 + q]));
            mx = wave_max_u32(mx);
            if (lane == 0) atomicMax(&s_sum[1], mx);
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const uint32_t ov = eight_max_all(f2u(sv[Q0 + q]));
            gv[Q0 + q] = u2f(ov);
            if ((fl[Q0 + q] & 8u) && (lane & 7) == 0) s_wv[par] = ov;
        }
    };
    // Which workgroups matter from the next round on; packs the slots when half of them will do.
    auto shrink = [&](auto tag) {
        constexpr int NS = decltype(tag)::value;
        int groups = 0;
        uint64_t act[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            if constexpr (kBoxesInLds) gv[q] = u2f(eight_max_all(f2u(sv[q])));
            const bool keep = (fl[q] & 1u) && wd[q] < fmaxf(gv[q], wv);
            // waited for: wanted until now
            fl[q] = (fl[q] & 12u) | ((fl[q] & 1u) << 1) | (keep ? 1u : 0u);
            act[q] = __builtin_amdgcn_ballot_w64((fl[q] & 3u) != 0 && (lane & 7) == 0);
            groups += __builtin_popcountll(act[q]);
        }
        if constexpr (NS > 1) {
            if (groups <= 8 * (NS / 2)) {
                constexpr int ND = NS / 2;
                int from[ND];  // source lane + 64 * source slot
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    int r = d * 8 + (lane >> 3);  // rank of the group this lane gets
                    from[d] = -1;
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        const int n = __builtin_popcountll(act[q]);
                        if (r >= 0 && r < n) {
                            uint64_t b = act[q];
                            for (int k = 0; k < r; ++k) b &= b - 1;
                            from[d] = (int)__builtin_ctzll(b) + (lane & 7) + 64 * q;
                        }
                        r -= n;
                    }
                }
                auto move = [&](auto &arr) {
                    using E = std::remove_reference_t<decltype(arr[0])>;
                    E t[ND];
#pragma unroll
                    for (int d = 0; d < ND; ++d) {
                        t[d] = arr[0];
#pragma unroll
                        for (int q = 0; q < NS; ++q) {
                            const E o = __shfl(arr[q], from[d] & 63);
                            t[d] = (from[d] >> 6) == q ? o : t[d];
                        }
                    }
#pragma unroll
                    for (int d = 0; d < ND; ++d) arr[d] = t[d];
                };
                move(wd); move(ud); move(sv); move(ss); move(sx); move(sy); move(sz); move(si); move(off); move(fl);
#pragma unroll
                for (int d = 0; d < ND; ++d)
                    if (from[d] < 0) fl[d] = 0;
                cur = ND;
            }
        }
    };
    for (;; ++round) {
        const uint32_t par = round & 1;
        wg_barrier();  // 0: candidates as published for this round
        uint32_t h0 = 0, h1 = 0;
        if ((round & 3) == 0) {
            if (enough) {
                const uint32_t b = (f2u(wv) >> kLocalBinShift) + 1 + tid;
                for (uint32_t c = b + kThreads; c <= maxbin; c += kThreads)
                    h1 += __hip_atomic_load(&hist[local_bin_place(c)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (b <= maxbin) h0 = __hip_atomic_load(&hist[local_bin_place(b)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                // picks of each unit so far
                for (int u = tid; u < U; u += kThreads)
                    h1 += __hip_atomic_load(&count[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lane == 0) __hip_atomic_store(&count[unit], (uint32_t)np, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        // ---- while the records travel: candidates against this workgroup's own units ----
        {
            const int c = lane & 7, k = lane >> 3;
            const u32x4 mA = candA[c], mB = candB[c], oA = candA[k], oB = candB[k];
            const Box ob = ubox[k];
            const float pv = u2f(mA.x), px = u2f(mB.x), py = u2f(mB.y), pz = u2f(mB.z);
            const uint64_t kp = ((uint64_t)mA.x << 32) | ~mA.y, ku = ((uint64_t)oA.x << 32) | ~oA.y;
            const bool near = box_dist(ob, px, py, pz) < pv;
            const bool hid = (u2f(oA.z) >= pv) | (sqdist(u2f(oB.x), u2f(oB.y), u2f(oB.z), px, py, pz) < pv);
            const uint64_t bm = __builtin_amdgcn_ballot_w64((mA.x == 0u) | ((ku > kp) & near & hid));  // of itself no key is greater
            uint32_t o = (uint32_t)bm | (uint32_t)(bm >> 32);
            o |= o >> 16;
            o |= o >> 8;
            open = ~o & 0xffu;
            thr = u2f(~row_max_uniform(lane < 8 && ((open >> c) & 1u) ? ~mA.x : 0u));
        }
        if (cur == 1) {
            gather(std::integral_constant<int, 1>{}, s0);
        } else if (cur == 2 || P > kGatherRows) {
            gather(std::integral_constant<int, 2>{}, s0);
            if (cur == 4) gather(std::integral_constant<int, 2>{}, s2);
        } else {
            gather(std::integral_constant<int, 4>{}, s0);
        }
        // the unit's pick of the round before goes to the list now, out of the exchange's way
        if (!logged) {
            if (np >= p1 - p0) {  // a point picked twice: coordinates that are not finite
                bad = true;
                s_twice = 1;
            } else if (lane == 0) {
                picks[np] = u32x4{f2u(lv), li, round - 1, 0u};
                atomicAdd(&hist[local_bin_place(f2u(lv) >> kLocalBinShift)], 1u);
            }
            ++np;
            logged = true;
        }
        if (bad) s_bad = 1;
        if (round > 1 && (round & 3) == 0) {
            uint32_t sum = h0 + h1;
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            if (lane == 0 && sum) atomicAdd(&s_sum[0], sum);
        }
        wg_barrier();  // 1: both lists, s_wv, s_sum
        const uint32_t seen = s_sum[par], counts = s_n[par];
        const uint32_t wvb = s_wv[par], isbad = s_bad;
        const u32x4 e_first = plist[lane], r0 = rlist[lane][0], r1 = rlist[lane][1];
        wv = u2f(wvb);
        if (isbad) break;
        if (round == 1) maxbin = seen >> kLocalBinShift;
        const bool reached = round > 1 && (round & 3) == 0 && seen >= (uint32_t)(a.M - 1);
        const bool over = enough && reached;
        enough = enough || reached;
        if (tid == 0) s_sum[par ^ 1] = s_n[par ^ 1] = 0;
        if (wv == 0.f || over) {
            // nothing left here that belongs to the samples
            publish(round + 1, false, true);
            break;
        }
        // ---- apply the picks of the round before; is the published candidate still what it was? ----
        const int npl = (int)(counts & 0xffffu), nrl = (int)(counts >> 16);
        bool changed = false;
        bool pick = (open >> wave) & 1u;
        for (int c0 = 0; c0 < npl; c0 += kWave) {
            u32x4 e = c0 == 0 ? e_first : plist[c0 + lane];
            const float ex_ = u2f(e.x), ey_ = u2f(e.y), ez_ = u2f(e.z), ev_ = fminf(best.v, u2f(e.w));
            const bool in = c0 + lane < npl;
            const bool hit = in && unit_dist(ex_, ey_, ez_) < ev_;
            const bool low = in && sqdist(best.x, best.y, best.z, ex_, ey_, ez_) < ev_;
            pick = pick && __builtin_amdgcn_ballot_w64(low) == 0;
            uint64_t hits = __builtin_amdgcn_ballot_w64(hit);
            changed = changed || hits != 0;
            while (hits) {
                // two at a time: their arithmetic is independent
                const int h0 = (int)__builtin_ctzll(hits);
                hits &= hits - 1;
                const int h1 = hits ? (int)__builtin_ctzll(hits) : h0;
                hits &= hits - 1;
                const float ax = readlane_f(ex_, h0), ay = readlane_f(ey_, h0), az = readlane_f(ez_, h0), av = readlane_f(u2f(e.w), h0);
                const float cx = readlane_f(ex_, h1), cy = readlane_f(ey_, h1), cz = readlane_f(ez_, h1), cv = readlane_f(u2f(e.w), h1);
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    float d = sqdist(x[j], y[j], z[j], ax, ay, az), f = sqdist(x[j], y[j], z[j], cx, cy, cz);
                    d = d < av ? d : __builtin_inff();
                    f = f < cv ? f : __builtin_inff();
                    m[j] = min3_dist(m[j], d, f);
                    few_rows<P>(j);
                }
            }
        }
        // ---- does a unit come before it with a point in its ball? ----
        if (pick) {
            const uint64_t kp = ((uint64_t)f2u(best.v) << 32) | ~best.i;
            auto holds = [&](const u32x4 &e0, const u32x4 &e1, int c) {
                const uint64_t ke = ((uint64_t)e0.x << 32) | ~e0.y;
                const bool above = c < nrl && ke > kp;
                if (__builtin_amdgcn_ballot_w64(above) == 0) return false;
                const Box eb = sbox[above ? e1.z : 0u];
                const bool blk = above && box_dist(eb, best.x, best.y, best.z) < best.v &&
                                 (u2f(e0.z) >= best.v || sqdist(u2f(e0.w), u2f(e1.x), u2f(e1.y), best.x, best.y, best.z) < best.v);
                return __builtin_amdgcn_ballot_w64(blk) != 0;
            };
            pick = !holds(r0, r1, lane);
            for (int c0 = kWave; c0 < nrl && pick; c0 += 2 * kWave) {
                const int c = c0 + lane, d = (c + kWave) & (kList - 1);
                const u32x4 a0 = rlist[c][0], a1 = rlist[c][1];
                const u32x4 b0 = rlist[d][0], b1 = rlist[d][1];
                pick = !holds(a0, a1, c);
                if (pick && c0 + kWave < nrl) pick = !holds(b0, b1, c + kWave);
            }
        }
        if (pick) {
            lv = best.v;
            li = best.i;
            logged = false;
            apply(best.x, best.y, best.z, best.v);
        }
        if (pick || changed) best = unit_best<P>(x, y, z, m, id, lane);
        publish(round + 1, pick, false);
        if (cur == 1) shrink(std::integral_constant<int, 1>{});
        else if (cur == 2) shrink(std::integral_constant<int, 2>{});
        else shrink(std::integral_constant<int, 4>{});
    }
    if (lane == 0) a.npicks[cloud * U + unit] = np < p1 - p0 ? np : p1 - p0;
    __syncthreads();
    if (tid == 0) {
        if (s_bad) {
            int expected = 0;
            __hip_atomic_compare_exchange_strong(a.status, &expected, s_twice ? kErrInconsistent : kErrGaveUp, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int P>
hipError_t launch_t(LocalArgs &a, int clouds, hipStream_t s) {
    void *params[] = {&a};
    return hipLaunchCooperativeKernel((const void *)k_fps_local<P>, dim3(clouds * a.G), dim3(kThreads), params, 0, s);
}

// Rows of 64 points per unit.
#define FFPS_LOCAL_ROWS(X) X(1) X(2) X(3) X(4) X(6) X(8) X(12) X(16) X(24) X(32) X(40)
constexpr int kMaxRows = 40;
constexpr int kUnitMax = kMaxRows * kWave;

}  // namespace

LocalPlan plan_fps_local(int B, int N, int num_cu) {
    const int maxG = num_cu < kMaxGridWG ? num_cu : kMaxGridWG;
    LocalPlan p = {0, 0, 0};
    const int need = (N + kWaves * kUnitMax - 1) / (kWaves * kUnitMax);
    if (need > maxG) return p;
    int g = (N + kThreads - 1) / kThreads;  // a row of points per unit
    const int share = maxG / (B < maxG ? B : maxG);
    if (g > share) g = share;
    if (g < need) g = need;
    p.wg_per_cloud = g;
    p.units_per_cloud = g * kWaves;
    p.clouds_per_launch = maxG / g < B ? maxG / g : B;
    return p;
}

LocalBuffers carve_local(char *base, int B, int N, const LocalPlan &p, size_t *bytes) {
    LocalBuffers l;
    size_t o = 0;
    auto take = [&](size_t n) {
        const size_t at = o;
        o += (n + 255) / 256 * 256;
        return base + at;
    };
    const int tiles = order_tiles(N);
    const size_t n = (size_t)B * N;
    l.pts = take(n * 16);
    l.picks = take(n * 16);
    l.npicks = (int *)take((size_t)B * p.units_per_cloud * 4);
    l.exchange_bytes_per_cloud = (size_t)8 * p.units_per_cloud * 16;
    l.zeroed = take((size_t)B * l.exchange_bytes_per_cloud);
    l.hist = (uint32_t *)take((size_t)B * kLocalWords * 4);
    l.cursor = (uint32_t *)take((size_t)B * kLocalBins * 4);
    l.zero_bytes = (size_t)(base + o - l.zeroed);
    l.runs = take((size_t)B * kLocalBins * 8);
    l.nruns = (int *)take((size_t)B * 4);
    l.boxes = (float *)take((size_t)B * tiles * 24);
    l.codes = (uint16_t *)take(n * 2);
    l.hist1 = (uint32_t *)take((size_t)B * tiles * 1024);
    l.hist2 = (uint32_t *)take((size_t)B * tiles * 512);
    if (bytes) *bytes = o;
    return l;
}

int local_capacity() { return kMaxGridWG * kWaves * kUnitMax; }

size_t local_workspace_bound(int B, int N) {
    // no device gives a cloud more workgroups than this, whatever it has
    LocalPlan p = plan_fps_local(B, N, kMaxGridWG);
    const int need = (N + kWaves * kUnitMax - 1) / (kWaves * kUnitMax);
    if (p.wg_per_cloud < need) p.wg_per_cloud = need;
    p.units_per_cloud = p.wg_per_cloud * kWaves;
    size_t bytes = 0;
    carve_local(nullptr, B, N, p, &bytes);
    return bytes;
}

hipError_t launch_local(const float *xyz, const LocalBuffers &l, int B, int N, int M, int start, const int *start_dev, const LocalPlan &p,
                        int *status, int spin_limit, hipStream_t s) {
    const int rows = ((N + p.units_per_cloud - 1) / p.units_per_cloud + kWave - 1) / kWave;
    for (int b = 0; b < B; b += p.clouds_per_launch) {
        const int clouds = B - b < p.clouds_per_launch ? B - b : p.clouds_per_launch;
        LocalArgs a;
        a.xyz = xyz + (size_t)b * N * 3;
        a.pts = (const u32x4 *)l.pts + (size_t)b * N;
        a.N = N; a.M = M; a.start = start; a.start_dev = start_dev ? start_dev + b : nullptr;
        a.G = p.wg_per_cloud;
        a.exchange = l.zeroed + (size_t)b * l.exchange_bytes_per_cloud;
        a.picks = (u32x4 *)l.picks + (size_t)b * N;
        a.npicks = l.npicks + (size_t)b * p.units_per_cloud;
        a.hist = l.hist + (size_t)b * kLocalWords;
        a.status = status;
        a.spin_limit = spin_limit < 0 ? kSpinLimit : spin_limit;
        hipError_t e = hipErrorInvalidValue;
#define X(R) if (e == hipErrorInvalidValue && rows <= (R)) e = launch_t<R>(a, clouds, s);
        FFPS_LOCAL_ROWS(X)
#undef X
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ffps
