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
// round makes as many picks as there are separate maxima (397 on average, 148 rounds)
// and a pick is applied where it can matter: about 130 distances per point, not 50,000.
// What is left is the latency of a round, which is what everything below is about.
//
//   - Points are sorted along a space-filling curve first (spatial.hip); a UNIT, one
//     wave, holds a stretch of it (up to 40 rows of 64 points), eight units make a workgroup.
//     Up to 24 rows are held in registers; beyond, their distances and a part of them are.
//   - Per round a unit publishes its two best points (value and coordinates, of the best its index), a bound of
//     the values of all others, and whether the candidate it published the round before was picked:
//     48 bytes.  Every lane reads the records of up to four units, eight lanes for a
//     workgroup, those of neighbouring workgroups in different waves.
//   - A workgroup needs the records of another only while the distance of their points is
//     below the larger of their largest values.  Both sides see the same records and drop
//     each other in the same round, so late rounds exchange with a few neighbours and
//     neighbourhoods far apart may be many rounds apart.
//   - A candidate is a pick when no unit holds a point before it in its ball: a unit does
//     not if its best comes later; or if its best lies outside, its second does or comes later, and the
//     others come later or its box lies outside.  (Without the second point: 178 rounds in place of 148, 100 in
//     place of 89 for 45,678 points to 5001.)  Only rounds with one slot a lane read the second points: earlier ones
//     gather more records and make few picks.
//   - A workgroup stops when as many picks as samples have values in bins above that
//     of its largest value: nothing it holds can belong to the samples any more.  Picks
//     beyond the samples are left out by the final sort (spatial.hip): 18 % more than the 50,000 of a
//     room, 45 % more than 5001 of 45,678, 37 % more than 16,384 of a LiDAR frame.
//
// Measured, exact FPS of a room of 200,000 points to 50,000 samples, sorts included:
// 0.63 ms against 4.44 ms with k_fps_grid; 45,678 points to 5,001: 0.34 against 0.84 ms;
// five million to 1024: 0.92 ms against 4.7 ms with k_fps_stream.
// Before the second points, loops by the number of slots, lanes' states as masks in scalar registers and a unit's own pick
// applied beside the others': 0.84, 0.43 and 1.2 ms.
//
// Every wait is bounded as in fps_exchange.h.  A point that is picked twice (coordinates that are not
// finite) ends the workgroup with the status of inconsistent results; those that wait for it look at the
// status now and then and leave, too.
#include "fps_exchange.h"
#include "fps_local.h"
#include "fps_record.h"
#include "fps_space.h"

namespace ffps {

namespace {

constexpr int kWaves = 8;  // units of a workgroup, two waves per SIMD
constexpr int kThreads = kWaves * kWave;
constexpr uint32_t kTagWindow = 1u << 20;  // "this round or a later one"
constexpr int kPollsPerLook = 1024;        // at records that are missing, between two looks at the status

// The round a chunk is of, if it is whole.
__device__ __forceinline__ uint32_t chunk_round(const u32x4 &c, uint32_t which) { return record_check(c.x, c.y, c.z, which, c.w); }

// 16 bytes of every unit, side by side: the boxes, then the records of even and of odd rounds.
constexpr int kBoxPlanes = 4, kRecordPlanes = 3;
constexpr int kPlanes = kBoxPlanes + 2 * kRecordPlanes;

struct LocalArgs {
    const float *xyz;     // [clouds][N][3] as the caller has them, for the first sample
    const u32x4 *pts;     // [clouds][N] along the curve: {x, y, z, index}
    int N, M, start;
    const int *start_dev;
    int G;                // workgroups per cloud
    char *exchange;       // per cloud kPlanes planes of 16 bytes per unit, cleared
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

// sum over the wave
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    v += dpp_or_zero<kDppRowShr1>(v);
    v += dpp_or_zero<kDppRowShr2>(v);
    v += dpp_or_zero<kDppRowShr4>(v);
    v += dpp_or_zero<kDppRowShr8>(v);
    return (uint32_t)(readlane_i((int)v, 15) + readlane_i((int)v, 31) + readlane_i((int)v, 47) + readlane_i((int)v, 63));
}

__device__ __forceinline__ Box box_shfl(const Box &a, int l) {
    return Box{__shfl(a.lx, l), __shfl(a.ly, l), __shfl(a.lz, l), __shfl(a.hx, l), __shfl(a.hy, l), __shfl(a.hz, l)};
}
// An address that is the same in all lanes, in scalar registers whatever the compiler knows of it.
__device__ __forceinline__ const char *uniform_address(const char *p) {
    const uint64_t v = (uint64_t)p;
    return (const char *)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
}
// The records of NS slots: 16 bytes at off in each of two or three planes, read past the caches that are not shared by
// the whole device.  The planes' addresses are scalars, which the compiler may just have taken from a vector
// register: five wait states before they are used as addresses, and it does not look into the block.
template <int NS, bool THREE>
__device__ __forceinline__ void load_records(const char *p0, const char *p1, const char *p2, const uint32_t *off, u32x4 (&a)[NS],
                                             u32x4 (&b)[NS], u32x4 (&c)[NS]) {
    static_assert(NS == 1 || (!THREE && (NS == 2 || NS == 4)), "");
    if constexpr (THREE) {
        asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %3, %4 sc1\n\tglobal_load_dwordx4 %1, %3, %5 sc1\n\t"
                     "global_load_dwordx4 %2, %3, %6 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(a[0]), "=&v"(b[0]), "=&v"(c[0])
                     : "v"(off[0]), "s"(p0), "s"(p1), "s"(p2) : "memory");
    } else if constexpr (NS == 1) {
        asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %2, %3 sc1\n\tglobal_load_dwordx4 %1, %2, %4 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(a[0]), "=&v"(b[0])
                     : "v"(off[0]), "s"(p0), "s"(p1) : "memory");
    } else if constexpr (NS == 2) {
        asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %4, %6 sc1\n\tglobal_load_dwordx4 %1, %4, %7 sc1\n\t"
                     "global_load_dwordx4 %2, %5, %6 sc1\n\tglobal_load_dwordx4 %3, %5, %7 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(a[0]), "=&v"(b[0]), "=&v"(a[1]), "=&v"(b[1])
                     : "v"(off[0]), "v"(off[1]), "s"(p0), "s"(p1) : "memory");
    } else {
        asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %8, %12 sc1\n\tglobal_load_dwordx4 %1, %8, %13 sc1\n\t"
                     "global_load_dwordx4 %2, %9, %12 sc1\n\tglobal_load_dwordx4 %3, %9, %13 sc1\n\t"
                     "global_load_dwordx4 %4, %10, %12 sc1\n\tglobal_load_dwordx4 %5, %10, %13 sc1\n\t"
                     "global_load_dwordx4 %6, %11, %12 sc1\n\tglobal_load_dwordx4 %7, %11, %13 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(a[0]), "=&v"(b[0]), "=&v"(a[1]), "=&v"(b[1]), "=&v"(a[2]), "=&v"(b[2]), "=&v"(a[3]), "=&v"(b[3])
                     : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(p0), "s"(p1) : "memory");
    }
}

// The points of a lane: in registers up to so many rows, with their indices up to fewer (only that of a unit's best
// point is ever needed).
constexpr int kRegRows = 24, kRegIndexRows = 16;
// Beyond, some rows are and the others are read again where a pick reaches the unit (a fifth of the units in a round).
// us for 3.0, 3.3 and 4.3 million points of rooms to 1000, 1000 and 200 samples (24, 32 and 40 rows): all in registers 731,
// 842 and 831 (52, 149 and 228 spilled; without second points), all read again 787, 879 and 759, as here 683, 787 and 706.
constexpr int held_rows(int P) { return P <= kRegRows ? P : 48 - P; }
constexpr int kRowsAtOnce = 8;  // that are read again
// Where points are read, every few rows the compiler may not mix with those before them: it would have
// dozens of rows on their way at once and spill the distances.
template <int P>
__device__ __forceinline__ void few_rows(int j) {
    if (P > kRegIndexRows && (j & (kRowsAtOnce - 1)) == kRowsAtOnce - 1) __builtin_amdgcn_sched_barrier(0);
}

// The two best points of a unit and a value that no other of its points exceeds, the same in all lanes of the unit.
struct Best {
    float v, x, y, z;
    uint32_t i;
    float v2, x2, y2, z2;
    float v3;
};

template <int P>
struct Points {
    static constexpr int kRows = held_rows(P);  // in registers
    static constexpr bool kAll = kRows == P, kIndices = P <= kRegIndexRows;
    float x[kRows], y[kRows], z[kRows];
    uint32_t id[kIndices ? P : 1];
    const u32x4 *pts;  // first point of the unit
    int n, lane;       // points of the unit
    __device__ __forceinline__ u32x4 read(int i) const { return (uint32_t)i < (uint32_t)n ? pts[i] : u32x4{0u, 0u, 0u, kNoIndex}; }
    __device__ __forceinline__ u32x4 at(int j) const {
        if (j < kRows) return u32x4{f2u(x[j < kRows ? j : 0]), f2u(y[j < kRows ? j : 0]), f2u(z[j < kRows ? j : 0]), 0u};
        return read(j * kWave + lane);
    }
    __device__ __forceinline__ uint32_t index(int j) const {
        if constexpr (kIndices) return id[j];
        const int i = j * kWave + here();
        return i < n ? reinterpret_cast<const uint32_t *>(pts + i)[3] : kNoIndex;
    }
    // The lane, in a way that keeps the addresses of all rows from being worked out ahead of the rounds and kept.
    __device__ __forceinline__ int here() const {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
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
__device__ __forceinline__ Best unit_best(const Points<P> &p, const float (&m)[P], int lane) {
    Best b;
    float t1 = m[0], t2 = 0.f;
#pragma unroll
    for (int j = 1; j < P; ++j) {
        t2 = __builtin_amdgcn_fmed3f(t1, t2, m[j]);
        t1 = fmaxf(t1, m[j]);
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
            if (!Points<P>::kIndices && __builtin_amdgcn_ballot_w64(f2u(m[j]) == T1) == 0) continue;
            const uint32_t i = p.index(j);
            const bool e = f2u(m[j]) == T1 && i < mi;
            mi = e ? i : mi;
            jr = e ? j : jr;
        }
        const uint32_t lo = wave_min_u32(mi);
        own = __builtin_amdgcn_ballot_w64(mi == lo);
    }
    const int wl = (int)__builtin_ctzll(own);
    // Of equal seconds any will do: the third value is the same then.  So it is taken to be where a lane
    // holds the two best: its own third value is not known.
    const uint32_t rest = lane == wl ? f2u(t2) : f2u(t1);
    const uint32_t T2 = wave_max_u32(rest);
    const int wl2 = first_lane(rest == T2);
    b.v2 = u2f(T2);
    int jr2 = 0;
#pragma unroll
    for (int j = P - 1; j > 0; --j) jr2 = f2u(m[j]) == T2 ? j : jr2;
    if constexpr (P > 1) jr2 = f2u(m[0]) == T2 ? 0 : jr2;
    if constexpr (Points<P>::kAll) {
        auto point = [&](int jr_, int l, float &ox, float &oy, float &oz, bool index_too) {
            uint32_t oi = 0;
            if constexpr (P > 4) {
                const int row = readlane_i(jr_, l);
                pick_xyz<P>(p.x, p.y, p.z, row, l, ox, oy, oz);
                if constexpr (Points<P>::kIndices) {
#pragma unroll
                    for (int j = 0; j < P; ++j)
                        if (row == j) oi = (uint32_t)readlane_i((int)p.id[j], l);
                } else if (index_too) {
                    oi = p.read(row * kWave + l).w;
                }
            } else {
                float bx = p.x[0], by = p.y[0], bz = p.z[0];
                uint32_t bi = p.id[0];
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    bx = jr_ == j ? p.x[j] : bx; by = jr_ == j ? p.y[j] : by; bz = jr_ == j ? p.z[j] : bz;
                    bi = jr_ == j ? p.id[j] : bi;
                }
                ox = readlane_f(bx, l); oy = readlane_f(by, l); oz = readlane_f(bz, l);
                oi = (uint32_t)readlane_i((int)bi, l);
            }
            return oi;
        };
        b.i = point(jr, wl, b.x, b.y, b.z, true);
        (void)point(jr2, wl2, b.x2, b.y2, b.z2, false);
    } else {
        // Both at once, by lanes 0 and 1.  Lanes of others are read before the lanes go separate ways: where only some
        // are active, the others' values need not have been worked out.
        const int i1 = readlane_i(jr, wl) * kWave + wl, i2 = readlane_i(jr2, wl2) * kWave + wl2;
        const u32x4 q = p.read(lane & 1 ? i2 : i1);
        b.x = readlane_f(u2f(q.x), 0); b.y = readlane_f(u2f(q.y), 0); b.z = readlane_f(u2f(q.z), 0);
        b.i = (uint32_t)readlane_i((int)q.w, 0);
        b.x2 = readlane_f(u2f(q.x), 1); b.y2 = readlane_f(u2f(q.y), 1); b.z2 = readlane_f(u2f(q.z), 1);
    }
    b.v3 = u2f(wave_max_u32(lane == wl2 ? f2u(t2) : rest));
    return b;
}

// Rows up to which the records of four slots are gathered at once; beyond, the registers that
// takes are dearer than a second wait (at 24 to 40 rows; 12 and 16 rows were not tried).
constexpr int kGatherRows = 16;

// What scalar registers do not hold (54 to 82 of them up to 12 rows, 108, 138, 211 and 313 from 16 to 40) is kept in lanes of one or two
// vector registers.  Up to 12 rows half of that is read in the rounds: 38 to 46 instructions of 2500 to 3600 in the loop with
// four slots, 7 to 15 of 1200 to 2700 in the others; at 16 rows 60, 37 and 27, at 24 80, 67 and 45, at 40 204, 164 and 152 of 5600 to 7000.
template <int P>
__global__ __launch_bounds__(kThreads, 2) void k_fps_local(LocalArgs a) {
    constexpr int kSlots = 4;
    constexpr int kList = kSlots * kThreads;
    __shared__ __attribute__((aligned(16))) u32x4 plist[kList];     // new picks that may matter here
    __shared__ __attribute__((aligned(16))) u32x4 rlist[2 * kList];  // units that may hold a candidate back: two or three words of 16 bytes
    __shared__ Box sbox[kList];                                     // boxes of all units
    // of this workgroup's units: {value, index, value', value''}, {x, y, z, -}, {x', y', z', -}
    __shared__ u32x4 candA[kWaves], candB[kWaves], candC[kWaves];
    __shared__ Box ubox[kWaves], boxA[kWaves], boxB[kWaves];  // a unit's two boxes and their union
    __shared__ Box wboxes[2];                                 // the workgroup's two boxes
    __shared__ uint32_t s_n[2], s_sum[2], s_bad, s_twice;
    __shared__ uint32_t s_groups[4];  // most groups of eight lanes a wave waits for, by rounds: written between two of them, without a barrier

    const int G = a.G, U = G * kWaves;
    const int cloud = blockIdx.x / G, w = blockIdx.x - cloud * G;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = w * kWaves + wave;
    const u32x4 *pts = a.pts + (size_t)cloud * a.N;
    char *ex = const_cast<char *>(uniform_address(a.exchange + (size_t)cloud * kPlanes * U * 16));
    const size_t plane = (size_t)(uint32_t)__builtin_amdgcn_readfirstlane(U * 16);  // boxes: planes 0 to 3; records: planes 4 to 6 (even rounds) and 7 to 9
    uint32_t *hist = a.hist + (size_t)cloud * kLocalWords, *count = hist + kLocalBins;
    const int start = a.start_dev ? a.start_dev[cloud] : a.start;

    // ---- points of this unit ----
    const int p0 = (int)((long)unit * a.N / U), p1 = (int)((long)(unit + 1) * a.N / U);
    u32x4 *picks = a.picks + (size_t)cloud * a.N + p0;
    int np = 0;  // picks of this unit in its list
    float m[P];
    Points<P> p;
    p.pts = pts + p0;
    p.n = p1 - p0;
    p.lane = lane;
    // The unit's points in their order as two boxes, cut at the widest step: the order jumps
    // now and then, and one box around both ends of a jump would be met by most picks.
    Box ba = no_box(), bb = no_box();
    {
        const float *q = a.xyz + ((size_t)cloud * a.N + start) * 3;
        const float qx = q[0], qy = q[1], qz = q[2];
#pragma unroll
        for (int j = 0; j < Points<P>::kRows; ++j) {
            const u32x4 o = p.read(j * kWave + lane);
            p.x[j] = u2f(o.x); p.y[j] = u2f(o.y); p.z[j] = u2f(o.z);
            if constexpr (Points<P>::kIndices) p.id[j] = o.w;
            few_rows<P>(j);
        }
        float g = 0.f;
        int at = (p1 - p0) / 2;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = j * kWave + lane;
            const u32x4 o = p.at(j);
            const float ox = u2f(o.x), oy = u2f(o.y), oz = u2f(o.z);
            m[j] = i < p.n ? min_dist(__builtin_inff(), sqdist(ox, oy, oz, qx, qy, qz)) : 0.f;
            float nx = __shfl(ox, (lane + 1) & 63), ny = __shfl(oy, (lane + 1) & 63), nz = __shfl(oz, (lane + 1) & 63);
            if (j + 1 < P) {
                const u32x4 f = j + 1 < Points<P>::kRows ? p.at(j + 1) : p.read((j + 1) * kWave);
                const float fx = readlane_f(u2f(f.x), 0), fy = readlane_f(u2f(f.y), 0), fz = readlane_f(u2f(f.z), 0);
                nx = lane == 63 ? fx : nx; ny = lane == 63 ? fy : ny; nz = lane == 63 ? fz : nz;
            }
            const float d = i + 1 < p.n ? sqdist(ox, oy, oz, nx, ny, nz) : 0.f;
            at = d > g ? i : at;
            g = fmaxf(g, d);
            few_rows<P>(j);
        }
        const uint32_t top = wave_max_u32(f2u(g));
        at = readlane_i(at, first_lane(f2u(g) == top));
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = j * kWave + lane;
            const u32x4 r = p.at(j);
            const Box o = {u2f(r.x), u2f(r.y), u2f(r.z), u2f(r.x), u2f(r.y), u2f(r.z)};
            if (i < p.n && i <= at) ba = box_or(ba, o);
            if (i < p.n && i > at) bb = box_or(bb, o);
            few_rows<P>(j);
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            ba = box_or(ba, box_shfl_xor(ba, o));
            bb = box_or(bb, box_shfl_xor(bb, o));
        }
    }
    Best best = unit_best<P>(p, m, lane);
    auto publish = [&](uint32_t round, bool picked, bool stopped) {
        if (lane == 0) {
            char *buf = ex + plane * (kBoxPlanes + kRecordPlanes * (round & 1)) + (size_t)unit * 16;
            u32x4 A, B, C;
            A.x = f2u(best.v) | (stopped ? 0x80000000u : 0u);
            A.y = index_word(best.i, f2u(best.v2), f2u(best.v3), picked);
            A.z = f2u(best.v2);
            A.w = record_check(A.x, A.y, A.z, kTagA, round);
            B.x = f2u(best.x); B.y = f2u(best.y); B.z = f2u(best.z);
            B.w = record_check(B.x, B.y, B.z, kTagB, round);
            C.x = f2u(best.x2); C.y = f2u(best.y2); C.z = f2u(best.z2);
            C.w = record_check(C.x, C.y, C.z, kTagC, round);
            store_chunk(buf, A);
            store_chunk(buf + plane, B);
            store_chunk(buf + 2 * plane, C);
            candA[wave] = u32x4{f2u(best.v), best.i, f2u(best.v2), f2u(best.v3)};
            candB[wave] = B;
            candC[wave] = C;
        }
    };
    if (lane == 0) {
        auto put = [&](int k, float c0, float c1, float c2) {
            u32x4 A = {f2u(c0), f2u(c1), f2u(c2), 0u};
            A.w = record_check(A.x, A.y, A.z, kTagBox, (uint32_t)(k + 1));
            store_chunk(ex + plane * k + (size_t)unit * 16, A);
        };
        put(0, ba.lx, ba.ly, ba.lz); put(1, ba.hx, ba.hy, ba.hz);
        put(2, bb.lx, bb.ly, bb.lz); put(3, bb.hx, bb.hy, bb.hz);
        boxA[wave] = ba;
        boxB[wave] = bb;
        ubox[wave] = box_or(ba, bb);
    }
    publish(1, false, false);
    if (tid < 2) s_n[tid] = s_sum[tid] = 0;
    if (tid < 4) s_groups[tid] = 0;
    if (tid == 0) s_bad = s_twice = 0;

    // ---- slots: the units this lane keeps track of, eight lanes per workgroup ----
    float wd[kSlots], ud[kSlots];   // distance of its workgroup's box, and of its own, from this workgroup's box
    float gv[kSlots];               // largest value of its workgroup
    float sv[kSlots], sx[kSlots], sy[kSlots], sz[kSlots];  // its candidate of the round before
    uint32_t off[kSlots];           // its place, or that of this wave's unit where nothing is waited for
    uint64_t want[kSlots], wait[kSlots];  // lanes whose unit is wanted, and lanes whose record is waited for
    const uint32_t here = (uint32_t)unit * 16;
    int cur = U > 2 * kThreads ? 4 : U > kThreads ? 2 : 1;  // slots in use, by all waves of the workgroup
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
        u32x4 ra[NS], rb[NS], rc[NS], rd[NS];
        uint32_t o[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            // workgroup q * 64 + (lane / 8) * 8 + wave: neighbours along the order go to different waves
            const int s = Q0 + q, g = s * 64 + (lane >> 3) * 8 + wave;
            const bool ok = g < G;
            o[q] = ok ? (uint32_t)(g * 8 + (lane & 7)) * 16 : here;
            off[s] = o[q];
            want[s] = wait[s] = __builtin_amdgcn_ballot_w64(ok);
        }
        for (int spin = 0;; ++spin) {
            load_records<NS, false>(ex, ex + plane, nullptr, o, ra, rb, rc);
            load_records<NS, false>(ex + 2 * plane, ex + 3 * plane, nullptr, o, rc, rd, rd);
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
            sbox[o[q] >> 4] = box_or(A, B);
            // this workgroup's own units hold nothing back from here: they are compared in LDS
            ud[s] = (o[q] >> 7) == (uint32_t)w ? __builtin_inff() : fminf(fminf(box_box(w1, A), box_box(w1, B)), fminf(box_box(w2, A), box_box(w2, B)));
            Box o1, o2;
            two_boxes(A, B, lane, o1, o2);
            wd[s] = fminf(fminf(box_box(w1, o1), box_box(w1, o2)), fminf(box_box(w2, o1), box_box(w2, o2)));
            sv[s] = sx[s] = sy[s] = sz[s] = gv[s] = 0.f;
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
    uint32_t round = 1;
    bool enough = false;    // as many picks as samples, not counting which
    uint32_t open = 0;      // bit c: candidate c is not held back by a unit of this workgroup
    float thr = 0.f;        // the smallest value among those
    // Gathers the records of this round and adds to the two lists.  TWO: with the second points.
    auto gather = [&](auto tag, auto first, auto two) {
        constexpr int NS = decltype(tag)::value, Q0 = decltype(first)::value;
        constexpr bool TWO = decltype(two)::value;
        u32x4 ra[NS], rb[NS], rc[NS];
        const uint32_t par = round & 1;
        const char *b0 = uniform_address(ex + plane * (kBoxPlanes + kRecordPlanes * par)), *b1 = b0 + plane, *b2 = b1 + plane;
        // Lanes whose record is not here yet.  A workgroup that is not wanted any more may be rounds ahead.
        auto missing = [&](int q) {
            const uint32_t da = chunk_round(ra[q], kTagA) - round;
            uint32_t d = da | (chunk_round(rb[q], kTagB) - round);
            if constexpr (TWO) d |= chunk_round(rc[q], kTagC) - round;
            return (__builtin_amdgcn_ballot_w64(d != 0u) & want[Q0 + q]) |
                   (__builtin_amdgcn_ballot_w64(da >= kTagWindow) & wait[Q0 + q] & ~want[Q0 + q]);
        };
        load_records<NS, TWO>(b0, b1, b2, off + Q0, ra, rb, rc);
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            uint64_t ms = missing(q);
            for (int spin = 0; ms != 0; ++spin) {
                if (spin >= a.spin_limit || ((spin & (kPollsPerLook - 1)) == kPollsPerLook - 1 &&
                                             __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    bad = true;
                    break;
                }
                // only what is missing is read again: polling everything would be in the way of
                // those who are waited for
                const bool again = __builtin_amdgcn_inverse_ballot_w64(ms);
                const uint32_t o[1] = {again ? off[Q0 + q] : here};
                u32x4 ta[1], tb[1], tc[1];
                load_records<1, TWO>(b0, b1, b2, o, ta, tb, tc);
                if (again) {
                    ra[q] = ta[0]; rb[q] = tb[0];
                    if constexpr (TWO) rc[q] = tc[0];
                }
                ms = missing(q);
            }
        }
        uint64_t pm[NS], rm[NS];
        u32x4 pe[NS];
        int np_w = 0, nr_w = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int s = Q0 + q;
            const uint64_t stop = __builtin_amdgcn_ballot_w64((int)ra[q].x < 0) & want[s];
            pm[q] = __builtin_amdgcn_ballot_w64((int)ra[q].y < 0) & want[s];
            pe[q] = u32x4{f2u(sx[s]), f2u(sy[s]), f2u(sz[s]), f2u(sv[s])};
            if (pm[q]) pm[q] &= __builtin_amdgcn_ballot_w64(group_dist(sx[s], sy[s], sz[s]) < fminf(wv, sv[s]));
            sv[s] = u2f(ra[q].x & 0x7fffffffu);
            sx[s] = u2f(rb[q].x); sy[s] = u2f(rb[q].y); sz[s] = u2f(rb[q].z);
            want[s] &= ~stop;
            wait[s] &= ~stop;
            rm[q] = __builtin_amdgcn_ballot_w64(ud[s] < wv) & __builtin_amdgcn_ballot_w64(sv[s] >= thr) & want[s];
            np_w += __builtin_popcountll(pm[q]);
            nr_w += __builtin_popcountll(rm[q]);
        }
        if (np_w + nr_w) {
            uint32_t old = 0;
            if (lane == 0) old = atomicAdd(&s_n[par], (uint32_t)(np_w | (nr_w << 16)));
            old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
            int pbase = (int)(old & 0xffffu), rbase = (int)(old >> 16);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int s = Q0 + q;
                if (__builtin_amdgcn_inverse_ballot_w64(pm[q])) plist[pbase + lanes_below(pm[q])] = pe[q];
                if (__builtin_amdgcn_inverse_ballot_w64(rm[q])) {
                    u32x4 *e = rlist + (TWO ? 3 : 2) * (rbase + lanes_below(rm[q]));
                    e[0] = u32x4{f2u(sv[s]), ra[q].y & kRecordIndex, ra[q].z, TWO ? bound_of_others(ra[q].z, ra[q].y) : 0u};
                    e[1] = u32x4{f2u(sx[s]), f2u(sy[s]), f2u(sz[s]), off[s] >> 4};
                    if constexpr (TWO) e[2] = rc[q];
                }
                pbase += __builtin_popcountll(pm[q]);
                rbase += __builtin_popcountll(rm[q]);
            }
        }
        if (round == 1) {
            uint32_t mx = f2u(wv);
#pragma unroll
            for (int q = 0; q < NS; ++q) mx = umax(mx, f2u(sv[Q0 + q]));
            mx = wave_max_u32(mx);
            if (lane == 0) atomicMax(&s_sum[1], mx);
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) gv[Q0 + q] = u2f(eight_max_all(f2u(sv[Q0 + q])));
    };
    // Which workgroups matter from the next round on; packs the slots when half of them will do.
    auto shrink = [&](auto tag, int groups_before) {
        constexpr int NS = decltype(tag)::value;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const uint64_t keep = __builtin_amdgcn_ballot_w64(wd[q] < fmaxf(gv[q], wv)) & want[q];
            wait[q] = want[q];  // wanted until now
            want[q] = keep;
            off[q] = __builtin_amdgcn_inverse_ballot_w64(wait[q]) ? off[q] : here;
        }
        if constexpr (NS > 1) {
            constexpr int ND = NS / 2;
            constexpr uint64_t kFirsts = 0x0101010101010101ull;
            int groups = 0;
#pragma unroll
            for (int q = 0; q < NS; ++q) groups += __builtin_popcountll(wait[q] & kFirsts);
            if (lane == 0) atomicMax(&s_groups[(round + 1) & 3], (uint32_t)groups);
            if (groups_before <= 8 * ND) {  // of every wave the round before; there are never more later
                int from[ND];  // source lane + 64 * source slot
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    int r = d * 8 + (lane >> 3);  // rank of the group this lane gets
                    from[d] = -1;
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        const int n = __builtin_popcountll(wait[q] & kFirsts);
                        if (r >= 0 && r < n) {
                            uint64_t b = wait[q] & kFirsts;
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
                move(wd); move(ud); move(sv); move(sx); move(sy); move(sz); move(off);
                uint64_t nwant[ND], nwait[ND];
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    bool keep = false;
#pragma unroll
                    for (int q = 0; q < NS; ++q) keep = keep || ((from[d] >> 6) == q && ((want[q] >> (from[d] & 63)) & 1u));
                    nwait[d] = __builtin_amdgcn_ballot_w64(from[d] >= 0);
                    nwant[d] = __builtin_amdgcn_ballot_w64(keep);
                }
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    want[d] = nwant[d];
                    wait[d] = nwait[d];
                    off[d] = from[d] >= 0 ? off[d] : here;
                }
                cur = ND;
            }
        }
    };
    // Rounds with as many slots; false after the last one.
    auto rounds = [&](auto tag) {
        constexpr int NS = decltype(tag)::value;
        constexpr bool TWO = NS == 1;
        for (;; ++round) {
            const uint32_t par = round & 1;
            wg_barrier();  // 0: candidates as published for this round
            // every fourth round: loads that nothing waits for before the records are here
            uint32_t h[4] = {0u, 0u, 0u, 0u};
            if ((round & 3) == 0) {
                if (enough) {
                    const uint32_t b = (f2u(wv) >> kLocalBinShift) + 1 + tid;
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (b + k * kThreads <= maxbin) h[k] = __hip_atomic_load(&hist[local_bin_place(b + k * kThreads)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    for (uint32_t c = b + 2 * kThreads; c <= maxbin; c += kThreads)
                        h[2] += __hip_atomic_load(&hist[local_bin_place(c)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    // picks of each unit so far
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (tid + k * kThreads < U) h[k] = __hip_atomic_load(&count[tid + k * kThreads], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (lane == 0) __hip_atomic_store(&count[unit], (uint32_t)np, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            // ---- while the records travel: candidates against this workgroup's own units ----
            {
                const int c = lane & 7, k = lane >> 3;
                const u32x4 mA = candA[c], mB = candB[c], oA = candA[k], oB = candB[k], oC = candC[k];
                const Box ob = ubox[k];
                const float pv = u2f(mA.x), px = u2f(mB.x), py = u2f(mB.y), pz = u2f(mB.z);
                const uint64_t kp = ((uint64_t)mA.x << 32) | ~mA.y, ku = ((uint64_t)oA.x << 32) | ~oA.y;
                const bool hid = (sqdist(u2f(oB.x), u2f(oB.y), u2f(oB.z), px, py, pz) < pv) |
                                 ((oA.z >= mA.x) & (sqdist(u2f(oC.x), u2f(oC.y), u2f(oC.z), px, py, pz) < pv)) |
                                 ((oA.w >= mA.x) & (box_dist(ob, px, py, pz) < pv));
                const uint64_t bm = __builtin_amdgcn_ballot_w64((mA.x == 0u) | ((ku > kp) & hid));  // of itself no key is greater
                uint32_t o = (uint32_t)bm | (uint32_t)(bm >> 32);
                o |= o >> 16;
                o |= o >> 8;
                open = ~o & 0xffu;
                thr = u2f(~row_max_uniform(lane < 8 && ((open >> c) & 1u) ? ~mA.x : 0u));
                wv = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)eight_max_all(mA.x)));
            }
            if constexpr (NS == 4 && P > kGatherRows) {
                gather(s2, s0, std::false_type{});
                gather(s2, s2, std::false_type{});
            } else {
                gather(tag, s0, std::integral_constant<bool, TWO>{});
            }
            if (bad && lane == 0) { s_bad = 1; atomicOr(&s_n[par], 0x80000000u); }
            if (round > 1 && (round & 3) == 0) {
                const uint32_t sum = wave_sum_u32(h[0] + h[1] + h[2] + h[3]);
                if (lane == 0 && sum) atomicAdd(&s_sum[0], sum);
            }
            wg_barrier();  // 1: both lists, s_sum
            const uint32_t seen = s_sum[par], counts = s_n[par], groups = NS > 1 ? s_groups[round & 3] : 0u;
            const u32x4 e_first = plist[lane];
            const u32x4 *rl = rlist + (TWO ? 3 : 2) * lane;
            const u32x4 r0 = rl[0], r1 = rl[1], r2 = rl[TWO ? 2 : 0];
            if ((int)counts < 0) return false;  // this workgroup has given up
            if (round == 1) maxbin = seen >> kLocalBinShift;
            const bool reached = round > 1 && (round & 3) == 0 && seen >= (uint32_t)(a.M - 1);
            const bool over = enough && reached;
            enough = enough || reached;
            if (tid == 0) s_sum[par ^ 1] = s_n[par ^ 1] = s_groups[(round + 2) & 3] = 0;
            if (wv == 0.f || over) {
                // nothing left here that belongs to the samples
                publish(round + 1, false, true);
                return false;
            }
            // ---- apply the picks of the round before; is the published candidate still what it was? ----
            const int npl = (int)(counts & 0xffffu), nrl = (int)(counts >> 16);
            bool changed = false;
            bool pick = (open >> wave) & 1u;
            u32x4 e = e_first;
            uint64_t hits = 0;
            auto apply_hits = [&]() {
                changed = changed || hits != 0;
                // two at a time: their arithmetic is independent
                auto two_hits = [&](uint64_t &todo, auto &&update) {
                    const int h0 = (int)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    const int h1 = todo ? (int)__builtin_ctzll(todo) : h0;
                    todo &= todo - 1;
                    const float ax = readlane_f(u2f(e.x), h0), ay = readlane_f(u2f(e.y), h0), az = readlane_f(u2f(e.z), h0), av = readlane_f(u2f(e.w), h0);
                    const float cx = readlane_f(u2f(e.x), h1), cy = readlane_f(u2f(e.y), h1), cz = readlane_f(u2f(e.z), h1), cv = readlane_f(u2f(e.w), h1);
                    update([&](float &m_, float x_, float y_, float z_) {
                        float d = sqdist(x_, y_, z_, ax, ay, az), f = sqdist(x_, y_, z_, cx, cy, cz);
                        d = d < av ? d : __builtin_inff();
                        f = f < cv ? f : __builtin_inff();
                        m_ = min3_dist(m_, d, f);
                    });
                };
                using Pts = Points<P>;
                if constexpr (Pts::kAll) {
                    while (hits)
                        two_hits(hits, [&](auto &&one) {
#pragma unroll
                            for (int j = 0; j < P; ++j) one(m[j], p.x[j], p.y[j], p.z[j]);
                        });
                } else if (hits) {
                    // Rows beyond the unit's points read those that follow, or the list of picks behind the points of
                    // the last cloud: their distance is 0 and stays that.  Two lots of rows are on their way.
                    const u32x4 *from = p.pts + p.here();
                    float rx[2][kRowsAtOnce], ry[2][kRowsAtOnce], rz[2][kRowsAtOnce];
                    auto fetch = [&](int g) {
#pragma unroll
                        for (int k = 0; k < kRowsAtOnce; ++k) {
                            const float *q = reinterpret_cast<const float *>(from + (g + k) * kWave);
                            rx[(g / kRowsAtOnce) & 1][k] = q[0]; ry[(g / kRowsAtOnce) & 1][k] = q[1]; rz[(g / kRowsAtOnce) & 1][k] = q[2];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    fetch(Pts::kRows);
                    fetch(Pts::kRows + kRowsAtOnce);
                    for (uint64_t todo = hits; todo;)
                        two_hits(todo, [&](auto &&one) {
#pragma unroll
                            for (int j = 0; j < Pts::kRows; ++j) one(m[j], p.x[j], p.y[j], p.z[j]);
                        });
#pragma unroll
                    for (int g = Pts::kRows; g < P; g += kRowsAtOnce) {
                        const int c = (g / kRowsAtOnce) & 1;
                        for (uint64_t todo = hits; todo;)
                            two_hits(todo, [&](auto &&one) {
#pragma unroll
                                for (int k = 0; k < kRowsAtOnce; ++k) one(m[g + k], rx[c][k], ry[c][k], rz[c][k]);
                            });
                        __builtin_amdgcn_sched_barrier(0);
                        if (g + 2 * kRowsAtOnce < P) fetch(g + 2 * kRowsAtOnce);
                    }
                    hits = 0;
                }
            };
            for (int c0 = 0; c0 < npl; c0 += kWave) {
                if (c0) {
                    apply_hits();
                    e = plist[c0 + lane];
                }
                const float ex_ = u2f(e.x), ey_ = u2f(e.y), ez_ = u2f(e.z), ev_ = fminf(best.v, u2f(e.w));
                const bool in = c0 + lane < npl;
                hits = __builtin_amdgcn_ballot_w64(in & (unit_dist(ex_, ey_, ez_) < ev_));
                pick = pick && __builtin_amdgcn_ballot_w64(in & (sqdist(best.x, best.y, best.z, ex_, ey_, ez_) < ev_)) == 0;
            }
            // ---- does a unit come before it with a point in its ball? ----
            if (pick) {
                const uint64_t kp = ((uint64_t)f2u(best.v) << 32) | ~best.i;
                auto holds = [&](const u32x4 &e0, const u32x4 &e1, const u32x4 &e2, int c) {
                    const bool above = c < nrl && ((((uint64_t)e0.x << 32) | ~e0.y) > kp);
                    if (__builtin_amdgcn_ballot_w64(above) == 0) return false;
                    bool blk = sqdist(u2f(e1.x), u2f(e1.y), u2f(e1.z), best.x, best.y, best.z) < best.v;
                    bool more = u2f(e0.z) >= best.v;
                    if constexpr (TWO) {
                        blk = blk | (more & (sqdist(u2f(e2.x), u2f(e2.y), u2f(e2.z), best.x, best.y, best.z) < best.v));
                        more = u2f(e0.w) >= best.v;
                    }
                    more = more & above;
                    blk = blk & above;
                    if (__builtin_amdgcn_ballot_w64(more)) {
                        const Box eb = sbox[more ? e1.w : 0u];
                        blk = blk | (more & (box_dist(eb, best.x, best.y, best.z) < best.v));
                    }
                    return __builtin_amdgcn_ballot_w64(blk) != 0;
                };
                pick = !holds(r0, r1, r2, lane);
                for (int c0 = kWave; c0 < nrl && pick; c0 += kWave) {
                    const u32x4 *r = rlist + (TWO ? 3 : 2) * (c0 + lane);
                    pick = !holds(r[0], r[1], r[TWO ? 2 : 0], c0 + lane);
                }
            }
            const float lv = best.v;
            const uint32_t li = best.i;
            if (pick) {
                // beside those that reach the unit, in a lane without one of them
                if (hits == ~0ull) apply_hits();
                const uint64_t to = ~hits & (hits + 1);
                const bool me = __builtin_amdgcn_inverse_ballot_w64(to);
                e.x = me ? f2u(best.x) : e.x; e.y = me ? f2u(best.y) : e.y; e.z = me ? f2u(best.z) : e.z; e.w = me ? f2u(best.v) : e.w;
                hits |= to;
            }
            apply_hits();
            if (changed) best = unit_best<P>(p, m, lane);
            publish(round + 1, pick, false);
            // the list of picks, out of the exchange's way
            if (pick) {
                if (np >= p1 - p0) {  // a point picked twice: coordinates that are not finite
                    bad = true;
                    s_twice = 1;
                } else if (lane == 0) {
                    picks[np] = u32x4{f2u(lv), li, round, 0u};
                    atomicAdd(&hist[local_bin_place(f2u(lv) >> kLocalBinShift)], 1u);
                }
                ++np;
            }
            shrink(tag, round > 1 ? (int)groups : 8 * kSlots);
            if (NS > 1 && cur < NS) {
                ++round;
                return true;
            }
        }
    };
    if (cur != 4 || rounds(std::integral_constant<int, 4>{})) {
        if (cur != 2 || rounds(s2)) rounds(s1);
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
static_assert(kMaxGridWG * kWaves * kUnitMax <= (1 << kIndexBitsOfRecord), "an index and the bound of a record are one word");

}  // namespace

// Workgroups of a cloud.  A row of points per unit is where a unit costs least, but smaller ones make fewer rounds, as
// long as there are not so many that the first rounds, in which all see all, cost more than that saves.  us with
// 512, 256 and 171 points per workgroup: 9000 points to 4000 435, 342, 318 (128 points: 295); 16,384 to 4096 369, 333, 316;
// 30,000 of a room to 2000 295, 288, 318; 30,000 of a LiDAR frame to 2500 465, 368, 359; 45,678 to 5001 341, 355, 364.
// So up to 88 workgroups have down to 128 points; the line is where 88 of them have 512 points each, 45,056.  With 512 points, 88
// workgroups and 256 points, a cube / a room / planes / LiDAR: 34,000 to 3777 356, 344, 385 / 324, 319, 319 / 363, 352, 377 / 388, 351,
// 357; 42,000 to 4666 377, 365, 414 / 341, 333, 347 / 388, 382, 395 / 368, 370, 355; 45,678 to 5075 381, 394, 402 / 345, 358, 351 / 382,
// 398, 389 / 388, 424, 375; 64,000 to 7111 401, 418, 441 / 368, 393, 400 / 417, 439, 439 / 448, 479, 450.
// With a quarter of the points as samples most rounds are late ones: 60,000
// to 25,000 500, 462, 472; 120,000 to 30,000 591, 561, 568; 60,000 to 5000 326, 339, 351: 256 points there.
LocalPlan plan_fps_local(int B, int N, int M, int num_cu) {
    const int maxG = num_cu < kMaxGridWG ? num_cu : kMaxGridWG;
    LocalPlan p = {0, 0, 0};
    const int need = (N + kWaves * kUnitMax - 1) / (kWaves * kUnitMax);
    if (need > maxG) return p;
    auto per = [&](int points) { return (N + points - 1) / points; };
    int g = per(kThreads);
    if (g < 88) g = per(128) < 88 ? per(128) : 88;
    if ((long)M * 4 >= N && g < per(256)) g = per(256);
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
    l.exchange_bytes_per_cloud = (size_t)kPlanes * p.units_per_cloud * 16;
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
    LocalPlan p = plan_fps_local(B, N, N, kMaxGridWG);  // nor has fewer samples more of them
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
