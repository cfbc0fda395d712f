// The two sorts around k_fps_local (fps_local.hip): the points along a space-filling curve
// before it, the picks by (value descending, index ascending) after it.
//
// Points: 15-bit Hilbert codes of a 32^3 grid over the cloud (finer grids make no fewer rounds:
// a unit of 98 points of the 200,000-point room covers about two cells) or, for a cloud that does not fill
// its box, 15-bit keys that ascend with 30-bit codes (fps_space.h: 256 splitters, 128 places between two);
// a radix sort of 8 and 7 bits.  Both passes are stable, so the order, and with it every round of the
// kernel, is the same in each run.  Five launches: boxes of tiles; keys and counts of the low digit; low digit;
// counts of the high digit in tiles of that order; high digit.  The points themselves move in both passes (gathered at random
// by the second one alone, five million took 104 us there and 34 in the first).
// A block adds up the counts of all tiles itself instead of a scan of its own.  (The high digits
// counted by the pass that moves the low ones, with an atomic in memory per point, took 256 us of
// five million points; the pass and the counts by themselves took 60 and 18 us then.)
//
// Picks: k_fps_local counts them in 8192 bins by value (32 bins to a factor of two), so a pick's
// bin is known at once; bins are sorted in LDS, by 1024 sub-bins first.
#include "fps_device.h"
#include "fps_launch.h"
#include "fps_local.h"
#include "fps_space.h"

namespace ffps {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kOT = 512;               // threads of the ordering kernels
constexpr int kOW = kOT / kWave;
constexpr int kLowBins = 256, kHighBins = 128;  // 15 code bits in two digits

// First and last point of a tile.
__device__ __forceinline__ void tile_range(int N, int tiles, int t, int &lo, int &hi) {
    const int per = ((N + tiles - 1) / tiles + kOT - 1) / kOT * kOT;
    lo = min(N, t * per);
    hi = min(N, lo + per);
}

// Sum over the lanes up to this one, and over the waves of the block before it: an exclusive prefix; `total` receives the sum.
template <int WAVES>
__device__ __forceinline__ uint32_t block_before(uint32_t v, uint32_t *part, int tid, uint32_t *total) {
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t s = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = __shfl_up(s, o);
        s += lane >= o ? u : 0u;
    }
    if (lane == 63) part[wave] = s;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t c = part[w];
        before += w < wave ? c : 0u;
        all += c;
    }
    *total = all;
    return before + s - v;
}
// Points of a thread that are on their way at once in the passes over a cloud.  One after another, five million points
// took 20, 28 and 18 us (boxes, keys, counts), 12, 26 and 19 now, and 62 and 116 us the two passes that move them, 44 and 41 now.
constexpr int kTogether = 4;

struct Ext { float lo[3], hi[3]; };

__device__ __forceinline__ void block_box(Ext &e, float (*sh)[6], int tid) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            e.lo[k] = fminf(e.lo[k], __shfl_xor(e.lo[k], o));
            e.hi[k] = fmaxf(e.hi[k], __shfl_xor(e.hi[k], o));
        }
    }
    if ((tid & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            sh[tid >> 6][k] = e.lo[k];
            sh[tid >> 6][3 + k] = e.hi[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        for (int v = 0; v < kOW; ++v) {
            e.lo[k] = fminf(e.lo[k], sh[v][k]);
            e.hi[k] = fmaxf(e.hi[k], sh[v][3 + k]);
        }
    }
}

// Box of each tile; clears the words the later kernels count and poll in.
__global__ __launch_bounds__(kOT) void k_order_box(const float *__restrict__ xyz, int N, int tiles, float *__restrict__ boxes,
                                                   uint32_t *__restrict__ zero, long zero_words, int *__restrict__ status) {
    __shared__ float sh[kOW][6];
    const int tid = threadIdx.x, t = blockIdx.x, b = blockIdx.y;
    const long nthr = (long)gridDim.x * gridDim.y * kOT, me = ((long)b * gridDim.x + t) * kOT + tid;
    for (long i = me; i < zero_words; i += nthr) zero[i] = 0u;
    if (status && me < kStatusWords) status[me] = 0;
    int lo, hi;
    tile_range(N, tiles, t, lo, hi);
    const float *p = xyz + (size_t)b * N * 3;
    Ext e;
#pragma unroll
    for (int k = 0; k < 3; ++k) { e.lo[k] = __builtin_inff(); e.hi[k] = -__builtin_inff(); }
    for (int i0 = lo + tid; i0 < hi; i0 += kTogether * kOT) {
        float v[kTogether][3];
#pragma unroll
        for (int j = 0; j < kTogether; ++j) {
            const float *q = p + 3 * (size_t)min(i0 + j * kOT, hi - 1);
            v[j][0] = q[0]; v[j][1] = q[1]; v[j][2] = q[2];
        }
#pragma unroll
        for (int j = 0; j < kTogether; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                e.lo[k] = fminf(e.lo[k], v[j][k]);
                e.hi[k] = fmaxf(e.hi[k], v[j][k]);
            }
    }
    block_box(e, sh, tid);
    if (tid < 6) boxes[((size_t)b * tiles + t) * 6 + tid] = tid < 3 ? e.lo[tid] : e.hi[tid - 3];
}

// Frame and splitters of a cloud that does not fill its box, from one point of each of 256 stretches of it.
// Every block finds the same ones by itself (about 3 us, in clouds of this kind alone).
constexpr int kSplitBits = 8, kSplitters = 1 << kSplitBits, kPlaces = 128, kCodeBits = 10;  // code bits per axis
static_assert(2 * kSplitters == kOT && kSplitters * kPlaces == kLowBins * kHighBins, "two threads per splitter; keys of two digits");
struct Splits {
    float co[3][kSplitters];
    Spread part[3];
    __attribute__((aligned(16))) uint32_t codes[kSplitters];
    uint32_t rank[kSplitters];
    uint32_t at[kSplitters + 1];  // the splitters
    float per[kSplitters];        // places per code from one to the next
};
__device__ __forceinline__ Frame find_splitters(const float *__restrict__ p, int N, int tid, Splits &sh) {
    const int lane = tid & 63, wave = tid >> 6, j = tid & (kSplitters - 1);
    const float *q = p + (size_t)sample_index<kSplitBits>(j, N) * 3;
    const float x = q[0], y = q[1], z = q[2];
    if (tid < kSplitters) {
        sh.co[0][j] = x; sh.co[1][j] = y; sh.co[2][j] = z;
        sh.rank[j] = 0u;
    }
    __syncthreads();
    if (wave < 3) {
        const Spread s = spread_of(sh.co[wave][lane * (kSplitters / kFramePoints)], lane);
        if (lane == 0) sh.part[wave] = s;
    }
    __syncthreads();
    const Spread parts[3] = {sh.part[0], sh.part[1], sh.part[2]};
    const Frame f = frame_of(parts);
    // the last bits of a code tell equal ones apart
    const uint32_t code = (code_of<kCodeBits>(f, x, y, z) & ~(uint32_t)(kSplitters - 1)) | (uint32_t)j;
    if (tid < kSplitters) sh.codes[j] = code;
    __syncthreads();
    // a splitter's place: the two threads of it compare one half of the others each
    const int h0 = tid < kSplitters ? 0 : kSplitters / 2;
    uint32_t n = 0;
#pragma unroll 8
    for (int i = h0; i < h0 + kSplitters / 2; i += 4) {
        const u32x4 o = *reinterpret_cast<const u32x4 *>(&sh.codes[i]);
        n += (o.x < code ? 1u : 0u) + (o.y < code ? 1u : 0u) + (o.z < code ? 1u : 0u) + (o.w < code ? 1u : 0u);
    }
    atomicAdd(&sh.rank[j], n);
    __syncthreads();
    if (tid < kSplitters) sh.at[sh.rank[j]] = sh.rank[j] ? code : 0u;
    if (tid == kSplitters) sh.at[kSplitters] = 1u << (3 * kCodeBits);
    __syncthreads();
    if (tid < kSplitters) sh.per[tid] = (float)kPlaces / (float)(sh.at[tid + 1] - sh.at[tid]);
    __syncthreads();
    return f;
}

// Keys, and how often each low digit occurs in a tile.
__global__ __launch_bounds__(kOT) void k_order_code(const float *__restrict__ xyz, int N, int tiles, const float *__restrict__ boxes,
                                                    uint16_t *__restrict__ codes, uint32_t *__restrict__ hist) {
    __shared__ float sh[kOW][6];
    __shared__ uint32_t cnt[kLowBins];
    __shared__ Splits sp;
    const int tid = threadIdx.x, t = blockIdx.x, b = blockIdx.y;
    const float *p = xyz + (size_t)b * N * 3;
    const float *q = p + (size_t)sample_index<kSplitBits>((tid & 63) * (kSplitters / kFramePoints), N) * 3;
    const float qx = q[0], qy = q[1], qz = q[2];
    if (tid < kLowBins) cnt[tid] = 0;
    Ext e;
#pragma unroll
    for (int k = 0; k < 3; ++k) { e.lo[k] = __builtin_inff(); e.hi[k] = -__builtin_inff(); }
    for (int i = tid; i < tiles; i += kOT) {
        const float *q = boxes + ((size_t)b * tiles + i) * 6;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            e.lo[k] = fminf(e.lo[k], q[k]);
            e.hi[k] = fmaxf(e.hi[k], q[3 + k]);
        }
    }
    block_box(e, sh, tid);
    const float side = fmaxf(fmaxf(e.hi[0] - e.lo[0], e.hi[1] - e.lo[1]), e.hi[2] - e.lo[2]);
    const float scale = side > 0.f ? 32.f / side : 0.f;
    int lo, hi;
    tile_range(N, tiles, t, lo, hi);
    auto put = [&](int i, uint32_t key) {
        codes[(size_t)b * N + i] = (uint16_t)key;
        atomicAdd(&cnt[key & (kLowBins - 1)], 1u);
    };
    if (fills_box(qx, qy, qz, e.lo, side)) {
        for (int i0 = lo + tid; i0 < hi; i0 += kTogether * kOT) {
            float v[kTogether][3];
#pragma unroll
            for (int j = 0; j < kTogether; ++j) {
                const float *q = p + 3 * (size_t)min(i0 + j * kOT, hi - 1);
                v[j][0] = q[0]; v[j][1] = q[1]; v[j][2] = q[2];
            }
#pragma unroll
            for (int j = 0; j < kTogether; ++j) {
                uint32_t c[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) c[k] = (uint32_t)fmaxf(0.f, fminf(31.f, (v[j][k] - e.lo[k]) * scale));
                const uint32_t key = hilbert_code<5>(c[0], c[1], c[2]);
                if (i0 + j * kOT < hi) put(i0 + j * kOT, key);
            }
        }
    } else {
        const Frame f = find_splitters(p, N, tid, sp);
        for (int i0 = lo + tid; i0 < hi; i0 += kTogether * kOT) {
            uint32_t code[kTogether], s[kTogether];
#pragma unroll
            for (int k = 0; k < kTogether; ++k) {
                const float *v = p + 3 * (size_t)min(i0 + k * kOT, hi - 1);
                code[k] = code_of<kCodeBits>(f, v[0], v[1], v[2]);
            }
#pragma unroll
            for (int k = 0; k < kTogether; ++k) s[k] = splitter_of<kSplitBits>(sp.at, code[k]);
#pragma unroll
            for (int k = 0; k < kTogether; ++k) {
                const uint32_t place = umin(kPlaces - 1, (uint32_t)((float)(code[k] - sp.at[s[k]]) * sp.per[s[k]]));
                if (i0 + k * kOT < hi) put(i0 + k * kOT, s[k] * kPlaces + place);
            }
        }
    }
    __syncthreads();
    if (tid < kLowBins) hist[((size_t)b * tiles + t) * kLowBins + tid] = cnt[tid];
}

// One pass of a stable radix sort: a block moves the elements of its tile behind those of
// earlier tiles and, within the tile, behind those of earlier waves.  `get(i)` is element i, `digit(e)` its digit, `fetch(e, i)` what `put(x, pos)` puts in its place.  What bounds it is latency, so elements are loaded, and moved, a
// few rows at a time, the first rows before the counts of the tiles; these are added up by all threads, some to a digit.
template <int BITS>
struct PassShared {
    uint32_t cnt[kOW][1 << BITS], before[kOT], total[kOT], part[kOW];
};
template <int BITS, typename G, typename D, typename F, typename PU>
__device__ __forceinline__ void stable_pass(const uint32_t *__restrict__ hist, int tiles, int t, int lo, int hi, int tid,
                                            PassShared<BITS> &sh, G get, D digit, F fetch, PU put) {
    constexpr int NB = 1 << BITS, kRows = 8;
    static_assert(NB <= kOT && kOT % NB == 0, "threads per digit");
    const int lane = tid & 63, wave = tid >> 6;
    const int rows = (hi - lo + kOT - 1) / kOT, w0 = lo + wave * rows * kWave + lane;
    decltype(get(0)) e[kRows];
    auto on = [&](int r) { return r < rows && w0 + r * kWave < hi; };
    auto load = [&](int r0) {
#pragma unroll
        for (int k = 0; k < kRows; ++k) e[k] = get(min(w0 + (r0 + k) * kWave, hi - 1));  // others' are not used
    };
    load(0);
    for (int i = tid; i < kOW * NB; i += kOT) (&sh.cnt[0][0])[i] = 0;
    // elements of each digit in earlier tiles, and in all of them
    uint32_t before = 0, total = 0;
#pragma unroll 8
    for (int k = tid / NB; k < tiles; k += kOT / NB) {
        const uint32_t h = hist[(size_t)k * NB + (tid & (NB - 1))];
        before += k < t ? h : 0u;
        total += h;
    }
    sh.before[tid] = before;
    sh.total[tid] = total;
    __syncthreads();
    if (tid < NB) {
#pragma unroll
        for (int g = NB; g < kOT; g += NB) {
            before += sh.before[g + tid];
            total += sh.total[g + tid];
        }
    }
    for (int r0 = 0;;) {
#pragma unroll
        for (int k = 0; k < kRows; ++k)
            if (on(r0 + k)) atomicAdd(&sh.cnt[wave][digit(e[k])], 1u);
        r0 += kRows;
        if (r0 >= rows) break;
        load(r0);
    }
    if (rows > kRows) load(0);
    uint32_t all;
    uint32_t at = block_before<kOW>(tid < NB ? total : 0u, sh.part, tid, &all) + before;
    if (tid < NB) {
        for (int v = 0; v < kOW; ++v) {
            const uint32_t c = sh.cnt[v][tid];
            sh.cnt[v][tid] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int r0 = 0;;) {
        uint32_t pos[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const bool ok = on(r0 + k);
            const uint32_t d = digit(e[k]);
            const uint64_t m = same_digit<BITS>(d, __builtin_amdgcn_ballot_w64(ok));
            const uint32_t base = sh.cnt[wave][d];
            const int r_in = lanes_below(m);
            wave_lds_order();  // all lanes have read the count
            if (ok && r_in == 0) sh.cnt[wave][d] = base + (uint32_t)__builtin_popcountll(m);
            wave_lds_order();  // and it is written before the next row reads it
            pos[k] = base + r_in;
        }
        decltype(fetch(e[0], 0)) x[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) x[k] = fetch(e[k], min(w0 + (r0 + k) * kWave, hi - 1));
#pragma unroll
        for (int k = 0; k < kRows; ++k)
            if (on(r0 + k)) put(x[k], pos[k]);
        r0 += kRows;
        if (r0 >= rows) break;
        load(r0);
    }
}

// A point on its way: in its last word the index below, the high digit above.
constexpr int kIndexBits = 25;

__global__ __launch_bounds__(kOT) void k_order_low(const float *__restrict__ xyz, int N, int tiles, const uint16_t *__restrict__ codes,
                                                   const uint32_t *__restrict__ hist, u32x4 *__restrict__ elems) {
    __shared__ PassShared<8> sh;
    const int tid = threadIdx.x, t = blockIdx.x, b = blockIdx.y;
    int lo, hi;
    tile_range(N, tiles, t, lo, hi);
    const uint16_t *c = codes + (size_t)b * N;
    const float *p = xyz + (size_t)b * N * 3;
    u32x4 *out = elems + (size_t)b * N;
    stable_pass<8>(hist + (size_t)b * tiles * kLowBins, tiles, t, lo, hi, tid, sh, [&](int i) { return (uint32_t)c[i]; },
                   [&](uint32_t e) { return e & (kLowBins - 1); },
                   [&](uint32_t e, int i) {
                       const float *q = p + 3 * (size_t)i;
                       return u32x4{f2u(q[0]), f2u(q[1]), f2u(q[2]), (e >> 8) << kIndexBits | (uint32_t)i};
                   },
                   [&](const u32x4 &x, uint32_t pos) { out[pos] = x; });
}

// How often each high digit occurs in a tile.
__global__ __launch_bounds__(kOT) void k_order_count(int N, int tiles, const u32x4 *__restrict__ elems, uint32_t *__restrict__ hist2) {
    __shared__ uint32_t cnt[kHighBins];
    const int tid = threadIdx.x, t = blockIdx.x, b = blockIdx.y;
    if (tid < kHighBins) cnt[tid] = 0;
    __syncthreads();
    int lo, hi;
    tile_range(N, tiles, t, lo, hi);
    const u32x4 *in = elems + (size_t)b * N;
    for (int i0 = lo + tid; i0 < hi; i0 += kTogether * kOT) {
        uint32_t e[kTogether];
#pragma unroll
        for (int j = 0; j < kTogether; ++j) e[j] = in[min(i0 + j * kOT, hi - 1)].w;
#pragma unroll
        for (int j = 0; j < kTogether; ++j)
            if (i0 + j * kOT < hi) atomicAdd(&cnt[e[j] >> kIndexBits], 1u);
    }
    __syncthreads();
    if (tid < kHighBins) hist2[((size_t)b * tiles + t) * kHighBins + tid] = cnt[tid];
}

__global__ __launch_bounds__(kOT) void k_order_high(int N, int tiles, const u32x4 *__restrict__ elems,
                                                    const uint32_t *__restrict__ hist2, u32x4 *__restrict__ pts) {
    __shared__ PassShared<7> sh;
    const int tid = threadIdx.x, t = blockIdx.x, b = blockIdx.y;
    int lo, hi;
    tile_range(N, tiles, t, lo, hi);
    const u32x4 *in = elems + (size_t)b * N;
    u32x4 *out = pts + (size_t)b * N;
    stable_pass<7>(hist2 + (size_t)b * tiles * kHighBins, tiles, t, lo, hi, tid, sh, [&](int i) { return in[i]; },
                   [&](const u32x4 &e) { return e.w >> kIndexBits; },
                   [&](const u32x4 &e, int) { return u32x4{e.x, e.y, e.z, e.w & ((1u << kIndexBits) - 1u)}; },
                   [&](const u32x4 &x, uint32_t pos) { out[pos] = x; });
}

// ---- the picks in their order ----------------------------------------------------
constexpr int kFT = 1024;
constexpr int kSortMax = 2048;  // picks of a bin that are sorted in LDS: those of a room of 50,000 samples are 900 to 1800
constexpr int kSubBits = 10, kSubBins = 1 << kSubBits;  // next bits of a value
constexpr uint32_t kSubMax = 64;                        // picks that share them and are compared with one another

struct FinishArgs {
    int N, M, U;                // points, samples, units of a cloud
    const int *start_dev;
    int start;
    const u32x4 *picks;         // [B][N] per unit {value, index, round, -}
    const int *npicks;          // [B][U]
    const uint32_t *hist;       // [B][kLocalWords]: picks per bin
    uint32_t *cursor;           // [B][kLocalBins], zero
    u32x2 *runs;                // [B][kLocalBins] {first place, picks} of the bins in use
    int *nruns;                 // [B]
    uint64_t *keys;             // [B][N]
    uint64_t *spare;            // [B][2 N]: the lists, which are done with by the time it is used
    int32_t *idx;
    long idx_stride;
    float *md;
    long md_stride;
    int *status;
};

// Place of a bin in LDS, where neighbours and every 64th bin lie in different banks.
__device__ __forceinline__ uint32_t bank_place(uint32_t bin) { return bin ^ ((bin >> 6) & 31u); }

// Places of the bins (largest values first), then every pick into its bin.  What bounds it is latency: of the counts, which
// are read as they lie, of two scans and of two passes over lists of a few picks, a row of 16 lanes for each of 64 units at once.
__global__ __launch_bounds__(kFT) void k_finish_bins(FinishArgs a) {
    __shared__ uint32_t base[kLocalBins], cnt[kLocalBins], part[2 * (kFT / kWave)];
    const int tid = threadIdx.x, b = blockIdx.y;
    const uint32_t *hist = a.hist + (size_t)b * kLocalWords;
    constexpr int per = kLocalBins / kFT;
    {
        uint32_t h[per];
#pragma unroll
        for (int k = 0; k < per; ++k) h[k] = hist[k * kFT + tid];
#pragma unroll
        for (int k = 0; k < per; ++k) {
            const uint32_t w = (uint32_t)(k * kFT + tid), bin = (w & 127u) << 6 | w >> 7;
            cnt[bank_place(bin)] = h[k];
        }
        static_assert(kLocalBins == 64 * 128, "the inverse of local_bin_place");
    }
    __syncthreads();
    // thread t: bins kLocalBins - 1 - t * per downwards
    uint32_t h[per], sum = 0, used = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        h[k] = cnt[bank_place(kLocalBins - 1 - (tid * per + k))];
        sum += h[k];
        used += h[k] ? 1u : 0u;
    }
    uint32_t total;
    const uint32_t first = block_before<kFT / kWave>(sum, part, tid, &total);
    uint32_t at = first;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const uint32_t place = bank_place(kLocalBins - 1 - (tid * per + k));
        base[place] = at;
        cnt[place] = 0;
        at += h[k];
    }
    if (blockIdx.x == 0) {
        // the bins that hold samples, for the next kernel; samples beyond the picks repeat point 0
        const uint32_t n = first < (uint32_t)(a.M - 1) ? used : 0u;
        uint32_t runs;
        uint32_t r = block_before<kFT / kWave>(n, part + kFT / kWave, tid, &runs);
        if (n) {
            uint32_t p = first;
#pragma unroll
            for (int k = 0; k < per; ++k) {
                if (h[k]) a.runs[(size_t)b * kLocalBins + r++] = u32x2{p, h[k]};
                p += h[k];
            }
        }
        if (tid == 0) {
            a.nruns[b] = (int)runs;
            a.idx[b * a.idx_stride] = a.start_dev ? a.start_dev[b] : a.start;
            if (a.md) a.md[b * a.md_stride] = __builtin_inff();
        }
        for (uint32_t k = total + tid; k < (uint32_t)(a.M - 1); k += kFT) {
            a.idx[b * a.idx_stride + 1 + k] = 0;
            if (a.md) a.md[b * a.md_stride + 1 + k] = 0.f;
        }
    }
    __syncthreads();
    // units of this block, a row of lanes each
    const int u0 = (int)((long)blockIdx.x * a.U / gridDim.x), u1 = (int)((long)(blockIdx.x + 1) * a.U / gridDim.x);
    const int row = tid >> 4, l16 = tid & 15;
    const u32x4 *picks = a.picks + (size_t)b * a.N;
    auto bin_of = [](uint32_t v) { return bank_place((v >> kLocalBinShift) & (kLocalBins - 1)); };
    for (int u = u0 + row; u < u1; u += kFT / 16) {
        const u32x4 *l = picks + (int)((long)u * a.N / a.U);
        const int n = a.npicks[(size_t)b * a.U + u];
        for (int k = l16; k < n; k += 16) atomicAdd(&cnt[bin_of(l[k].x)], 1u);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const uint32_t bin = (uint32_t)(k * kFT + tid), place = bank_place(bin), c = cnt[place];
        if (c) cnt[place] = base[place] + atomicAdd(&a.cursor[(size_t)b * kLocalBins + bin], c);
    }
    __syncthreads();
    uint32_t rounds = 0;
    for (int u = u0 + row; u < u1; u += kFT / 16) {
        const u32x4 *l = picks + (int)((long)u * a.N / a.U);
        const int n = a.npicks[(size_t)b * a.U + u];
        for (int k = l16; k < n; k += 16) {
            const u32x4 p = l[k];
            const uint32_t place = bin_of(p.x);
            if (base[place] < (uint32_t)(a.M - 1)) rounds = umax(rounds, p.z);
            const uint32_t pos = atomicAdd(&cnt[place], 1u);
            a.keys[(size_t)b * a.N + pos] = ((uint64_t)p.x << 32) | (uint32_t)~p.y;
        }
    }
    rounds = wave_max_u32(rounds);
    if ((tid & 63) == 0 && rounds) __hip_atomic_fetch_max(a.status + 1, (int)rounds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sorts each bin (descending keys) and writes the samples.  A bitonic sort of each bin in LDS took 39 us of 50,000 samples of
// 200,000 points; by sub-bins 7.  (The kernel above: 30 us of eight clouds of 4096 samples with each bin read where it
// lies, a wave per unit and 32 blocks per cloud; 12.)
__global__ __launch_bounds__(256) void k_finish_sort(FinishArgs a) {
    __shared__ uint64_t s[kSortMax];
    __shared__ uint32_t sub[kSubBins];
    __shared__ uint32_t cnt[256], part[4], most[4];
    const int tid = threadIdx.x, b = blockIdx.y, wave = tid >> 6;
    const int n_runs = a.nruns[b];
    auto put = [&](uint32_t place, uint64_t key) {
        if (place < (uint32_t)(a.M - 1)) {
            a.idx[b * a.idx_stride + 1 + place] = (int32_t)~(uint32_t)key;
            if (a.md) a.md[b * a.md_stride + 1 + place] = u2f((uint32_t)(key >> 32));
        }
    };
    for (int j = blockIdx.x; j < n_runs; j += gridDim.x) {
        const u32x2 run = a.runs[(size_t)b * kLocalBins + j];
        uint64_t *keys = a.keys + (size_t)b * a.N + run.x;
        const int n = (int)run.y;
        if (n <= kSortMax) {
            // by the next bits of the value, then among those that share them
            uint64_t key[kSortMax / 256];
            uint32_t at[kSortMax / 256];
#pragma unroll
            for (int k = 0; k < kSubBins / 256; ++k) sub[tid + k * 256] = 0;
#pragma unroll
            for (int k = 0; k < kSortMax / 256; ++k) {
                const int i = tid + k * 256;
                key[k] = i < n ? keys[i] : 0ull;
            }
            __syncthreads();
            auto sub_of = [](uint64_t x) { return kSubBins - 1 - (((uint32_t)(x >> 32) >> (kLocalBinShift - kSubBits)) & (kSubBins - 1)); };
#pragma unroll
            for (int k = 0; k < kSortMax / 256; ++k) at[k] = tid + k * 256 < n ? atomicAdd(&sub[sub_of(key[k])], 1u) : 0u;
            __syncthreads();
            uint32_t c[kSubBins / 256], sum = 0, top = 0;
#pragma unroll
            for (int k = 0; k < kSubBins / 256; ++k) {
                c[k] = sub[tid * (kSubBins / 256) + k];
                sum += c[k];
                top = umax(top, c[k]);
            }
            top = wave_max_u32(top);
            if ((tid & 63) == 0) most[wave] = top;
            uint32_t all;
            uint32_t p = block_before<4>(sum, part, tid, &all);
            top = umax(umax(most[0], most[1]), umax(most[2], most[3]));
#pragma unroll
            for (int k = 0; k < kSubBins / 256; ++k) {
                sub[tid * (kSubBins / 256) + k] = p;
                p += c[k];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kSortMax / 256; ++k)
                if (tid + k * 256 < n) s[sub[sub_of(key[k])] + at[k]] = key[k];
            __syncthreads();
            if (top <= kSubMax) {
                for (int i = tid; i < n; i += 256) {
                    const uint64_t x = s[i];
                    const uint32_t d = sub_of(x), e0 = sub[d], e1 = d + 1 < kSubBins ? sub[d + 1] : (uint32_t)n;
                    uint32_t place = e0;
                    for (uint32_t e = e0; e < e1; ++e) place += s[e] > x ? 1u : 0u;
                    put(run.x + place, x);
                }
                __syncthreads();
                continue;
            }
            // many of nearly one value
            int size = 2;
            while (size < n) size <<= 1;
            for (int i = n + tid; i < size; i += 256) s[i] = 0ull;
            __syncthreads();
            for (int k = 2; k <= size; k <<= 1) {
                for (int o = k >> 1; o > 0; o >>= 1) {
                    for (int i = tid; i < size / 2; i += 256) {
                        const int p = 2 * i - (i & (o - 1)), q = p + o;
                        const uint64_t x = s[p], y = s[q];
                        const bool up = (p & k) != 0;  // ascending half
                        if ((x < y) != up) { s[p] = y; s[q] = x; }
                    }
                    __syncthreads();
                }
            }
            for (int i = tid; i < n; i += 256) put(run.x + i, s[i]);
            __syncthreads();
        } else {
            // many picks of nearly one value (lattices): a radix sort of the complements by this
            // block alone, 8 bits at a time, four waves taking 64 keys each in turn
            uint64_t *src = keys, *dst = a.spare + (size_t)b * 2 * a.N + run.x;
            for (int shift = 0; shift < 64; shift += 8) {
                cnt[tid] = 0;
                __syncthreads();
                for (int i = tid; i < n; i += 256) atomicAdd(&cnt[(uint32_t)(~src[i] >> shift) & 255u], 1u);
                __syncthreads();
                const uint32_t own = cnt[tid];
                for (int o = 1; o < 256; o <<= 1) {
                    const uint32_t v = tid >= o ? cnt[tid - o] : 0u;
                    __syncthreads();
                    cnt[tid] += v;
                    __syncthreads();
                }
                const uint32_t at = cnt[tid] - own;
                __syncthreads();
                cnt[tid] = at;
                const bool one_digit = __syncthreads_or(own == (uint32_t)n);
                if (one_digit) continue;
                for (int i0 = 0; i0 < n; i0 += 256) {
                    const int i = i0 + tid;
                    const bool ok = i < n;
                    const uint64_t key = ok ? src[i] : 0ull;
                    const uint32_t d = (uint32_t)(~key >> shift) & 255u;
                    const uint64_t m = same_digit<8>(d, __builtin_amdgcn_ballot_w64(ok));
                    for (int v = 0; v < 4; ++v) {
                        if (wave == v) {
                            const uint32_t base = cnt[d];
                            const int r_in = lanes_below(m);
                            wave_lds_order();  // all lanes have read the count
                            if (ok && r_in == 0) cnt[d] = base + (uint32_t)__builtin_popcountll(m);
                            if (ok) dst[base + r_in] = key;
                        }
                        __syncthreads();
                    }
                }
                uint64_t *t = src; src = dst; dst = t;
                __syncthreads();
            }
            for (int i = tid; i < n; i += 256) put(run.x + i, src[i]);
            __syncthreads();
        }
    }
}

}  // namespace

int order_tiles(int N) {
    const int t = (N + 2047) / 2048;
    return t < 1 ? 1 : t > 256 ? 256 : t;
}

hipError_t launch_order(const float *xyz, int B, int N, const LocalBuffers &l, int *clear_status, hipStream_t s) {
    if (N > 1 << kIndexBits) return hipErrorInvalidValue;
    const int tiles = order_tiles(N);
    const dim3 grid(tiles, B);
    u32x4 *elems = (u32x4 *)l.picks;  // the picks come later
    k_order_box<<<grid, dim3(kOT), 0, s>>>(xyz, N, tiles, l.boxes, (uint32_t *)l.zeroed, (long)(l.zero_bytes / 4), clear_status);
    k_order_code<<<grid, dim3(kOT), 0, s>>>(xyz, N, tiles, l.boxes, l.codes, l.hist1);
    k_order_low<<<grid, dim3(kOT), 0, s>>>(xyz, N, tiles, l.codes, l.hist1, elems);
    k_order_count<<<grid, dim3(kOT), 0, s>>>(N, tiles, elems, l.hist2);
    k_order_high<<<grid, dim3(kOT), 0, s>>>(N, tiles, elems, l.hist2, (u32x4 *)l.pts);
    return hipGetLastError();
}

hipError_t launch_finish(const LocalBuffers &l, int B, int N, int M, int units, int start, const int *start_dev, int32_t *idx, long idx_stride,
                         float *md, long md_stride, int *status, hipStream_t s) {
    FinishArgs a;
    a.N = N; a.M = M; a.U = units; a.start = start; a.start_dev = start_dev;
    a.picks = (const u32x4 *)l.picks; a.npicks = l.npicks; a.hist = l.hist; a.cursor = l.cursor;
    a.runs = (u32x2 *)l.runs; a.nruns = l.nruns; a.keys = (uint64_t *)l.pts; a.spare = (uint64_t *)l.picks;
    a.idx = idx; a.idx_stride = idx_stride; a.md = md; a.md_stride = md_stride; a.status = status;
    // a unit per row of lanes; with many clouds no more blocks than CUs, since all of a cloud scan its 8192 bins
    const int rows = kFT / 16, full = (units + rows - 1) / rows, share = 256 / B > 1 ? 256 / B : 1;
    const int gb = full < share ? full : share;
    k_finish_bins<<<dim3(gb, B), dim3(kFT), 0, s>>>(a);
    k_finish_sort<<<dim3(B >= 8 ? 64 : 256, B), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace ffps
