// Index bookkeeping around the FPS loop: candidate pruning and the fill of
// FPS-Prune (Alg. 1, layer 1), and the gathers / prefix copies of the stage
// chain (Alg. 1, layers 2..L; Sec. 3.3).  All O(N) integer work.
#include "fps_device.h"
#include "fps_launch.h"

namespace ffps {

namespace {

constexpr int kT = 256;

inline int blocks_for(size_t n, int per_block = kT, int cap = 4096) {
    size_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (size_t)cap) b = cap;
    return (int)b;
}

__global__ void k_fill_zero(uint32_t *p, size_t words) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < words;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// Position i of the ascending candidate list.  The raw list
// raw[j] = (start + floor(j*N/Nc)) mod N wraps once, at j0; the sorted list is
// the wrapped tail followed by the unwrapped head, i.e. raw[(i + j0) mod Nc].
__device__ __forceinline__ int cand_at(int i, int N, int Nc, int start, int j0) {
    long j = (long)i + j0;
    if (j >= Nc) j -= Nc;
    return (int)(((long)start + (j * (long)N) / Nc) % N);
}

// What a later launch of the call needs cleared, by the threads of this one: a launch for it alone takes 4.5 us.
__device__ __forceinline__ void also_clear(const Cleared &c) {
    const size_t me = (blockIdx.y * (size_t)gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t all = (size_t)gridDim.x * gridDim.y * blockDim.x;
    if (c.status && me < (size_t)kStatusWords) c.status[me] = 0;
    for (size_t i = me; i < c.words; i += all) c.bitmap[i] = 0u;
}

__global__ void k_gather_candidates(const float *__restrict__ xyz, int N, int Nc, int start, int j0,
                                    float *__restrict__ cxyz, Cleared clear) {
    also_clear(clear);
    const int b = blockIdx.y;
    const float *src = xyz + (size_t)b * N * 3;
    float *dst = cxyz + (size_t)b * Nc * 3;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < Nc; i += gridDim.x * blockDim.x) {
        int c = cand_at(i, N, Nc, start, j0);
        dst[3 * (size_t)i + 0] = src[3 * (size_t)c + 0];
        dst[3 * (size_t)i + 1] = src[3 * (size_t)c + 1];
        dst[3 * (size_t)i + 2] = src[3 * (size_t)c + 2];
    }
}

// Sample j of the first stage into the prefixes of it that are the deeper ones.
__device__ __forceinline__ void put_prefixes(int32_t *row, int j, int32_t v, const Prefixes &p) {
    for (int l = 0; l < p.n && j < p.len[l]; ++l) row[p.at[l] + j] = v;
}

__global__ void k_map_candidates(const int32_t *__restrict__ loc, long loc_stride, int N, int Nc,
                                 int start, int j0, int k, int32_t *__restrict__ idx,
                                 long idx_stride, uint32_t *__restrict__ marked, Prefixes stages) {
    const int b = blockIdx.y;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < k; j += gridDim.x * blockDim.x) {
        const int c = cand_at(loc[b * loc_stride + j], N, Nc, start, j0);
        idx[b * idx_stride + j] = c;
        put_prefixes(idx + b * idx_stride, j, c, stages);
        if (marked) atomicOr(&marked[(size_t)b * ((N + 31) / 32) + (c >> 5)], 1u << (c & 31));
    }
}

// bm[b] |= the k picks of cloud b (bitmap cleared beforehand)
__global__ void k_mark_picks(int N, int k, const int32_t *__restrict__ idx_all, long idx_stride, uint32_t *__restrict__ bitmap_all) {
    const int b = blockIdx.y;
    uint32_t *bm = bitmap_all + (size_t)b * ((N + 31) / 32);
    const int32_t *idx = idx_all + b * idx_stride;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < k; j += gridDim.x * blockDim.x) {
        const int v = idx[j];
        atomicOr(&bm[v >> 5], 1u << (v & 31));
    }
}

constexpr int kTileBlocks = 256;  // blocks of a cloud at most: each counts the words before its own tiles again

// Exclusive prefix over a block of 1024 of one count per thread; `total` receives the sum.
__device__ __forceinline__ int block_prefix(int cnt, int *part, int tid, int *total) {
    const int lane = tid & 63, wave = tid >> 6;
    int s = cnt;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(s, off);
        s += lane >= off ? v : 0;
    }
    if (lane == 63) part[wave] = s;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const int c = part[w];
        before += w < wave ? c : 0;
        all += c;
    }
    __syncthreads();
    if (total) *total = all;
    return before + s - cnt;
}

// First tile of a block.
__device__ __forceinline__ int first_tile(int tiles, int block, int blocks) { return (int)((long)tiles * block / blocks); }

// Fill of FPS-Prune, a tile of the bitmap per block (beyond 2.1 million points several, so that the
// counting does not grow with the square of the points): ranks of the free indices by popcount
// (a block counts the words of the tiles before its own again: 25 KB for 200,000 points) and
// scan, then every free index decides on its own whether
// some j maps to its rank: fill[j] = free[floor(j*F/R)], F = N - k.  Since
// F >= R the ranks floor(j*F/R) are distinct, and rank r is hit exactly by
// j = ceil(r*R/F) when floor(j*F/R) == r.
// Clouds of one block are marked here as well, in the same launch: their threads take a word each.  Beyond, a thread
// takes a byte, so that there are enough blocks: 200,000 points are 25 of them.  (Seven blocks of 1024 words took
// 10.8 us; one block for clouds of all sizes 51 us.)
template <int BITS>
__global__ __launch_bounds__(1024) void k_fill(int N, int tiles, int k, int R, int32_t *__restrict__ idx_all,
                                               long idx_stride, uint32_t *__restrict__ bitmap_all) {
    __shared__ int part[16];
    constexpr int kTileWords = 1024 * BITS / 32;
    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    const int words = (N + 31) / 32;
    uint32_t *bm = bitmap_all + (size_t)b * words;
    int32_t *idx = idx_all + b * idx_stride;

    if constexpr (BITS == 32) {
        for (int i = tid; i < words; i += 1024) bm[i] = 0u;
        __syncthreads();
        for (int j = tid; j < k; j += 1024) {
            int v = idx[j];
            atomicOr(&bm[v >> 5], 1u << (v & 31));
        }
        __syncthreads();
    }
    int before = 0;
    const int t0 = first_tile(tiles, blockIdx.x, gridDim.x), t1 = first_tile(tiles, blockIdx.x + 1, gridDim.x);
    for (int wd = tid; wd < t0 * kTileWords; wd += 1024) before += __popc(~bm[wd]);
    if (t0 > 0) (void)block_prefix(before, part, tid, &before);
    const long F = (long)N - k;
    for (int tile = t0; tile < t1; ++tile) {
        const int wd = tile * kTileWords + tid / (32 / BITS), bit0 = tid % (32 / BITS) * BITS;
        uint32_t free_bits = 0u;
        if (wd < words) free_bits = ~bm[wd] & ((wd == words - 1 && (N & 31)) ? ((1u << (N & 31)) - 1u) : 0xffffffffu);
        if constexpr (BITS < 32) free_bits &= ((1u << BITS) - 1u) << bit0;
        // Rank r is taken by fill slot j = ceil(r*R/F) iff floor(j*F/R) == r, i.e. iff
        // acc = j*F - r*R lies in [0, R).  One division finds j for the thread's first
        // rank; from rank to rank acc drops by R and, when it goes negative, j steps up.
        int total = 0;
        const long r = before + block_prefix(__popc(free_bits), part, tid, &total);  // rank of the first free index
        before += total;
        long j = (r * R + F - 1) / F;
        long acc = j * F - r * R;
        while (free_bits) {
            const int bit = __ffs(free_bits) - 1;
            free_bits &= free_bits - 1;
            if (acc < R && j < R) idx[k + j] = wd * 32 + bit;
            acc -= R;
            if (acc < 0) {
                ++j;
                acc += F;
            }
        }
    }
}

__global__ void k_gather_points(const float *__restrict__ xyz, int N, const int32_t *__restrict__ sel,
                                long sel_stride, int S, float *__restrict__ dst) {
    const int b = blockIdx.y;
    const float *src = xyz + (size_t)b * N * 3;
    float *out = dst + (size_t)b * S * 3;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < S; j += gridDim.x * blockDim.x) {
        int c = sel[b * sel_stride + j];
        out[3 * (size_t)j + 0] = src[3 * (size_t)c + 0];
        out[3 * (size_t)j + 1] = src[3 * (size_t)c + 1];
        out[3 * (size_t)j + 2] = src[3 * (size_t)c + 2];
    }
}

// out[b][j][0..C) = rows[b][sel[b][j]][0..C): one thread per output float, so
// consecutive threads write consecutive addresses.
__global__ void k_gather_rows(const float *__restrict__ rows, int N, int C,
                              const int32_t *__restrict__ sel, long sel_stride, int S,
                              float *__restrict__ out) {
    const int b = blockIdx.y;
    const float *src = rows + (size_t)b * N * C;
    float *dst = out + (size_t)b * S * C;
    const size_t total = (size_t)S * C;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const size_t j = e / C;
        const int c = (int)(e - j * C);
        dst[e] = src[(size_t)sel[b * sel_stride + j] * C + c];
    }
}

__global__ void k_compose(const int32_t *__restrict__ prev, long prev_stride,
                          const int32_t *__restrict__ loc, long loc_stride, int S,
                          int32_t *__restrict__ out, long out_stride, Cleared clear, Prefixes stages) {
    also_clear(clear);
    const int b = blockIdx.y;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < S; j += gridDim.x * blockDim.x) {
        const int32_t c = prev[b * prev_stride + loc[b * loc_stride + j]];
        out[b * out_stride + j] = c;
        put_prefixes(out + b * out_stride, j, c, stages);
    }
}

__global__ void k_copy_prefix(const int32_t *__restrict__ src, long src_stride, int S,
                              int32_t *__restrict__ out, long out_stride) {
    const int b = blockIdx.y;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < S; j += gridDim.x * blockDim.x)
        out[b * out_stride + j] = src[b * src_stride + j];
}

__global__ void k_copy_prefixes(int32_t *__restrict__ idx, long stride, Prefixes p) {
    int32_t *row = idx + blockIdx.y * stride;
    for (int l = 0; l < p.n; ++l)
        for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < p.len[l]; j += gridDim.x * blockDim.x) row[p.at[l] + j] = row[j];
}

// ---- seeded random select / fill --------------------------------------------
// Seeded bijection of [0, N): a 4-round Feistel network over 2h bits,
// 2^(2h) >= N, with a 32-bit integer mixer as round function, walked until the
// value falls below N.  Stateless: every element is computed on its own.
struct Perm {
    uint32_t n, mask, k0, k1;
    int h;
};
__host__ __device__ inline Perm make_perm(int N, uint64_t seed) {
    Perm p;
    p.n = (uint32_t)N;
    p.h = 1;
    while ((1ull << (2 * p.h)) < (unsigned long long)N) ++p.h;
    p.mask = (1u << p.h) - 1u;
    p.k0 = (uint32_t)seed;
    p.k1 = (uint32_t)(seed >> 32);
    return p;
}
__device__ __forceinline__ uint32_t perm_mix(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}
__device__ __forceinline__ uint32_t perm_at(const Perm &p, uint32_t j) {
    uint32_t x = j;
    do {
        uint32_t l = (x >> p.h) & p.mask, r = x & p.mask;
#pragma unroll
        for (uint32_t round = 0; round < 4; ++round) {
            uint32_t f = perm_mix(r ^ (((round & 1) ? p.k1 : p.k0) + 0x9E3779B9u * (round + 1))) & p.mask;
            uint32_t t = l ^ f;
            l = r;
            r = t;
        }
        x = (l << p.h) | r;
    } while (x >= p.n);
    return x;
}
constexpr uint64_t kFillSeedXor = 0xD1B54A32D192ED03ull;

// bitmap[b] |= { perm_{seed+b}(j) : j < Nc }   (bitmap cleared beforehand)
__global__ void k_perm_mark(int N, int Nc, uint64_t seed, uint32_t *__restrict__ bitmap_all, Cleared clear) {
    also_clear(clear);
    const int b = blockIdx.y;
    uint32_t *bm = bitmap_all + (size_t)b * ((N + 31) / 32);
    const Perm p = make_perm(N, seed + (uint64_t)b);
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < Nc; j += gridDim.x * blockDim.x) {
        uint32_t t = perm_at(p, (uint32_t)j);
        atomicOr(&bm[t >> 5], 1u << (t & 31));
    }
}

// The candidate set in ascending order with the candidates' coordinates, a tile of the bitmap per
// block; `start` takes the place of the last drawn candidate when it was not drawn.  A wave takes
// two words at a time, a lane per bit, so that list and coordinates are written side by side.
// 4096 points are a tile, 73 blocks for 300,000 points.  (Ten blocks of 32,768 points took 20 us, one
// block 429 us.)
constexpr int kCompactWords = 128;
__global__ __launch_bounds__(1024) void k_perm_compact(const float *__restrict__ xyz_all, int N, int tiles, int Nc,
                                                       int start, uint64_t seed,
                                                       const uint32_t *__restrict__ bitmap_all,
                                                       int32_t *__restrict__ cand_all,
                                                       float *__restrict__ cxyz_all,
                                                       int *__restrict__ spos_all) {
    __shared__ int part[16];
    __shared__ uint32_t bits_of[kCompactWords];
    __shared__ int rank_of[kCompactWords];
    const int b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int words = (N + 31) / 32;
    const uint32_t *bm = bitmap_all + (size_t)b * words;
    const float *xyz = xyz_all + (size_t)b * N * 3;
    int32_t *cand = cand_all + (size_t)b * Nc;
    float *cxyz = cxyz_all + (size_t)b * Nc * 3;
    const bool drawn = (bm[start >> 5] >> (start & 31)) & 1u;
    const int last = drawn ? -1 : (int)perm_at(make_perm(N, seed + (uint64_t)b), (uint32_t)(Nc - 1));
    auto word = [&](int wd) {
        uint32_t v = bm[wd];
        if (!drawn) {
            if (wd == last >> 5) v &= ~(1u << (last & 31));
            if (wd == start >> 5) v |= 1u << (start & 31);
        }
        return v;
    };
    int before = 0;
    const int t0 = first_tile(tiles, blockIdx.x, gridDim.x), t1 = first_tile(tiles, blockIdx.x + 1, gridDim.x);
    for (int wd = tid; wd < t0 * kCompactWords; wd += 1024) before += __popc(word(wd));
    if (t0 > 0) (void)block_prefix(before, part, tid, &before);
    for (int tile = t0; tile < t1; ++tile) {
        const int wd0 = tile * kCompactWords;
        const uint32_t own = tid < kCompactWords && wd0 + tid < words ? word(wd0 + tid) : 0u;
        int total = 0;
        const int r = before + block_prefix(__popc(own), part, tid, &total);
        before += total;
        if (tid < kCompactWords) {
            bits_of[tid] = own;
            rank_of[tid] = r;
        }
        __syncthreads();
        for (int p = wave; p < kCompactWords / 2; p += 16) {
            const int t = 2 * p + (lane >> 5);
            const uint32_t v = bits_of[t];
            if ((v >> (lane & 31)) & 1u) {
                const int at = rank_of[t] + __popc(v & ((1u << (lane & 31)) - 1u));
                const int i = (wd0 + t) * 32 + (lane & 31);
                cand[at] = i;
                cxyz[3 * (size_t)at + 0] = xyz[3 * (size_t)i + 0];
                cxyz[3 * (size_t)at + 1] = xyz[3 * (size_t)i + 1];
                cxyz[3 * (size_t)at + 2] = xyz[3 * (size_t)i + 2];
                if (i == start) spos_all[b] = at;
            }
        }
        __syncthreads();
    }
}

// The seeded fill: idx[k + r] = r-th index, in the order of a second permutation of [0, N), that
// is not among the picks (marked in the bitmap); r < R.  The first k + R places hold R such indices.  A tile of
// 1024 places per block, twice: the first launch finds the index at each place (-1: a pick) and counts the others, the
// second puts them where they belong.  What bounds the first is the longest walk of a wave's lanes until the permutation
// falls below N.  16,384 samples of 300,000 points: 22 and 23 us with all places and tiles of 4096, found in both launches.
constexpr int kPermTile = 1024;
__global__ __launch_bounds__(kPermTile) void k_fill_perm_find(int N, int places, uint64_t seed, const uint32_t *__restrict__ bitmap_all,
                                                              int32_t *__restrict__ at_all, int *__restrict__ free_all) {
    __shared__ int part[16];
    const int b = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x, j = tile * kPermTile + tid;
    const uint32_t *bm = bitmap_all + (size_t)b * ((N + 31) / 32);
    int at = -1;
    if (j < places) {
        at = (int)perm_at(make_perm(N, (seed + (uint64_t)b) ^ kFillSeedXor), (uint32_t)j);
        if ((bm[at >> 5] >> (at & 31)) & 1u) at = -1;
        at_all[(size_t)b * places + j] = at;
    }
    int total = 0;
    (void)block_prefix(at >= 0 ? 1 : 0, part, tid, &total);
    if (tid == 0) free_all[(size_t)b * gridDim.x + tile] = total;
}
__global__ __launch_bounds__(kPermTile) void k_fill_perm_put(int places, int k, int R, int32_t *__restrict__ idx_all, long idx_stride,
                                                             const int32_t *__restrict__ at_all, const int *__restrict__ free_all) {
    __shared__ int part[16];
    const int b = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x, j = tile * kPermTile + tid;
    const int *nfree = free_all + (size_t)b * gridDim.x;
    const int at = j < places ? at_all[(size_t)b * places + j] : -1;
    int before = 0;
    for (int t = tid; t < tile; t += kPermTile) before += nfree[t];
    (void)block_prefix(before, part, tid, &before);
    const int r = before + block_prefix(at >= 0 ? 1 : 0, part, tid, nullptr);
    if (at >= 0 && r < R) idx_all[b * idx_stride + k + r] = at;
}

// Reference point for the multi-workgroup kernels: `iters` plain grid barriers
// (one device-scope atomic arrive + a bounded spin on the counter per barrier).
__global__ __launch_bounds__(256) void k_barrier_probe(unsigned *counter, int iters, int *status) {
    const unsigned G = gridDim.x;
    for (int it = 1; it <= iters; ++it) {
        __syncthreads();
        if (threadIdx.x == 0) {
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            int spin = 0;
            while (__hip_atomic_load(counter, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < G * (unsigned)it) {
                if (++spin > (1 << 22)) {
                    __hip_atomic_store(status, -5, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
        }
        __syncthreads();
        if (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
    }
}

inline int wrap_point(int N, int Nc, int start) {
    // smallest j with start + floor(j*N/Nc) >= N, capped at Nc (no wrap)
    long j0 = (((long)N - start) * Nc + N - 1) / N;
    return (int)(j0 > Nc ? Nc : j0);
}

}  // namespace

// Diagnostic: sustained rate of the arithmetic of a distance update.  Every lane
// keeps 16 independent values and applies subtract, multiply, add, minimum to
// each of them `iters` times: individually rounded fp32 operations with no
// memory traffic, the mix of Eq. 1's inner loop.  One word per wave goes to
// `sink` so that the work cannot be dropped.
__global__ __launch_bounds__(1024) void k_alu_probe(int iters, float seed, float *sink) {
    constexpr int CH = 16;
    float a[CH];
    const float b = seed + (float)threadIdx.x * 1e-3f, c = 0.999f;
#pragma unroll
    for (int i = 0; i < CH; ++i) a[i] = (float)(i + (int)threadIdx.x);
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            a[i] = __fsub_rn(a[i], b);
            a[i] = __fmul_rn(a[i], c);
            a[i] = __fadd_rn(a[i], b);
            a[i] = fminf(a[i], 1e30f);
        }
    }
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) t += a[i];
    if ((threadIdx.x & 63) == 0) sink[(blockIdx.x * blockDim.x + threadIdx.x) >> 6] = t;
}

hipError_t launch_alu_probe(float *sink, int num_wg, int waves_per_wg, int iters, hipStream_t s) {
    k_alu_probe<<<dim3(num_wg), dim3(64 * waves_per_wg), 0, s>>>(iters, 1.0f, sink);
    return hipGetLastError();
}

hipError_t launch_barrier_probe(unsigned *counter, int *status, int num_wg, int iters, hipStream_t s) {
    void *params[] = {&counter, &iters, &status};
    return hipLaunchCooperativeKernel((const void *)k_barrier_probe, dim3(num_wg), dim3(256), params,
                                      0, s);
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    size_t words = bytes / 4;
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for(words)), dim3(kT), 0, s, (uint32_t *)p, words);
    return hipGetLastError();
}

hipError_t launch_gather_candidates(const float *xyz, int B, int N, int Nc, int start, float *cxyz,
                                    const Cleared &clear, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_candidates, dim3(blocks_for(Nc), B), dim3(kT), 0, s, xyz, N, Nc,
                       start, wrap_point(N, Nc, start), cxyz, clear);
    return hipGetLastError();
}

hipError_t launch_map_candidates(const int32_t *loc, long loc_stride, int B, int N, int Nc,
                                 int start, int k, int32_t *idx, long idx_stride, uint32_t *marked, const Prefixes &stages,
                                 hipStream_t s) {
    hipLaunchKernelGGL(k_map_candidates, dim3(blocks_for(k), B), dim3(kT), 0, s, loc, loc_stride, N,
                       Nc, start, wrap_point(N, Nc, start), k, idx, idx_stride, marked, stages);
    return hipGetLastError();
}

size_t bitmap_words(int B, int N) { return (size_t)B * ((N + 31) / 32); }

// Clears the bitmap, where it is not, and marks the picks in it.
static hipError_t mark_picks(int B, int N, int k, const int32_t *idx, long idx_stride, uint32_t *bitmap, bool cleared, hipStream_t s) {
    const size_t words = bitmap_words(B, N);
    if (!cleared) hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for(words)), dim3(kT), 0, s, bitmap, words);
    hipLaunchKernelGGL(k_mark_picks, dim3(blocks_for(k), B), dim3(kT), 0, s, N, k, idx, idx_stride, bitmap);
    return hipGetLastError();
}

static int tiles_of(int N, int tile_words) { return ((N + 31) / 32 + tile_words - 1) / tile_words; }
static int tile_blocks(int tiles) { return tiles < kTileBlocks ? tiles : kTileBlocks; }

bool fill_marks_itself(int N) { return tiles_of(N, 1024) == 1; }

hipError_t launch_fill(int B, int N, int k, int R, int32_t *idx, long idx_stride, uint32_t *bitmap, bool marked,
                       hipStream_t s) {
    if (R <= 0) return hipSuccess;
    if (fill_marks_itself(N)) {
        hipLaunchKernelGGL(k_fill<32>, dim3(1, B), dim3(1024), 0, s, N, 1, k, R, idx, idx_stride, bitmap);
        return hipGetLastError();
    }
    if (!marked) {
        hipError_t e = mark_picks(B, N, k, idx, idx_stride, bitmap, false, s);
        if (e != hipSuccess) return e;
    }
    const int tiles = tiles_of(N, 256);
    hipLaunchKernelGGL(k_fill<8>, dim3(tile_blocks(tiles), B), dim3(1024), 0, s, N, tiles, k, R, idx, idx_stride, bitmap);
    return hipGetLastError();
}

hipError_t launch_perm_candidates(const float *xyz, int B, int N, int Nc, int start, uint64_t seed,
                                  uint32_t *bitmap, int32_t *cand, float *cxyz, int *spos,
                                  const Cleared &clear, hipStream_t s) {
    const size_t words = bitmap_words(B, N);
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for(words)), dim3(kT), 0, s, bitmap, words);
    hipLaunchKernelGGL(k_perm_mark, dim3(blocks_for(Nc), B), dim3(kT), 0, s, N, Nc, seed, bitmap, clear);
    const int tiles = tiles_of(N, kCompactWords);
    hipLaunchKernelGGL(k_perm_compact, dim3(tile_blocks(tiles), B), dim3(1024), 0, s, xyz, N, tiles, Nc, start, seed, bitmap, cand,
                       cxyz, spos);
    return hipGetLastError();
}

size_t fill_perm_count_words(int N) { return (size_t)(N + kPermTile - 1) / kPermTile; }

hipError_t launch_fill_perm(int B, int N, int k, int R, uint64_t seed, int32_t *idx, long idx_stride,
                            uint32_t *bitmap, bool cleared, int32_t *at, int *counts, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    hipError_t e = mark_picks(B, N, k, idx, idx_stride, bitmap, cleared, s);
    if (e != hipSuccess) return e;
    const int places = k + R;
    const dim3 grid((unsigned)fill_perm_count_words(places), B);
    hipLaunchKernelGGL(k_fill_perm_find, grid, dim3(kPermTile), 0, s, N, places, seed, bitmap, at, counts);
    hipLaunchKernelGGL(k_fill_perm_put, grid, dim3(kPermTile), 0, s, places, k, R, idx, idx_stride, at, counts);
    return hipGetLastError();
}

hipError_t launch_gather_points(const float *xyz, int B, int N, const int32_t *sel, long sel_stride,
                                int S, float *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_points, dim3(blocks_for(S), B), dim3(kT), 0, s, xyz, N, sel,
                       sel_stride, S, dst);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float *rows, int B, int N, int C, const int32_t *sel,
                              long sel_stride, int S, float *out, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_rows, dim3(blocks_for((size_t)S * C), B), dim3(kT), 0, s, rows, N, C,
                       sel, sel_stride, S, out);
    return hipGetLastError();
}

hipError_t launch_compose(const int32_t *prev, long prev_stride, const int32_t *loc, long loc_stride,
                          int B, int S, int32_t *out, long out_stride, const Cleared &clear, const Prefixes &stages, hipStream_t s) {
    hipLaunchKernelGGL(k_compose, dim3(blocks_for(S), B), dim3(kT), 0, s, prev, prev_stride, loc,
                       loc_stride, S, out, out_stride, clear, stages);
    return hipGetLastError();
}

hipError_t launch_copy_prefix(const int32_t *src, long src_stride, int B, int S, int32_t *out,
                              long out_stride, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_prefix, dim3(blocks_for(S), B), dim3(kT), 0, s, src, src_stride, S,
                       out, out_stride);
    return hipGetLastError();
}

hipError_t launch_copy_prefixes(int32_t *idx, long stride, int B, const Prefixes &p, hipStream_t s) {
    if (p.n < 1 || p.n > kMaxPrefixes) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy_prefixes, dim3(blocks_for(p.len[0]), B), dim3(kT), 0, s, idx, stride, p);
    return hipGetLastError();
}

}  // namespace ffps
