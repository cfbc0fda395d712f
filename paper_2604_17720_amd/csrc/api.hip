// C-ABI layer: argument validation, workspace carving and kernel dispatch.
// Every step of the sampling path runs in the kernels of this library; the
// host side only validates, sizes and enqueues.
#include <hip/hip_runtime.h>
#include <string.h>

#include <mutex>

#include "../../include/flashfps.h"
#include "fps_block.h"
#include "fps_launch.h"
#include "fps_local.h"

static_assert(ffps::kErrGaveUp == FFPS_ERR_TIMEOUT && ffps::kErrInconsistent == FFPS_ERR_INTERNAL,
              "the kernels write these codes into the status word");

namespace {

using namespace ffps;

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// The helper kernels of FPS-Prune and of the stage chain put the cloud number
// in gridDim.y, which the hardware limits to 65535.
constexpr int kMaxBatchHelpers = 65535;

struct Workspace {  // byte offsets into the caller's workspace
    size_t status, exchange, cxyz, loc, bitmap, mind, cand, spos, local, local_bytes;
    size_t least;  // what every call needs
    size_t total;  // with the local-maximum kernel's area, which comes last
    // A workspace between the two holds for the kernels without that area.
    void limit(size_t ws_bytes) {
        if (ws_bytes < total) local_bytes = ws_bytes - local;
    }
};

// Least points x samples of k_fps_local, and its least samples; and the most points per sample of clouds that go there
// with less work, 0 where there are too many of them, by the workgroups each has (see takes_local).
constexpr long kLocalWork = 1L << 25;
constexpr int kLocalSamples = 80;
constexpr int local_points_per_sample(int share) { return share >= 64 ? 5 : share >= 17 ? 3 : 0; }

Workspace carve(int B, int N, int M) {
    Workspace w;
    size_t o = 0;
    w.status = o;   o += kAlign;
    w.exchange = o; o += align_up((size_t)kMaxGridWG * grid_exchange_bytes_per_cloud());
    w.cxyz = o;     o += align_up((size_t)B * N * 3 * sizeof(float));
    w.loc = o;      o += align_up((size_t)B * M * sizeof(int32_t));
    w.bitmap = o;   o += align_up((size_t)B * ((N + 31) / 32) * sizeof(uint32_t));
    w.mind = o;     o += align_up((size_t)B * N * sizeof(float));
    w.cand = o;     o += align_up((size_t)B * N * sizeof(int32_t));
    w.spos = o;     o += align_up((size_t)B * sizeof(int));
    // Neither clouds of one workgroup nor too few samples go to the local-maximum kernel.  What a call samples on the
    // way (candidates, stages) has no more points and no more samples: never more work, but maybe fewer points per
    // sample, so that as few points as are not one workgroup's decide.
    const bool enough = (long)N * M >= kLocalWork || (long)M * local_points_per_sample(kMaxGridWG / B) > wgm_capacity();
    const bool local = N > wgm_capacity() && N <= local_capacity() && enough && M >= kLocalSamples && B <= kMaxBatchHelpers;
    w.least = w.local = o;
    w.local_bytes = local ? align_up(local_workspace_bound(B, N)) : 0;
    w.total = o + w.local_bytes;
    return w;
}

struct Device {
    int ok;      // FFPS_OK or an error code
    int num_cu;
};

// Facts about a device that never change while the process lives (is it a
// gfx950, how many CUs), looked up once per device: the full property query is
// far dearer than a small launch.  This cache is the library's only state.
constexpr int kMaxDevices = 64;
std::mutex g_device_mutex;
bool g_device_known[kMaxDevices];
Device g_device[kMaxDevices];

// Device memory of the allocation-free entry point: the status block and the
// exchange areas of one launch, i.e. everything exact FPS needs besides its
// inputs and outputs as long as the clouds fit in registers.  Every device the
// library runs on holds its own copy of this array until the process ends.  In
// host code the name is only a handle: the array's address on a device comes
// from hipGetSymbolAddress, asked once per device with that device current.
constexpr size_t kScratchBytes = kAlign + (size_t)kMaxGridWG * kExchangeBytesPerCloud;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
char *g_scratch_ptr[kMaxDevices];  // address of `scratch` on each device, null until asked

Device query_device_uncached(int dev) {
    Device d{FFPS_ERR_LAUNCH_FAILED, 0};
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return d;
    if (strncmp(p.gcnArchName, "gfx950", 6) != 0) {
        d.ok = FFPS_ERR_UNSUPPORTED_DEVICE;
        return d;
    }
    d.ok = FFPS_OK;
    d.num_cu = p.multiProcessorCount;
    return d;
}

// Properties of the current device.
Device query_device(int *dev_out = nullptr) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return Device{FFPS_ERR_LAUNCH_FAILED, 0};
    if (dev_out) *dev_out = dev;
    if (dev < 0 || dev >= kMaxDevices) return query_device_uncached(dev);
    std::lock_guard<std::mutex> lock(g_device_mutex);
    if (!g_device_known[dev]) {
        g_device[dev] = query_device_uncached(dev);
        // a failed query is tried again by the next call
        g_device_known[dev] = g_device[dev].ok != FFPS_ERR_LAUNCH_FAILED;
    }
    return g_device[dev];
}

// Address of `scratch` on the current device (number `dev`), or null.
char *scratch_of_current_device(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_device_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = (char *)p;
    }
    return g_scratch_ptr[dev];
}

inline int hip_rc(hipError_t e) { return e == hipSuccess ? FFPS_OK : FFPS_ERR_LAUNCH_FAILED; }

int check_common(const void *xyz, int B, int N, int M, int start, const void *idx) {
    if (!xyz || !idx) return FFPS_ERR_INVALID_ARG;
    if (B < 1 || N < 1 || M < 1 || M > N) return FFPS_ERR_INVALID_ARG;
    if (start < 0 || start >= N) return FFPS_ERR_INVALID_ARG;
    if ((long)B * N > (1L << 31) - 1) return FFPS_ERR_INVALID_ARG;
    return FFPS_OK;
}

// `variant` carries the kernel choice in its low byte and the optional
// picks-per-round cap above it (FFPS_VARIANT_WITH_PICKS).
inline int variant_kind(int variant) { return variant & 0xff; }
inline int variant_picks(int variant) {
    int p = (variant >> 8) & 0xff;
    return p == 0 ? kMaxPicksPerRound : p;
}
int check_variant(int variant) {
    if (variant < 0 || (variant >> 17) != 0) return FFPS_ERR_INVALID_ARG;
    int v = variant_kind(variant);
    return (v >= FFPS_VARIANT_AUTO && v <= FFPS_VARIANT_STREAM) ? FFPS_OK : FFPS_ERR_INVALID_ARG;
}

// The status word is cleared once per call; the exchange area before every
// grid launch (its tags restart at 1 in each launch).
int clear_status(char *ws, const Workspace &w, hipStream_t s) {
    return hip_rc(launch_fill_zero(ws + w.status, kAlign, s));
}
int clear_exchange(char *ws, const Workspace &w, int clouds, hipStream_t s) {
    return hip_rc(launch_fill_zero(ws + w.exchange, (size_t)clouds * grid_exchange_bytes_per_cloud(), s));
}

// Kernel variant that will run for clouds of N points, or a negative error.
int resolve_variant(int B, int N, int variant, const Device &dev) {
    int v = variant_kind(variant);
    if (v == FFPS_VARIANT_AUTO) {
        // Clouds that fit the multi-pick single-workgroup kernel run there, larger
        // ones on clusters of workgroups, those beyond the registers of the
        // device are streamed.
        if (N <= wgm_capacity())
            v = FFPS_VARIANT_WG;
        else if (N <= grid_capacity(dev.num_cu))
            v = FFPS_VARIANT_GRID;
        else
            v = FFPS_VARIANT_STREAM;
    }
    if (v == FFPS_VARIANT_WG && N > wg_capacity()) return FFPS_ERR_UNSUPPORTED_SIZE;
    if (v == FFPS_VARIANT_GRID && N > grid_capacity(dev.num_cu)) return FFPS_ERR_UNSUPPORTED_SIZE;
    if (v == FFPS_VARIANT_STREAM && N > stream_capacity()) return FFPS_ERR_UNSUPPORTED_SIZE;
    return v;
}

// Which kernel AUTO takes (clouds of at most 256 points: one wave, one pick per pass).
//
// k_fps_block against k_fps_wgm, one cloud, uniform / planes / a stretch of a LiDAR frame: 1024 points to 512 71, 72, 106
// against 121, 120, 153 us; 4096 to 1024 187, 232, 364 against 336, 364, 407; 4608 to 2304 333, 368, 760 against 639, 645,
// 705. Beyond 4608 points it needs 12 or 16 points per lane and a cloud is faster on many CUs unless its samples are few
// (5500 to 1375 283, 308, 516 against 236, 244, 232 of k_fps_local; to 343 133, 139, 183 against 161, 199, 249 of k_fps_grid,
// but 376 against 188 for a cube with tails), or unless there are many clouds, which then wait for one another: 8192 points
// to 4096, 64 clouds 761, 882, 1704 against 1332, 1327, 1474 us of k_fps_grid, 80 clouds 756, 885, 1701 against 1711, 1767,
// 1913.
constexpr int kOneWaveMax = kWaveCapacity;
constexpr int kBlockMax = 4608;
constexpr int kBlockManyClouds = 80;
bool takes_block(int B, int N) {
    return N > kOneWaveMax && (N <= kBlockMax || (N <= block_capacity() && B >= kBlockManyClouds));
}
// k_fps_local has a dearer start than k_fps_grid (two sorts, 45 us in all at 45,678 points, 60 at 200,000) and more rounds as
// long as the samples are few; its rounds do not grow with the points.  In us, k_fps_grid first, uniform / a room / planes /
// a LiDAR stretch: at points x samples = 2^25 8190 points to 4095 577:286, 594:267, 638:294, 667:262; 12,000 to 3000 462:277,
// 492:266, 521:295, 583:274; 24,000 to 1500 379:277, 396:266, 415:311, 501:280.
//
// Few clouds have many and small units (plan_fps_local) and go with less.  Ordinary clouds gain from a tenth of the points as
// samples on: 6000 to 1000 274:234, 268:208, 281:244, 360:214, to 1200 297:235, 302:220, 308:254, 378:217, to 3000 498:273,
// 493:244, 526:304, 581:246; eight clouds of 8000 to 2666 455:320, 502:320, 511:348, 631:333.  Clouds whose points share
// distances gain most, for k_fps_grid makes few picks a round there: a lattice of 5000 to 1250 4550:268, points on a raster
// (planes, 1/32) 493:258, to 2500 3918:286.  What the line waits for are clouds of tails, whose far points are most of the
// samples and lie in few units.  A cube with five points in a hundred at up to 100 times the extent / Cauchy distributed:
// 6000 to 1000 342:335, 298:348, to 1200 366:346, 336:373, to 1500 394:348, 376:392 (but 7000 to 1750 432:523, 409:410); 9000
// to 1500 401:480, 386:433, to 2250 485:499, 474:474; 16,000 to 1333 396:496, 374:487; eight clouds of 5000 to 1250 382:455,
// 346:412, to 1666 436:528, 416:443.  From a fifth of up to four clouds' points, a third of up to fifteen's, and beyond 8192
// points with 9 x 2^21, they lose a tenth at most times and a fifth at worst, where ordinary clouds gain a quarter to one
// half and more samples turn the order for all.
//
// The sorts grow with the points, and uniform clouds gain least: 100,000 to 340 312:332 (a room 386:273, LiDAR 525:287), to
// 700 386:364; 200,000 to 170 300:303 (383:251), to 340 361:346; a million to 100 356:338 (480:280).  Normally distributed
// ones lose up to a third (200,000 to 340 293:380, 100,000 to 700 343:365), tails more (224:384; with more samples the order
// turns: 300,000 to 16,384 normally distributed 2019:852, Cauchy 2015:2077, the cube with tails 2181:2549).  So the line
// beyond 65,536 points is 2^26.  Beyond the registers' 3.1 million points k_fps_grid gives way to k_fps_stream, which is the
// slower one with fewer samples already (64 of four million uniform points 685:504, of a room 995:440): 2^25 and 80 samples
// are a cautious line there.
//
// Many clouds leave each few workgroups, and what is gained shrinks, for LiDAR stretches first (uniform / a room / planes /
// LiDAR): 16 clouds (16 workgroups each) of 16,384 to 4096 804:526, 857:492, 857:556, 962:807; of 30,000 to 7500 1534:741,
// 1641:714, 1641:849, 1841:1665; 20 of 30,000 to 7500 1785:967, 1855:931, 1823:1115, 2032:2182, with tails 1898:2401, to
// 15,000 3248:1511, 3310:1411, 3308:1696, 3583:3004, tails 3409:3318; 32 of 9000 to 4500 928:691, 984:670, 1016:810,
// 1081:1114, tails 1002:1429; 64 of 30,000 to 7500 4600:2456, 4788:2430, 4772:2922, 5244:5638, tails 4864:6587.  From 12 x
// 2^25 on LiDAR stretches gain and tails break even; ordinary clouds would from a quarter of that.
//
// The sorts put the cloud number in gridDim.y: more clouds than that stay with k_fps_grid, which takes
// them in batches.
constexpr long kLocalWorkLarge = 1L << 26;  // beyond 65,536 points
constexpr long kLocalWorkMany = 3L << 27;   // many clouds
constexpr long kLocalWorkMedium = 9L << 21; // 8193 points and more, few per sample
bool takes_local(int B, int N, int M, int v, int num_cu) {
    const long work = (long)N * M;
    if (B > kMaxBatchHelpers || M < kLocalSamples) return false;
    if (v == FFPS_VARIANT_STREAM) return work >= kLocalWork;
    const int share = (num_cu < kMaxGridWG ? num_cu : kMaxGridWG) / B;  // workgroups of a cloud
    if (B > 1 && (share < 16 || (share == 16 && N > 1024 * share))) return work >= kLocalWorkMany;
    if (M < 96 + N / 65536) return false;
    if (N > 65536) return work >= kLocalWorkLarge;
    return work >= kLocalWork || ((long)M * local_points_per_sample(share) >= N && (N <= 8192 || work >= kLocalWorkMedium));
}

// Clouds that are rows of a larger array: point i of cloud b is row idx[b][i] of [B][points]
// points.  The kernels of one workgroup read through it and write rows, which spares a stage
// of a chain two launches (about 9 us).
struct Rows {
    const int32_t *idx;
    long stride;
    int points;
};
// AUTO without a cap on the picks of a round, which the kernels that pick local maxima do not know.
bool any_rounds(int M, int variant) { return variant_kind(variant) == FFPS_VARIANT_AUTO && ((variant >> 8) & 0xff) == 0 && M > 1; }
bool takes_wave(int N, int v) { return v == FFPS_VARIANT_WG && N <= kWaveCapacity; }
bool takes_rows(int B, int N, int M, int variant, const Device &dev) {
    return takes_wave(N, resolve_variant(B, N, variant, dev)) || (any_rounds(M, variant) && takes_block(B, N));
}

// The kernel that samples B clouds of N points to M, FFPS_KERNEL_*, or a negative error.  `local_bytes`:
// what the workspace has for k_fps_local; where that is too little the kernels without it run.
int kernel_for(int B, int N, int M, int variant, const Device &dev, size_t local_bytes) {
    const int v = resolve_variant(B, N, variant, dev);
    if (v < 0) return v;
    if (takes_wave(N, v)) return FFPS_KERNEL_WAVE;
    if (any_rounds(M, variant) && takes_block(B, N)) return FFPS_KERNEL_BLOCK;
    if (v == FFPS_VARIANT_WG) return FFPS_KERNEL_WG;
    if (any_rounds(M, variant) && takes_local(B, N, M, v, dev.num_cu)) {
        const LocalPlan plan = plan_fps_local(B, N, M, dev.num_cu);
        size_t bytes = 0;
        if (plan.wg_per_cloud > 0) {
            carve_local(nullptr, B, N, plan, &bytes);
            if (bytes <= local_bytes) return FFPS_KERNEL_LOCAL;
        }
    }
    return v == FFPS_VARIANT_GRID ? FFPS_KERNEL_GRID : FFPS_KERNEL_STREAM;
}

// Exact FPS of B clouds [N] into idx (row stride idx_stride).  Arguments are
// already validated.  `clear`: the status block is cleared first, by the kernel itself where
// that is safe.  `rows` only where takes_rows says so.
int run_exact(const float *xyz, int B, int N, int M, int start, const int *start_dev, int variant,
              int32_t *idx, long idx_stride, float *md, long md_stride, char *ws,
              const Workspace &w, const Device &dev, hipStream_t s, bool clear, const Rows *rows = nullptr) {
    const int kernel = kernel_for(B, N, M, variant, dev, w.local_bytes);
    if (kernel < 0) return kernel;
    if (kernel == FFPS_KERNEL_WAVE || kernel == FFPS_KERNEL_BLOCK) {
        const bool own = kernel == FFPS_KERNEL_WAVE || B == 1;
        int rc = clear && !own ? clear_status(ws, w, s) : FFPS_OK;
        if (rc) return rc;
        const BlockArgs a = {xyz, rows ? rows->points : N, rows ? rows->idx : nullptr, rows ? rows->stride : 0, N, M, start, start_dev,
                             idx, idx_stride, md, md_stride, (int *)(ws + w.status), clear && own};
        return hip_rc(kernel == FFPS_KERNEL_WAVE ? launch_fps_wave(a, B, s) : launch_fps_block(a, B, s));
    }
    if (clear && kernel != FFPS_KERNEL_LOCAL) {
        int rc = clear_status(ws, w, s);
        if (rc) return rc;
    }
    if (kernel == FFPS_KERNEL_WG)
        return hip_rc(launch_fps_wg(xyz, B, N, M, start, start_dev, idx, idx_stride, md, md_stride,
                                    variant_picks(variant), (int *)(ws + w.status), s));
    if (kernel == FFPS_KERNEL_LOCAL) {
        const LocalPlan plan = plan_fps_local(B, N, M, dev.num_cu);
        const LocalBuffers l = carve_local(ws + w.local, B, N, plan, nullptr);
        int *status = (int *)(ws + w.status);
        int rc = hip_rc(launch_order(xyz, B, N, l, clear ? status : nullptr, s));
        if (rc == FFPS_OK)
            rc = hip_rc(launch_local(xyz, l, B, N, M, start, start_dev, plan, status,
                                     (variant & FFPS_VARIANT_TEST_NO_WAIT) ? 0 : -1, s));
        if (rc == FFPS_OK)
            rc = hip_rc(launch_finish(l, B, N, M, plan.units_per_cloud, start, start_dev, idx, idx_stride, md,
                                      md_stride, status, s));
        return rc;
    }
    if (kernel == FFPS_KERNEL_GRID) {
        const GridPlan plan = plan_fps_grid(B, N, dev.num_cu);
        for (int b = 0; b < B; b += plan.clouds_per_launch) {
            const int clouds = B - b < plan.clouds_per_launch ? B - b : plan.clouds_per_launch;
            int rc = clear_exchange(ws, w, clouds, s);
            if (rc) return rc;
            hipError_t e = launch_fps_grid(xyz + (size_t)b * N * 3, clouds, N, M, start,
                                           start_dev ? start_dev + b : nullptr,
                                           idx + b * idx_stride, idx_stride,
                                           md ? md + b * md_stride : nullptr, md_stride,
                                           ws + w.exchange, (int *)(ws + w.status),
                                           plan.wg_per_cloud, variant_picks(variant),
                                           (variant & FFPS_VARIANT_TEST_NO_WAIT) ? 0 : -1, s);
            if (e != hipSuccess) return FFPS_ERR_LAUNCH_FAILED;
        }
        return FFPS_OK;
    }
    for (int b = 0; b < B; ++b) {
        int rc = clear_exchange(ws, w, 1, s);
        if (rc) return rc;
        hipError_t e = launch_fps_stream(xyz + (size_t)b * N * 3, (float *)(ws + w.mind) + (size_t)b * N,
                                         N, M, start, start_dev ? start_dev + b : nullptr,
                                         idx + b * idx_stride,
                                         md ? md + b * md_stride : nullptr, ws + w.exchange,
                                         (int *)(ws + w.status), dev.num_cu,
                                         variant_picks(variant), s);
        if (e != hipSuccess) return FFPS_ERR_LAUNCH_FAILED;
    }
    return FFPS_OK;
}

// `stages`: prefixes of the result that are wanted as well; n is 0 afterwards where they are written already.
int run_prune(const float *xyz, int B, int N, int M, int start, int keep_num, int keep_den,
              unsigned flags, uint64_t seed, int variant, int32_t *idx, long idx_stride, char *ws,
              const Workspace &w, const Device &dev, hipStream_t s, Prefixes *stages = nullptr) {
    int Nc, k, R;
    int rc = ffps_prune_sizes(N, M, keep_num, keep_den, flags, &Nc, &k, &R);
    if (rc) return rc;
    const bool perm = (flags & FFPS_FLAG_PERM) != 0;
    uint32_t *bitmap = (uint32_t *)(ws + w.bitmap);
    int *status = (int *)(ws + w.status);
    const size_t words = R > 0 ? bitmap_words(B, N) : 0;
    const Prefixes none = {};
    const bool along = stages && stages->n > 0 && Nc < N && stages->len[0] <= k;  // no stage reaches into the fill
    const Prefixes &put = along ? *stages : none;
    bool ready = false;  // the bitmap is as the fill wants it: picks marked, or cleared before drawn ones
    if (Nc < N) {
        float *cxyz = (float *)(ws + w.cxyz);
        int32_t *loc = (int32_t *)(ws + w.loc);
        ready = perm || !fill_marks_itself(N);
        if (perm) {
            int32_t *cand = (int32_t *)(ws + w.cand);
            int *spos = (int *)(ws + w.spos);
            rc = hip_rc(launch_perm_candidates(xyz, B, N, Nc, start, seed, bitmap, cand, cxyz, spos, Cleared{status, nullptr, 0}, s));
            if (rc) return rc;
            rc = run_exact(cxyz, B, Nc, k, 0, spos, variant, loc, k, nullptr, 0, ws, w, dev, s, false);
            if (rc) return rc;
            rc = hip_rc(launch_compose(cand, Nc, loc, k, B, k, idx, idx_stride, Cleared{nullptr, bitmap, words}, put, s));
        } else {
            rc = hip_rc(launch_gather_candidates(xyz, B, N, Nc, start, cxyz, Cleared{status, bitmap, ready ? words : 0}, s));
            if (rc) return rc;
            long j0 = (((long)N - start) * Nc + N - 1) / N;  // where the strided list wraps
            if (j0 > Nc) j0 = Nc;
            int spos = (int)((Nc - j0) % Nc);  // position of start_idx in the sorted list
            rc = run_exact(cxyz, B, Nc, k, spos, nullptr, variant, loc, k, nullptr, 0, ws, w, dev, s, false);
            if (rc) return rc;
            rc = hip_rc(launch_map_candidates(loc, k, B, N, Nc, start, k, idx, idx_stride, ready && words ? bitmap : nullptr, put, s));
        }
        if (rc) return rc;
        if (along) stages->n = 0;
    } else {
        rc = run_exact(xyz, B, N, k, start, nullptr, variant, idx, idx_stride, nullptr, 0, ws, w, dev, s, true);
        if (rc) return rc;
    }
    // the list of candidates is done with, and no kernel needs its distances any more
    if (perm)
        return hip_rc(launch_fill_perm(B, N, k, R, seed, idx, idx_stride, bitmap, ready, (int32_t *)(ws + w.mind), (int *)(ws + w.cand), s));
    return hip_rc(launch_fill(B, N, k, R, idx, idx_stride, bitmap, ready, s));
}

}  // namespace

extern "C" {

int ffps_version(void) { return 100; }

const char *ffps_strerror(int code) {
    switch (code) {
        case FFPS_OK: return "success";
        case FFPS_ERR_INVALID_ARG: return "invalid argument";
        case FFPS_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case FFPS_ERR_UNSUPPORTED_DEVICE: return "device is not gfx950";
        case FFPS_ERR_LAUNCH_FAILED: return "HIP call failed";
        case FFPS_ERR_TIMEOUT: return "a workgroup stopped waiting for another";
        case FFPS_ERR_UNSUPPORTED_SIZE: return "kernel variant cannot hold this cloud size";
        case FFPS_ERR_INTERNAL: return "a kernel found its own intermediate results inconsistent";
        default: return "unknown error code";
    }
}

int ffps_prune_sizes(int N, int M, int keep_num, int keep_den, unsigned flags, int *Nc, int *k,
                     int *R) {
    if (!Nc || !k || !R) return FFPS_ERR_INVALID_ARG;
    if (N < 1 || M < 1 || M > N) return FFPS_ERR_INVALID_ARG;
    if (keep_num < 1 || keep_den < 1 || keep_num > keep_den) return FFPS_ERR_INVALID_ARG;
    if (flags & ~(FFPS_FLAG_CP | FFPS_FLAG_IP | FFPS_FLAG_PERM)) return FFPS_ERR_INVALID_ARG;
    long nc = (flags & FFPS_FLAG_CP) ? ((long)N * keep_num + keep_den - 1) / keep_den : N;
    long kk = (flags & FFPS_FLAG_IP) ? ((long)M * keep_num + keep_den - 1) / keep_den : M;
    if (kk < 1 || kk > nc) return FFPS_ERR_INVALID_ARG;
    *Nc = (int)nc;
    *k = (int)kk;
    *R = M - (int)kk;
    return FFPS_OK;
}

int ffps_workspace_bytes(int B, int N, int M, size_t *bytes) {
    if (!bytes || B < 1 || N < 1 || M < 1 || M > N) return FFPS_ERR_INVALID_ARG;
    if ((long)B * N > (1L << 31) - 1) return FFPS_ERR_INVALID_ARG;
    *bytes = carve(B, N, M).total;
    return FFPS_OK;
}

int ffps_exact(const float *d_xyz, int B, int N, int M, int start_idx, int variant, int32_t *d_idx,
               float *d_maxdist, void *d_ws, size_t ws_bytes, void *stream) {
    int rc = d_ws ? check_common(d_xyz, B, N, M, start_idx, d_idx) : FFPS_ERR_INVALID_ARG;
    if (rc) return rc;
    if ((rc = check_variant(variant))) return rc;
    Workspace w = carve(B, N, M);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    w.limit(ws_bytes);
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    if ((rc = resolve_variant(B, N, variant, dev)) < 0) return rc;
    hipStream_t s = (hipStream_t)stream;
    return run_exact(d_xyz, B, N, M, start_idx, nullptr, variant, d_idx, M, d_maxdist, M,
                     (char *)d_ws, w, dev, s, true);
}

int ffps_exact_noalloc(const float *d_xyz, int B, int N, int M, int start_idx, int variant,
                       int32_t *d_idx, float *d_maxdist, int32_t *d_status, void *stream) {
    int dev_no = 0;
    int rc = check_common(d_xyz, B, N, M, start_idx, d_idx);
    if (rc) return rc;
    if ((rc = check_variant(variant))) return rc;
    Device dev = query_device(&dev_no);
    if (dev.ok) return dev.ok;
    if ((rc = resolve_variant(B, N, variant, dev)) < 0) return rc;
    // the streaming kernel needs N running distances per cloud: beyond this array
    if (rc == FFPS_VARIANT_STREAM) return FFPS_ERR_UNSUPPORTED_SIZE;
    char *ws = scratch_of_current_device(dev_no);
    if (!ws) return FFPS_ERR_LAUNCH_FAILED;
    Workspace w;
    const size_t none = ~(size_t)0;
    // the local-maximum kernel takes the exchange areas' place where its own area fits there
    w.status = 0; w.exchange = kAlign; w.least = w.total = kScratchBytes;
    w.local = kAlign; w.local_bytes = kScratchBytes - kAlign;
    w.cxyz = w.loc = w.bitmap = w.mind = w.cand = w.spos = none;  // not part of this path
    hipStream_t s = (hipStream_t)stream;
    rc = run_exact(d_xyz, B, N, M, start_idx, nullptr, variant, d_idx, M, d_maxdist, M, ws, w, dev, s, true);
    if (rc) return rc;
    if (d_status)
        rc = hip_rc(launch_copy_prefix((const int32_t *)(ws + w.status), 2, 1, 2, d_status, 2, s));
    return rc;
}

int ffps_prune(const float *d_xyz, int B, int N, int M, int start_idx, int keep_num, int keep_den,
               unsigned flags, uint64_t seed, int variant, int32_t *d_idx, int *k_out_host,
               void *d_ws, size_t ws_bytes, void *stream) {
    int rc = d_ws ? check_common(d_xyz, B, N, M, start_idx, d_idx) : FFPS_ERR_INVALID_ARG;
    if (rc) return rc;
    if (B > kMaxBatchHelpers) return FFPS_ERR_INVALID_ARG;
    if ((rc = check_variant(variant))) return rc;
    int Nc, k, R;
    if ((rc = ffps_prune_sizes(N, M, keep_num, keep_den, flags, &Nc, &k, &R))) return rc;
    Workspace w = carve(B, N, M);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    w.limit(ws_bytes);
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    if ((rc = resolve_variant(B, Nc, variant, dev)) < 0) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (k_out_host) *k_out_host = k;
    return run_prune(d_xyz, B, N, M, start_idx, keep_num, keep_den, flags, seed, variant, d_idx, M,
                     (char *)d_ws, w, dev, s);
}

int ffps_cached_stages(const float *d_xyz, int B, int N, int L, const int *M_stages, int start_idx,
                       int keep_num, int keep_den, unsigned flags, uint64_t seed, int mode,
                       int variant, int32_t *d_idx, void *d_ws, size_t ws_bytes, void *stream) {
    if (!M_stages || L < 1) return FFPS_ERR_INVALID_ARG;
    int rc = d_ws ? check_common(d_xyz, B, N, M_stages[0], start_idx, d_idx) : FFPS_ERR_INVALID_ARG;
    if (rc) return rc;
    if (B > kMaxBatchHelpers) return FFPS_ERR_INVALID_ARG;
    if ((rc = check_variant(variant))) return rc;
    if (mode != FFPS_MODE_CACHED && mode != FFPS_MODE_CHAIN) return FFPS_ERR_INVALID_ARG;
    long S = M_stages[0];
    for (int l = 1; l < L; ++l) {
        if (M_stages[l] < 1 || M_stages[l] > M_stages[l - 1]) return FFPS_ERR_INVALID_ARG;
        S += M_stages[l];
    }
    int Nc, k, R;
    if ((rc = ffps_prune_sizes(N, M_stages[0], keep_num, keep_den, flags, &Nc, &k, &R))) return rc;
    Workspace w = carve(B, N, M_stages[0]);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    w.limit(ws_bytes);
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    if ((rc = resolve_variant(B, Nc, variant, dev)) < 0) return rc;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)d_ws;

    long off = M_stages[0];
    int next = 1;  // first stage that is not among the prefixes
    auto some_stages = [&]() {
        Prefixes p = {};
        for (; p.n < kMaxPrefixes && next < L; ++p.n, ++next) {
            p.at[p.n] = off;
            p.len[p.n] = M_stages[next];
            off += M_stages[next];
        }
        return p;
    };
    Prefixes stages = {};
    if (mode == FFPS_MODE_CACHED) stages = some_stages();
    rc = run_prune(d_xyz, B, N, M_stages[0], start_idx, keep_num, keep_den, flags, seed, variant,
                   d_idx, S, ws, w, dev, s, &stages);
    if (rc) return rc;
    if (mode == FFPS_MODE_CACHED) {
        while (stages.n > 0 || next < L) {
            if (stages.n > 0 && (rc = hip_rc(launch_copy_prefixes(d_idx, S, B, stages, s)))) return rc;
            stages = some_stages();
        }
        return FFPS_OK;
    }
    const int32_t *prev = d_idx;
    for (int l = 1; l < L; ++l) {
        int32_t *cur = d_idx + off;
        const int n = M_stages[l - 1], m = M_stages[l];
        if (takes_rows(B, n, m, variant, dev)) {
            const Rows rows = {prev, S, N};
            rc = run_exact(d_xyz, B, n, m, 0, nullptr, variant, cur, S, nullptr, 0, ws, w, dev, s, false, &rows);
        } else {
            float *pxyz = (float *)(ws + w.cxyz);
            int32_t *loc = (int32_t *)(ws + w.loc);
            rc = hip_rc(launch_gather_points(d_xyz, B, N, prev, S, n, pxyz, s));
            if (rc) return rc;
            rc = run_exact(pxyz, B, n, m, 0, nullptr, variant, loc, m, nullptr, 0, ws, w, dev, s, false);
            if (rc) return rc;
            rc = hip_rc(launch_compose(prev, S, loc, m, B, m, cur, S, kClearNothing, Prefixes{}, s));
        }
        if (rc) return rc;
        prev = cur;
        off += m;
    }
    return FFPS_OK;
}

int ffps_describe_plan(int B, int N, int variant, int num_cu, int *kernel, int *wg_per_cloud,
                       int *units_per_cloud, int *clouds_per_launch) {
    if (B < 1 || N < 1 || num_cu < 1 || check_variant(variant)) return FFPS_ERR_INVALID_ARG;
    Device dev{FFPS_OK, num_cu};
    const int v = resolve_variant(B, N, variant, dev);
    if (v < 0) return v;
    int wg = 1, units = 0, clouds = B;
    if (v == FFPS_VARIANT_WG) {
        units = wg_units(N);
    } else if (v == FFPS_VARIANT_GRID) {
        const GridPlan plan = plan_fps_grid(B, N, num_cu);
        wg = plan.wg_per_cloud;
        units = plan.units_per_cloud;
        clouds = plan.clouds_per_launch;
    } else {
        wg = stream_workgroups(N, num_cu);
        units = wg;
        clouds = 1;
    }
    if (kernel) *kernel = v;
    if (wg_per_cloud) *wg_per_cloud = wg;
    if (units_per_cloud) *units_per_cloud = units;
    if (clouds_per_launch) *clouds_per_launch = clouds;
    return FFPS_OK;
}

int ffps_describe_kernel(int B, int N, int M, int variant, int num_cu, size_t ws_bytes, int *kernel) {
    if (!kernel || B < 1 || N < 1 || M < 1 || M > N || num_cu < 1 || check_variant(variant)) return FFPS_ERR_INVALID_ARG;
    if ((long)B * N > (1L << 31) - 1) return FFPS_ERR_INVALID_ARG;
    Workspace w = carve(B, N, M);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    w.limit(ws_bytes);
    const int k = kernel_for(B, N, M, variant, Device{FFPS_OK, num_cu}, w.local_bytes);
    if (k < 0) return k;
    *kernel = k;
    return FFPS_OK;
}

int ffps_last_status(const void *d_ws, void *stream) {
    if (!d_ws) return FFPS_ERR_INVALID_ARG;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return FFPS_ERR_LAUNCH_FAILED;
    int st = 0;
    if (hipMemcpy(&st, d_ws, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
        return FFPS_ERR_LAUNCH_FAILED;
    return st;
}

int ffps_gather_rows(const float *d_rows, int B, int N, int C, const int32_t *d_idx, long idx_stride,
                     int S, float *d_out, void *stream) {
    if (!d_rows || !d_idx || !d_out) return FFPS_ERR_INVALID_ARG;
    if (B < 1 || B > kMaxBatchHelpers || N < 1 || C < 1 || S < 1 || idx_stride < S) return FFPS_ERR_INVALID_ARG;
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    return hip_rc(launch_gather_rows(d_rows, B, N, C, d_idx, idx_stride, S, d_out, (hipStream_t)stream));
}

int ffps_barrier_probe(int iters, void *d_ws, size_t ws_bytes, void *stream, float *us_per_barrier) {
    if (!d_ws || !us_per_barrier || iters < 1 || iters > (1 << 20)) return FFPS_ERR_INVALID_ARG;
    Workspace w = carve(1, 1, 1);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)d_ws;
    int rc = clear_status(ws, w, s);
    if (rc) return rc;
    if ((rc = clear_exchange(ws, w, 1, s))) return rc;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return FFPS_ERR_LAUNCH_FAILED;
    int G = dev.num_cu < kMaxGridWG ? dev.num_cu : kMaxGridWG;
    hipError_t e = hipEventRecord(e0, s);
    if (e == hipSuccess)
        e = launch_barrier_probe((unsigned *)(ws + w.exchange), (int *)(ws + w.status), G, iters, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    float ms = 0.f;
    if (e != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        rc = FFPS_ERR_LAUNCH_FAILED;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    *us_per_barrier = ms * 1000.f / (float)iters;
    int st = 0;
    if (hipMemcpy(&st, ws + w.status, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
        return FFPS_ERR_LAUNCH_FAILED;
    return st;
}

int ffps_alu_probe(int waves_per_cu, int iters, void *d_ws, size_t ws_bytes, void *stream,
                   double *ops_per_s) {
    if (!d_ws || !ops_per_s || iters < 1 || iters > (1 << 20) || waves_per_cu < 1 || waves_per_cu > 32)
        return FFPS_ERR_INVALID_ARG;
    Workspace w = carve(1, 1, 1);
    if (ws_bytes < w.least) return FFPS_ERR_WORKSPACE_TOO_SMALL;
    Device dev = query_device();
    if (dev.ok) return dev.ok;
    hipStream_t s = (hipStream_t)stream;
    // up to 16 waves in a workgroup; more waves per CU as two workgroups per CU
    const int per_wg = waves_per_cu > 16 ? (waves_per_cu + 1) / 2 : waves_per_cu;
    const int num_wg = dev.num_cu * (waves_per_cu > 16 ? 2 : 1);
    if ((size_t)num_wg * per_wg * sizeof(float) > kExchangeBytesPerCloud) return FFPS_ERR_INVALID_ARG;
    float *sink = (float *)((char *)d_ws + w.exchange);
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return FFPS_ERR_LAUNCH_FAILED;
    int rc = FFPS_OK;
    hipError_t e = launch_alu_probe(sink, num_wg, per_wg, 16, s);  // warm-up
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    if (e == hipSuccess) e = launch_alu_probe(sink, num_wg, per_wg, iters, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    float ms = 0.f;
    if (e != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        rc = FFPS_ERR_LAUNCH_FAILED;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    // 16 values x 4 operations per lane and iteration
    *ops_per_s = (double)num_wg * per_wg * 64.0 * 16.0 * 4.0 * (double)iters / ((double)ms * 1e-3);
    return FFPS_OK;
}

int ffps_last_rounds(const void *d_ws, void *stream) {
    if (!d_ws) return FFPS_ERR_INVALID_ARG;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return FFPS_ERR_LAUNCH_FAILED;
    int st[2] = {0, 0};
    if (hipMemcpy(st, d_ws, sizeof(st), hipMemcpyDeviceToHost) != hipSuccess)
        return FFPS_ERR_LAUNCH_FAILED;
    return st[0] < 0 ? st[0] : st[1];
}

}  // extern "C"
