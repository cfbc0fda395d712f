// Host-side interface of the local-maximum kernel and of the two sorts around it.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ffps {

constexpr int kLocalBinShift = 18;  // a bin of pick values: sign, exponent and five bits of the fraction
constexpr int kLocalBins = 8192;
constexpr int kLocalMaxUnits = 2048;
constexpr int kLocalWords = kLocalBins + kLocalMaxUnits;  // picks per bin, picks per unit so far

// Place of a bin's counter: neighbours (the values of one stretch of the run) lie far apart, so that
// counting does not queue up at one memory channel.
__host__ __device__ __forceinline__ uint32_t local_bin_place(uint32_t bin) { return ((bin & 63u) << 7) | ((bin >> 6) & 127u); }

// How B clouds of N points, of which M are sampled, are laid over the device.
struct LocalPlan {
    int wg_per_cloud;       // 0: the kernel does not take such clouds
    int clouds_per_launch;
    int units_per_cloud;
};
LocalPlan plan_fps_local(int B, int N, int M, int num_cu);

struct LocalBuffers {  // device memory of one call
    void *pts;          // [B][N] 16 bytes: the points in order; later the keys of the picks
    void *picks;        // [B][N] 16 bytes: the picks of each unit
    int *npicks;        // [B][units]
    char *zeroed;       // exchange areas, then counters: cleared together by the first kernel
    uint32_t *hist;     // [B][kLocalWords]
    uint32_t *cursor;   // [B][kLocalBins]
    void *runs;         // [B][kLocalBins] 8 bytes
    int *nruns;         // [B]
    float *boxes;       // [B][tiles][6]
    uint16_t *codes;    // [B][N]
    uint32_t *hist1, *hist2;  // [B][tiles][256], [B][tiles][128]
    size_t zero_bytes;
    size_t exchange_bytes_per_cloud;
};
int order_tiles(int N);
// Bytes of a call's device memory, and its parts in an area of that size (256-byte aligned).
LocalBuffers carve_local(char *base, int B, int N, const LocalPlan &p, size_t *bytes);
int local_capacity();  // largest N on any device
size_t local_workspace_bound(int B, int N);  // over all devices

// `clear_status`: the call's status block, cleared as well, or null.
hipError_t launch_order(const float *xyz, int B, int N, const LocalBuffers &l, int *clear_status, hipStream_t s);
hipError_t launch_local(const float *xyz, const LocalBuffers &l, int B, int N, int M, int start, const int *start_dev, const LocalPlan &p,
                        int *status, int spin_limit, hipStream_t s);
hipError_t launch_finish(const LocalBuffers &l, int B, int N, int M, int units, int start, const int *start_dev, int32_t *idx,
                         long idx_stride, float *md, long md_stride, int *status, hipStream_t s);

}  // namespace ffps
