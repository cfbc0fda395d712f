// Host-side interface of the local-maximum kernel for clouds of one workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fps_launch.h"

namespace ffps {

struct BlockArgs {
    const float *xyz;
    long cloud_points;    // points from one cloud to the next
    const int32_t *sel;   // point i of the cloud is row sel[i] (null: i); samples are such rows, too
    long sel_stride;
    int N, M, start;
    const int *start_dev;
    int32_t *idx;
    long idx_stride;
    float *md;
    long md_stride;
    int *status;          // as for the other kernels
    bool clear;           // the kernel clears the status block itself
};
constexpr int kWaveCapacity = 256;  // largest N of one wave

// fps_wg.hip: one wave per cloud, one pick per pass; N <= kWaveCapacity
hipError_t launch_fps_wave(const BlockArgs &a, int B, hipStream_t s);
// fps_block.hip.  `clear` only with a single cloud: several write their rounds into the block.
int block_capacity();  // largest N; the smallest is 32
hipError_t launch_fps_block(const BlockArgs &a, int B, hipStream_t s);

}  // namespace ffps
