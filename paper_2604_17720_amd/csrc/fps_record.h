// The records that the units of k_fps_local publish: three chunks of 16 bytes.
//   A  value of the best point (bit 31: its workgroup has stopped) | index, steps of the bound << 23, bit 31: the
//      candidate of the round before was picked | value of the second point | check
//   B  coordinates of the best point | check
//   C  coordinates of the second point | check
// A check is the exclusive or of the other words with a constant of the chunk's kind and the round: cleared memory
// stands for no round, and a chunk two rounds old (the buffers alternate) is told from a new one.  Every chunk has all
// 32 bits of it.  So what no other point's value exceeds is a number of steps below the second value, where the index
// leaves room: of 2^14 units of a float's last place: never too low, at most 1/512 too high down to two thirds or three quarters of it.
// (As a word of its own beside a check of 8 bits it made the same rounds, within one of 85 to 214; rounded up to the
// upper half of a float 2 % more time.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ffps {

constexpr uint32_t kTagA = 0x9E3779B1u, kTagB = 0x85EBCA6Bu, kTagC = 0x27D4EB2Fu, kTagBox = 0x5F356495u;

// The last word of a chunk of `which` kind; of a whole chunk, the round.
__host__ __device__ inline uint32_t record_check(uint32_t x, uint32_t y, uint32_t z, uint32_t which, uint32_t round) {
    return x ^ y ^ z ^ which ^ round;
}

constexpr int kIndexBitsOfRecord = 23, kBoundShift = 14;
constexpr uint32_t kPickedBit = 0x80000000u, kRecordIndex = (1u << kIndexBitsOfRecord) - 1u, kBoundSteps = 255u;

// Values as bits; `others` is not above `second`.
__host__ __device__ inline uint32_t index_word(uint32_t index, uint32_t second, uint32_t others, bool picked) {
    const uint32_t steps = (second - others) >> kBoundShift;
    return index | (steps < kBoundSteps ? steps : kBoundSteps) << kIndexBitsOfRecord | (picked ? kPickedBit : 0u);
}
__host__ __device__ inline uint32_t bound_of_others(uint32_t second, uint32_t word) {
    return second - (((word >> kIndexBitsOfRecord) & kBoundSteps) << kBoundShift);
}

}  // namespace ffps
