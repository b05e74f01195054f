// Limits of addresses and launches, as plain host arithmetic (no HIP), so that a test can compile it by itself.
#pragma once
#include <stdint.h>

namespace ssgd {

// The steady-state kernels of the linear models gather rows through one buffer descriptor that spans the sample matrix:
// the row's place is the scalar offset, a lane's column the vector offset.  Such a load is out of range, and gives zeros,
// from vector offset >= size - scalar offset on, so a lane that must read zeros whatever the row needs a vector offset at
// or past the size itself.  (2^31 is not that for a matrix of more than 2 GiB: the lane would read the data 2 GiB further
// on.)  The last of the four words of the load does not wrap either.
constexpr uint32_t kPastMatrix = 0xFFFFFFF0u;
inline bool one_descriptor_spans(uint64_t N, uint64_t d) { return N * d * 4u <= kPastMatrix; }

// Schedule of the synchronous variants: updates (one wavefront each) of one launch.  A launch ends at 2^32 threads in one
// dimension, that is at 2^26 updates; longer segments take several launches, of far fewer updates, so that a test gets there.
constexpr int kSyncWaves = 4;
constexpr int64_t kSyncUpdatesPerLaunch = 1 << 16;
inline uint32_t sync_schedule_blocks(int64_t updates) { return (uint32_t)((updates + kSyncWaves - 1) / kSyncWaves); }

// Whether the workgroups of a cluster may take a CU each for themselves.  The clusters of several launches (contexts of one
// process run beside each other, one launch per hardware queue) can hold part of their CUs on an XCD and wait for the rest;
// with at most G - 1 each, one of them still finds its last CU as long as the others leave one free.  Two workgroups per CU
// leave twice the room.
constexpr int kXcds = 8, kHardwareQueues = 4;
inline bool whole_cus(int G, int cus) { return G == 1 || kHardwareQueues * (G - 1) < cus / kXcds; }

}  // namespace ssgd
