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

// Clusters of G workgroups that share the tiles of a replica's update (a team).  Every workgroup gets a CU to itself, and one
// CU per XCD stays free for the schedule.  A team on one XCD keeps to the rule above as a whole, in places of a CU (per_cu: 1
// or 2 workgroups fit).  Where that gives too few, the clusters are spread over the XCDs; then a launch takes at most a quarter
// of the places of an XCD, so that the launches of four queues fit side by side and none holds part of its places in vain.
// The size is the one with the least time per update, in cycles: the tiles of a member one after the other, and the members'
// gradient sums that everyone reads (a kilobyte per class row and member, 16 bytes per cycle).  (21 tiles of one slice, 15
// classes: 70 us per update alone, 12.8 with 8 members, 10.1 with 11.)
constexpr int kMostMembers = 32;
struct TeamShape { int members, spread; };
inline TeamShape team_shape(int64_t tiles, int G, int C, int64_t replicas, int cus, int per_cu) {
    const int64_t room = cus / kXcds, together = ((per_cu >= 2 ? 2 : 1) * room - 1) / kHardwareQueues + 1;
    const int64_t on_xcd = (replicas + kXcds - 1) / kXcds;
    const int64_t a = (room - 1) / (on_xcd * G), b = together / G;
    const int64_t local = a < b ? a : b;
    const int64_t wide = kXcds * ((together < room - 1 ? together : room - 1) / G) / replicas;
    int64_t most = local > wide ? local : wide;
    if (most > kMostMembers) most = kMostMembers;
    if (most > tiles) most = tiles;
    const int64_t tile = G == 1 ? 8000 : 12000, step = 2500;
    int64_t best = 1, least = tiles * tile;
    for (int64_t w = 2; w <= most; ++w) {
        const int64_t t = (tiles + w - 1) / w * tile + step + w * C * 64;
        if (t < least) { least = t; best = w; }
    }
    return {(int)best, best > 1 && best > local ? 1 : 0};
}

}  // namespace ssgd
