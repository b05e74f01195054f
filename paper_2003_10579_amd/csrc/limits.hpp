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
// Where workgroups wait for others on another XCD: a launch can hold all of its places on one XCD in vain.
inline bool whole_cus_spread(int on_xcd, int cus) { return kHardwareQueues * on_xcd <= cus / kXcds; }

// Clusters of G workgroups that share the tiles of a replica's update (a team).  Every workgroup gets a CU to itself, and one
// CU per XCD stays free for the schedule.  A team on one XCD keeps to the rule above as a whole, in places of a CU (per_cu: 1
// or 2 workgroups fit).  Where that gives too few, the clusters are spread over the XCDs; then a launch, which can hold all of its
// places on an XCD and wait for another, takes at most a quarter of the places of an XCD, so that the launches of four queues fit
// side by side.
// The size is the one with the least time per update, in cycles: the tiles of a member one after the other, and the members'
// gradient sums that everyone reads (a kilobyte per class row and member, 16 bytes per cycle).  (21 tiles of one slice, 15
// classes, one replica: 64 us per update alone, 9.3 with 11 members.)  A tile of least squares takes about half of what is counted
// here, which still leaves every team that the rule makes the better choice: over 144 shapes of both models and three variants, two to
// twelve tiles, runs are 1.10 (softmax, K-batch-async, 5 mini-batches of 16, d = 64: 7.2 -> 6.5 us per update) to 5.9 times
// as fast with a team; least squares, two tiles, d = 64, 3.9 -> 2.6.  What loses is a call of a single update, of which a team's meeting and
// the buffers armed for it are a larger part: up to 5 of 39 us (K-batch-async, 5 of 16, d = 200, 40 replicas), while with three
// slices it gains (softmax, K-sync, 2 of 64, d = 516, 2 replicas 40 -> 36 us); both go the same way, so that results do not depend on how a run is cut into calls.
constexpr int kMostMembers = 32;
struct TeamShape { int members, spread; };
inline TeamShape team_shape(int64_t tiles, int G, int C, int64_t replicas, int cus, int per_cu) {
    const int64_t room = cus / kXcds, places = (per_cu >= 2 ? 2 : 1) * room;
    const int64_t together = (places - 1) / kHardwareQueues + 1, quarter = places / kHardwareQueues;
    const int64_t on_xcd = (replicas + kXcds - 1) / kXcds;
    const int64_t a = (room - 1) / (on_xcd * G), b = together / G;
    const int64_t local = a < b ? a : b;
    const int64_t wide = kXcds * ((quarter < room - 1 ? quarter : room - 1) / G) / replicas;
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

// Updates of one launch of a team, which others that want its CUs wait for: at most so many tiles of a member one after the other
// (50 to 160 ms, a small part of the seconds after which a team that waits goes on without its members).
constexpr int64_t kTeamTilesPerLaunch = 1 << 14;
inline int64_t team_updates_per_launch(int64_t tiles, int members) {
    const int64_t turns = (tiles + members - 1) / members;
    return turns < kTeamTilesPerLaunch ? kTeamTilesPerLaunch / (turns > 0 ? turns : 1) : 1;
}

// The meeting of a team: a word counts its workgroups as they arrive.  Complete, it is a team; a workgroup that has waited too long
// (CUs that another launch holds) closes an incomplete meeting, by a compare-and-swap of the very count that it saw, and then the first
// member does the work alone whenever it gets its CUs: a cluster of one workgroup never gives up.  Whoever looks sees the same.
constexpr uint32_t kMeetingClosed = 1u << 31;
enum Meeting { kMeetingOpen = 0, kMeetingComplete = 1, kMeetingOff = 2 };
constexpr Meeting meeting(uint32_t word, uint32_t all) { return (word & kMeetingClosed) != 0 ? kMeetingOff : (word == all ? kMeetingComplete : kMeetingOpen); }

// Whether every workgroup of a team shares an L2 with those it exchanges with through one: the ids of their XCDs in the order
// [member][slice].  Members that are spread over XCDs exchange their sums through memory, so only the slices of a cluster have to sit
// together; a team that is not spread relies on one L2 as a whole (its sums, and gradients in flight in slots that all members use).
template <typename Id>
constexpr bool team_shares_l2(int members, int G, bool spread, Id id) {
    int first = 0;
    bool same = true;
    for (int q = 0; q < members * G; ++q) {
        const int xcd = id(q);
        if (q == 0 || (spread && q % G == 0)) first = xcd;
        same = same && xcd == first;
    }
    return same;
}

// Which of the two steady-state kernels of K-async is the faster one, for softmax, P <= 8 and updates of one tile: the one that
// keeps gradients in flight in LDS takes a CU per slice and one per replica, the tile kernel a CU or half of one per slice.  Times
// of a launch's update, in hundredths of the tile kernel's with a CU per workgroup (5.3 to 5.8 us): the other kernel's chain is
// shorter while updates rarely consume mini-batches of their own version (K = 2 of 8 workers, 16 replicas of d = 3072: 4.1 us; of 6: 5.9;
// K = 1 of 2: 5.5; K = 3 of 8: 6.3); with two workgroups per CU an update of the tile kernel takes 9.4 to 11.3 us.  Where replicas
// take several launches, these add up (40 replicas of d = 3072, K = 3 of 8: 18.3 us against 10.9; K = 2 of 8, 40 replicas: 11.8
// against 11.0, 48 replicas: 12.2 against 17).  Models of one slice have no exchange to hide: K = 1 only (of 8 workers 3.4 us against 3.8; K = 2 4.45 against 4.16).
inline bool defer_pays(int P, int K, int G, int64_t R, int defer_per_launch, int tile_per_launch, int cus) {
    if (defer_per_launch < 1) return false;
    if (tile_per_launch < 1) return true;
    if (G == 1) return K == 1 && R <= defer_per_launch;
    const int64_t one = 4 * K <= P ? 72 : (K == 1 ? 90 : 102);
    const int64_t rest = R % tile_per_launch;
    auto launch = [&](int64_t replicas) { return (replicas + kXcds - 1) / kXcds * kXcds * G > cus ? 170 : 100; };
    const int64_t tile = R / tile_per_launch * launch(tile_per_launch) + (rest > 0 ? launch(rest) : 0);
    return (R + defer_per_launch - 1) / defer_per_launch * one < tile;
}

}  // namespace ssgd
