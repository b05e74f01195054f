// Steady-state kernel of the linear models (Sec. 2.2, Eq. (2), Eq. (3)) for the common shapes:
// at most 15 classes, at least 4 columns, at most 64 contributors.  A step whose mini-batches do not
// fit one 64-row tile takes several: the synchronous variants take the rows of an iteration's K
// mini-batches 64 at a time, the gradient is summed over the tiles and the update follows the last
// one; the asynchronous ones take whole records per tile, or 64-row blocks of one record.
// (K-async of several tiles and rows of odd length took the general kernel before: P = 20, K = 5, m = 25, d = 785,
// 10 classes, 8 replicas: 50 us per update there, 16 here and 8 with a team.)
// Same cluster decomposition, state layout and arithmetic as the general kernel (linear.hip),
// which runs every other shape and may be mixed with this one launch by launch; what differs
// is the schedule inside a step:
//
//   TU  tile, lists and the updated weights are in LDS          (workgroup barrier)
//       partial logits on the fp32 MFMA units, stored to the cluster's exchange buffer;
//       the parked (stale) part of update v is fetched while the stores travel;
//       each wave polls the partial logits of its 16 rows from all G slices (a word is a
//       sentinel until it has been written), sums them in slice order and goes straight on
//       to residual / softmax in registers; the buffer of the exchange before is re-armed.
//       A cluster that does not sit on one XCD (no shared L2) exchanges through released
//       stores and an arrival counter instead, as does the first exchange of every launch.
//   D   delta in LDS                                            (workgroup barrier)
//       gradient slices delta^T X per record; added to the aggregate or parked;
//       a loader wave (of a team: the compute waves) sums delta's columns: bias gradient, loss, bias step
//   B   the tile has been read                                   (workgroup barrier)
//       compute waves: w -= (lr/K) * aggregate (after the last tile of the update);
//       loader waves: next tile -> LDS
//
// An update of several tiles can be shared by several clusters of its replica, a team (TEAM): each takes every so-many-th tile
// (whole records of the asynchronous variants), adds the gradients in flight that it has computed itself, and after its last
// tile the members exchange their sums, 16 bytes per thread and class row, added by everyone in the members' order, so that the
// weights, of which each has a copy, stay the same bit for bit.  The chain of an update is then one or two tiles long plus one
// exchange (about 2500 cycles) instead of all of them.  Softmax, 10 classes: K-async, P = 20, K = 5, m = 25, d = 785, 8 replicas
// (three tiles, three members) 16.4 -> 8.0 us per update; K-sync, K = 6, m = 84, d = 116, 6 replicas (eight tiles) 24.4 -> 4.9;
// K-batch-async, P = 8, K = 4, m = 115, d = 580, 15 replicas (four records of two tiles) 41.6 -> 14.4.
//
// Four compute waves, four loader waves.  A wave's vector-memory counter retires in order,
// so the long HBM gathers live in waves of their own: the loader waves fetch everything of
// the next tile (lists, sample ids, labels, rows) while the current one is computed, hold the
// rows in registers, and copy them to LDS between B and TU.
#include <type_traits>

#include "common.hpp"

namespace ssgd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int ROWS = 64;        // rows of the LDS tile
constexpr int SL = 256;         // columns per workgroup
constexpr int NTC = 256;        // compute threads
constexpr int LLOADS = 16;      // 16-byte loads per loader lane per tile
constexpr int KC = 64;          // list entries per step (one lane of a wave each)
constexpr int kAgentLoad = 16;  // cache policy: served by the L2, never by a CU's L1
constexpr int kStream = 2;      // cache policy: non-temporal
constexpr int kOwnSlot = 1 << 19;     // in a slot's number (lists in LDS): among the slots of this member of the team
constexpr uint32_t kNoRow = 0xFFFFFFFFu;
constexpr int kOutOfRange = (int)0x80000000;   // offset past any buffer of exchanged words or parked gradients: loads give 0, stores are dropped

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

struct Lds {
    float* tile;      // [64][SL]  16-byte chunk c of row r at chunk position c ^ (r & 15)
    float* wlds;      // [C][SL]   same swizzle, keyed by the class
    float* zbuf;      // [64][16]  delta
    uint32_t* rowid;  // [64]
    float* ylab;      // [64]
    float* bias;      // [16]
    float* small;     // [S][17]   bias gradient and mean loss of every parked slot
    int* ctl;         // [8]: 0 stop, 1 exchange through the shared L2, 2 cluster shares an XCD, 3 exchanges seen by wave 0,
                      //      4 K, 5 records, 6 parked gradients that update v consumes
                      //      TEAM: 2 the team as it runs: its members, or 1
    uint8_t* own;     // TEAM, [S] (the place of `small`): 1 where this member has computed the gradient in flight, in this launch
    int* s_stale;     // [KC] slots of those parked gradients, in the order of the consume list
    int* s_rec;       // [KC] compute list of v: slot of record r; bit 16: consumed by update v itself
};

// (kc: places of the two lists, 32 or 64: the second workgroup of a CU fits only while the lists are short)
__device__ __forceinline__ Lds carve(unsigned char* smem, int C, int S, int kc) {
    Lds l;
    l.tile = reinterpret_cast<float*>(smem);
    l.wlds = l.tile + ROWS * SL;
    l.zbuf = l.wlds + C * SL;
    l.rowid = reinterpret_cast<uint32_t*>(l.zbuf + ROWS * 16);
    l.ylab = reinterpret_cast<float*>(l.rowid + ROWS);
    l.bias = l.ylab + ROWS;
    l.ctl = reinterpret_cast<int*>(l.bias + 16);      // 16-byte aligned: words 4..7 are read as one vector
    l.s_stale = l.ctl + 8;
    l.s_rec = l.s_stale + kc;
    l.small = reinterpret_cast<float*>(l.s_rec + kc);
    l.own = reinterpret_cast<uint8_t*>(l.s_rec + kc);
    return l;
}

// value of lane ^ 1 / lane ^ 2 inside a quad: a data-parallel-primitive move, no LDS round trip
__device__ __forceinline__ float quad_xor1(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float quad_xor2(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
}
[[maybe_unused]] __device__ __forceinline__ float quad_lane0(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x00, 0xF, 0xF, false));   // quad_perm [0,0,0,0]
}

// value of lane ^ 16 / lane ^ 32
template <int MASK>
__device__ __forceinline__ float across(float x, int lane) {
    const uint32_t v = __float_as_uint(x);
    if constexpr (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return __uint_as_float((lane & 16) ? r[0] : r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return __uint_as_float((lane & 32) ? r[0] : r[1]);
    }
}

__device__ __forceinline__ void lds_barrier() {
    // orders LDS traffic only: outstanding global loads and stores stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ONE: the cluster is one workgroup (d <= 256).  Its partial logits are the logits: they change lanes inside the wave
// instead of going out to the exchange, and only the 64-column blocks that exist are loaded, written and contracted.
// Bound by the chain of one step, TU -> logits -> delta -> gradient -> update, beside the chain lists -> sample ids ->
// gather of the next tile.  (Least squares, d = 64, two mini-batches of 16, one replica: 1.4 us per update where the
// exchange through memory of the general kernel takes 8.6.)
// ROOMY: every workgroup takes a CU for itself.  Two waves per SIMD then have 256 registers each and no vector register is
// spilled; a spilled word that a loader wave reads back would wait for the gathers in front of it.  With 128, softmax spills 2 to 4 of
// them where records fill one tile, 10 to 14 where they are described one by one; of a team's forms two do, 11 (synchronous) and 14
// (whole records, several slices).  (1 to 4 % at d = 3072.  Not for
// clusters so wide that those of several launches could keep each other from becoming complete: LinArgs::whole_cus.  Not
// where a launch has more workgroups than the chip has CUs: 1024 replicas of least squares, d = 64, two mini-batches of 16,
// take 6.4 us per update with two workgroups per CU and 10.2 in rounds of one.)
// LATE: when a tile's rows are asked for: as soon as the tile in front of it is in LDS, or behind the description of the tile
// after it, some 3000 cycles later.  The gathers keep the memory path of the CU busy for 4000 cycles, and what the compute
// waves have to wait for meanwhile (parked gradients, partial logits and the stores in front of them) queues behind them, so
// they go late wherever there is an exchange: softmax, d = 3072, two mini-batches of 32, 8 replicas: K-sync 5.46 -> 4.85 us per
// update, K-batch-async 6.90 -> 6.05; early where nothing is waited for (synchronous iterations of one slice), and for
// synchronous iterations with two workgroups per CU (K-batch-sync of 16 x 128, 40 replicas: 285 early, 281 to 292 late).
template <int KIND, bool PROF, bool WHOLE, bool CHUNKED, bool BATCH, bool ONE, bool ROOMY, bool LATE, bool TEAM>
__global__ __launch_bounds__(512, ROOMY ? 2 : 4) void linear_tile_kernel(LinArgs a) {
    // consecutive block ids go to different XCDs: all slices of one cluster take block ids that
    // are congruent modulo 8 and share one L2
    const int xcd = blockIdx.x & 7, slot_in_xcd = blockIdx.x >> 3;
    int pos = slot_in_xcd / a.G, slice = slot_in_xcd % a.G;
    int member = 0;
    if constexpr (TEAM) { if (!a.spread) { member = pos % a.team; pos /= a.team; } }
    if (!TEAM && a.pair_cus > 0) {
        // The dispatcher hands the first pair_cus slots of an XCD to distinct CUs and the next pair_cus slots
        // to the same CUs again.  A cluster takes G CUs of one such layer, so the clusters on those G CUs
        // share them with each other only and run in alternation; the CUs left over hold one more cluster.
        const int L = a.pair_cus, layers = a.pair_layers;
        const int layer = slot_in_xcd / L, cu = slot_in_xcd % L;
        const int nb = L / a.G, Lr = L - nb * a.G;
        if (cu < nb * a.G) { pos = (cu / a.G) * layers + layer; slice = cu % a.G; }
        else { const int rem = (cu - nb * a.G) + layer * Lr; pos = nb * layers + rem / a.G; slice = rem % a.G; }
    }
    int cluster = pos * 8 + xcd;
    if constexpr (TEAM) { if (a.spread) { member = cluster % a.team; cluster /= a.team; } }
    if (cluster >= a.replicas) return;
    const int rep = a.replica0 + cluster;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = a.d, C = a.C, m = a.m, mp = a.mp, S = a.S, G = a.G;
    const int Kcap = a.tr.Kcap;
    const int64_t cap = a.tr.cap;
    const int col0 = slice * SL;
    const bool async = !CHUNKED && (!BATCH || a.variant == kAsync);      // K-async
    // A tile holds whole records of mp rows; when an iteration spans several tiles, a tile is one block of 64 rows
    // of the iteration's mini-batches, all of them part of the update.
    constexpr bool chunked = CHUNKED;
    // One slice: the loader waves draw the ids of the tile after next while the gradient is contracted, and ask for the labels
    // with the rows; wave 3, which takes the bias sums meanwhile, and wave 0, which has the lists, get the ids from wave 1.  (With all of it in front of barrier
    // D they took 2700 cycles there, the compute waves 1600: softmax, d = 60, 25 rows, 40 replicas 4.27 -> 4.07 us per update; a team,
    // least squares, d = 167, K-sync of 3 x 39 3.05 -> 2.64, softmax, d = 199, K-async of 2 x 62 6.0 -> 5.5.)
    constexpr bool SPLIT = ONE;
    // Records described one by one (BATCH: K-batch-async, and K-async when a version may have more records than a tile
    // holds), mini-batches of more than 64 rows: a tile is one block of 64 rows of one record; the record's gradient is
    // summed over its tiles in the slot of its worker
    const int spr = (BATCH && mp > ROWS) ? (mp + ROWS - 1) / ROWS : 1;      // tiles per record
    const int mpt = (chunked || spr > 1) ? ROWS : mp;
    const int nblk = ONE ? (d + 63) >> 6 : SL / 64;      // 64-column blocks in use
    const int crew = TEAM ? rep * a.team + member : rep;  // whose exchange buffers of partial logits

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int kc = Kcap > 32 ? KC : 32;      // places of the lists in LDS
    const Lds L = carve(smem, C, S, kc);

    if (wave >= 4) {
        // =============================== loader waves ===============================
        const int lw = wave - 4;
        const int32_t* tr_sel = a.tr.sel + (int64_t)rep * cap * Kcap;
        const int32_t* tr_tau = a.tr.tau + (int64_t)rep * cap * Kcap;
        const int32_t* tr_ord = a.tr.ord + (int64_t)rep * cap * Kcap;
        const __amdgpu_buffer_rsrc_t xrsrc = make_rsrc(a.X, (uint32_t)((uint64_t)a.N * d * 4u));
        const uint32_t row_bytes = (uint32_t)d * 4u;

        // tile row `lane` is sample s_of of record r_of
        const int r_of = lane / mp, s_of = lane % mp;
        // Row lw + 4 i of the tile is fetched by instruction i of this wave, one 16-byte chunk per lane.
        // The swizzle is applied on the global side: lane l fetches chunk l ^ key and writes position l.
        // A row may start at any 4-byte address, which is all that a 16-byte buffer load asks for.  The last chunk of a row
        // of odd length is read as the row's last four columns and moved into place on its way to LDS, zeros behind them:
        // nothing is read past the row.
        int goff[4];
        bool tail[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int key = (lw + 4 * q) & 15;
            const int col = col0 + 4 * (lane ^ key);
            tail[q] = col < d && col + 4 > d;
            goff[q] = (col < d) ? min(col, d - 4) * 4 : (int)kPastMatrix;    // past the end of the row: zeros
        }
        const int d_rem = d & 3;
        const bool has_tail = d_rem != 0 && slice == G - 1;
        float* const my_tile = L.tile + lw * SL + lane * 4;

        // A tile is described (sample ids, labels, lists: n_*) one turn before its rows are gathered; what is published is the
        // description p_* of the tile whose rows are in `pref`.
        f32x4 pref[LLOADS];
#pragma unroll
        for (int i = 0; i < LLOADS; ++i) pref[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        uint32_t row_id = kNoRow, p_row_id = kNoRow;
        float row_lab = 0.0f, p_row_lab = 0.0f;
        int n_K = 0, n_nrec = 0, n_nstale = 0, n_stale = 0, n_stale_pos = KC, n_rec_word = 0, n_rows = mpt, n_flags = 0;
        int p_K = 0, p_nrec = 0, p_nstale = 0, p_stale = 0, p_stale_pos = KC, p_rec_word = 0, p_rows = mpt, p_flags = 0;
        int64_t n_ver = 0, p_ver = 0;
        int q_sel = -1, q_tau = -1, q_ord = 0;   // lane l: entry l of the consume list of a later version, in flight
        int cur_sel = -1;                        // consume list of the version before the one being prepared

        // diagnostics: cycles between passing mark prof_a and the next passing of mark prof_b, summed in scalar registers
        uint32_t lp_acc = 0, lp_t0 = 0;
        const bool lprof = PROF && lw == a.prof_wave;
        auto lmark = [&](int q) {
            if constexpr (PROF) {
                if (lprof) {
                    if (16 + q == a.prof_a) lp_t0 = (uint32_t)clock64();
                    if (16 + q == a.prof_b) lp_acc += (uint32_t)clock64() - lp_t0;
                }
            }
        };

        // (every lane loads, on every turn: a load under a condition would be copied where the paths meet, and the copy
        // waits for it and for the gathers in front of it; lanes past the list are masked when it is taken)
        const int q_lane = min(lane, Kcap - 1);
        auto issue_lists = [&](int64_t ver) {
            q_sel = tr_sel[ver * Kcap + q_lane];
            q_tau = tr_tau[ver * Kcap + q_lane];
            q_ord = tr_ord[ver * Kcap + q_lane];
        };
        // The lists of version `ver` (in flight in q_*) become the description of its tiles.
        int h_worker = -1, h_ord = 0, h_nrec = 0, h_tiles = 1;
        // K-batch-async: the records of a version are described piecewise (version 0 has P + K - 1 of them):
        // the first `h_first` start a worker's mini-batch 0 (version 0: worker = record index; later: the worker whose
        // push triggered the update before), record h_first + j is the restart after push j of this update (lane j)
        int h_first = 0, h_trig = 0, h_trig_fresh = 0, h_nstale = 0;
        int h_rw = 0, h_ro = 0, h_rf = 0;        // lane j: worker, ordinal, consumed-by-this-update flag of restart j
        int h_csel = -1, h_ctau = -1, h_cord = 0;   // lane l: entry l of the consume list of the version
        const int rpt = TEAM && BATCH ? a.team_rpt : (spr > 1 ? 1 : ROWS / mp); // whole records per tile (or one block of a record)
        const int own_slots = TEAM && BATCH && a.own_slots > 0 ? kOwnSlot : 0;
        int team = 1, h_total = 1;               // TEAM: members; tiles of the version over all of them (records of several tiles: records)
        auto take_lists = [&](int64_t ver) {
            const int l_sel = lane < Kcap ? q_sel : -1, l_tau = lane < Kcap ? q_tau : -1, l_ord = lane < Kcap ? q_ord : 0;
            const int K = __popcll(__ballot(l_sel >= 0));
            int nrec = async ? __popcll(__ballot(cur_sel >= 0)) : K;
            int rec_slot = async ? cur_sel : lane;
            int rec_ord = async ? 0 : l_ord;
            int fr = (!async && lane < K) ? 1 : 0;
            if (async)
                for (int l = 0; l < K; ++l)
                    if (__builtin_amdgcn_readlane(l_tau, l) == (int32_t)ver && __builtin_amdgcn_readlane(l_sel, l) == rec_slot) fr = 1;
            if constexpr (BATCH) {
                // Mini-batches that start at version ver: at ver = 0 every worker's first one.  Later, K-async: those of
                // the workers that update ver - 1 consumed, all listed as restarts.
                if (async) {
                    h_first = (ver == 0) ? a.P : 0;
                    nrec = (ver == 0) ? a.P : nrec;
                    h_trig = 0; h_trig_fresh = 0;
                    h_rw = rec_slot; h_ro = 0; h_rf = fr;
                } else {
                // K-batch-async: the one of the worker whose push triggered update ver - 1; then, for each of the first
                // K - 1 pushes of update ver, the next mini-batch of the pushing worker (ordinal: how many it has started
                // at this version).
                const int Kprev = __popcll(__ballot(cur_sel >= 0));
                h_first = (ver == 0) ? a.P : 1;
                nrec = h_first + K - 1;
                h_trig = (ver == 0) ? 0 : __builtin_amdgcn_readlane(cur_sel, max(Kprev - 1, 0));
                h_rw = l_sel;
                h_ro = (l_tau == (int32_t)ver) ? l_ord + 1 : 0;
                h_rf = 0;          // is restart `lane` consumed by update ver itself?  and the trigger's mini-batch?
                h_trig_fresh = 0;
                for (int q = 0; q < K; ++q) {
                    const int cs = __builtin_amdgcn_readlane(l_sel, q), ct = __builtin_amdgcn_readlane(l_tau, q),
                              co = __builtin_amdgcn_readlane(l_ord, q);
                    if (ct == (int32_t)ver && cs == h_rw && co == h_ro) h_rf = 1;
                    if (ct == (int32_t)ver && cs == h_trig && co == 0) h_trig_fresh = 1;
                }
                }
                h_csel = l_sel; h_ctau = l_tau; h_cord = l_ord;
            }
            n_K = K;
            // parked gradients that update ver consumes: entries whose version is older, compacted
            bool is_stale = lane < K && l_tau != (int32_t)ver;
            int l_own = 0;
            if constexpr (TEAM && BATCH) {
                // each by the member that computed it: nobody reads what another CU has written.  Who computed those of earlier
                // launches follows from their place among the records of their version, so that the sums do not depend on
                // where a launch ended.
                if (lw == 0) {
                    const int q = is_stale ? l_sel : 0;
                    bool mine = is_stale && L.own[q] != 0;
                    if (mine) { L.own[q] = 0; l_own = own_slots; }
                    for (unsigned long long old = __ballot(is_stale && l_tau < (int32_t)a.v0); old != 0; old &= old - 1) {
                        const int l = __builtin_ctzll(old);
                        const int w = __builtin_amdgcn_readlane(l_sel, l), tau = __builtin_amdgcn_readlane(l_tau, l);
                        int place = w;
                        if (async) {
                            if (tau > 0) place = __builtin_ctzll(__ballot(tr_sel[(int64_t)(tau - 1) * Kcap + q_lane] == w) | (1ull << 63));
                        } else {
                            // a restart during update tau, or what its trigger (tau = 0: the worker) began at tau
                            const int o = __builtin_amdgcn_readlane(l_ord, l);
                            const int s_ = tr_sel[(int64_t)tau * Kcap + q_lane], t_ = tr_tau[(int64_t)tau * Kcap + q_lane],
                                      o_ = tr_ord[(int64_t)tau * Kcap + q_lane];
                            const int pushes = __popcll(__ballot(lane < Kcap && s_ >= 0));
                            const unsigned long long at = __ballot(lane < pushes - 1 && s_ == w && (t_ == tau ? o_ + 1 : 0) == o);
                            if (at != 0) place = (tau > 0 ? 1 : a.P) + __builtin_ctzll(at);
                            else if (tau > 0) place = 0;
                        }
                        if (lane == l) mine = (place / rpt) % team == member;
                    }
                    is_stale = mine;
                }
            }
            const unsigned long long smask = __ballot(is_stale);
            n_nstale = __popcll(smask);
            n_stale = (async || BATCH) ? (l_sel | l_own) : lane;
            n_stale_pos = is_stale ? __popcll(smask & ((1ull << lane) - 1ull)) : KC;
            if (chunked) {
                // every tile is one record of 64 rows that update ver consumes itself
                n_nrec = 1;
                n_rec_word = (lane == 0) ? (1 << 16) : 0;
            } else {
                n_nrec = nrec;
                n_rec_word = (lane < nrec) ? (rec_slot | (fr << 16)) : 0;      // K-batch-async: set per tile below
            }
            h_worker = async ? cur_sel : l_sel;      // lane r: worker of record r (not K-batch-async)
            h_ord = rec_ord;
            h_nrec = nrec;
            h_tiles = chunked ? max(1, (nrec * mp + ROWS - 1) / ROWS) : 1;
            if constexpr (BATCH) {
                h_nstale = n_nstale;
                h_tiles = spr > 1 ? max(1, nrec * spr) : max(1, (nrec + rpt - 1) / rpt);
            }
            if constexpr (TEAM) {
                // every team-th tile, or every team-th record of several tiles; an empty tile where none is left
                h_total = BATCH && spr > 1 ? nrec : h_tiles;
                h_tiles = max(1, (BATCH && spr > 1 ? spr : 1) * ((h_total - member + team - 1) / team));
            }
            cur_sel = l_sel;
            if constexpr (chunked) asm volatile("" : "+v"(h_worker), "+v"(h_ord) : : "memory");
            else asm volatile("" : "+v"(n_stale), "+v"(n_stale_pos), "+v"(n_rec_word), "+v"(cur_sel), "+v"(h_worker), "+v"(h_ord) : : "memory");
            if constexpr (BATCH) asm volatile("" : "+v"(h_rw), "+v"(h_ro), "+v"(h_rf), "+v"(h_csel), "+v"(h_ctau), "+v"(h_cord) : : "memory");
        };
        // Tile `t` of version `ver`: sample ids, lists; leaves the labels in flight.
        // (SPLIT, in the loop: lists by wave 0, which publishes them, ids by waves 1 and 2)
        auto describe_tile = [&](int64_t ver, int t_mine, bool all) {
            const bool lists = !SPLIT || all || lw == 0, draws = !SPLIT || all || lw == 1 || lw == 2;
            n_ver = ver;
            n_flags = (t_mine + 1 == h_tiles ? 1 : 0) | (t_mine == 0 ? 2 : 0);      // bit 0 last tile of its update, bit 1 first
            int t = t_mine;
            if constexpr (TEAM) t = BATCH && spr > 1 ? (member + team * (t_mine / spr)) * spr + t_mine % spr : member + team * t_mine;
            n_rows = mpt;                                                 // rows per record in this tile
            int rec = r_of, smp = s_of;
            if (chunked) {
                // one record; the contraction takes 32 rows at a time
                n_rows = (min(ROWS, h_nrec * mp - t * ROWS) > 32) ? ROWS : 32;
                if constexpr (TEAM) n_nrec = t < h_total ? 1 : 0;
                if (t > 0) { const int q = t * ROWS + lane; rec = q / mp; smp = q - rec * mp; }
            }
            int worker = 0, ordinal = 0;
            if constexpr (BATCH) {
                // records t * rpt .. of the version; the parked part of the update comes with the first tile
                const int tr0 = spr > 1 ? t / spr : t * rpt;       // first record of the tile
                const int blk = spr > 1 ? t % spr : 0;             // which block of 64 rows of its record
                rec = (r_of < rpt) ? tr0 + r_of : 0x7FFFFFF;
                if (spr > 1) { rec = tr0; smp = ROWS * blk + lane; n_rows = WHOLE ? ROWS : min(ROWS, mp - ROWS * blk); }
                n_nrec = spr > 1 ? 1 : min(rpt, h_nrec - t * rpt);
                if constexpr (TEAM) n_nrec = spr > 1 ? (tr0 < h_nrec ? 1 : 0) : max(0, n_nrec);
                n_nstale = (t_mine == 0) ? h_nstale : 0;
                // worker, ordinal and consumed-by-this-update flag of record q
                auto describe = [&](int q, int& w, int& o, int& f) {
                    const int j = min(max(q - h_first, 0), 63);
                    const int rw = __shfl(h_rw, j, 64), ro = __shfl(h_ro, j, 64), rf = __shfl(h_rf, j, 64);
                    if (q >= h_first) { w = rw; o = ro; f = rf; }
                    else if (ver != 0) { w = h_trig; o = 0; f = h_trig_fresh; }
                    else { w = q; o = 0; f = -1; }          // version 0: looked up below
                };
                int fr;
                if (draws) describe(rec, worker, ordinal, fr);
                if (lists) {
                int qw, qo, qf;
                describe(tr0 + lane, qw, qo, qf);
                if (ver == 0) {
                    // every worker's first mini-batch: consumed by update 0 if the list holds (worker, version 0, ordinal 0)
                    const int Kv = n_K;
                    int hit = 0;
                    for (int e = 0; e < Kv; ++e)
                        if (__builtin_amdgcn_readlane(h_csel, e) == qw && __builtin_amdgcn_readlane(h_ctau, e) == 0 &&
                            __builtin_amdgcn_readlane(h_cord, e) == 0) hit = 1;
                    if (qf < 0) qf = hit;
                }
                // bit 16: consumed by the update of its own version; bit 17: the record goes on in the next tile; bit 18: it
                // began in an earlier tile
                n_rec_word = (lane < n_nrec) ? (qw | (qf << 16) | ((blk + 1 < spr ? 1 : 0) << 17) | ((blk > 0 ? 1 : 0) << 18)) : 0;
                if constexpr (TEAM) {
                    if (lw == 0 && lane < n_nrec && qf == 0) {
                        L.own[qw] = 1;
                        n_rec_word |= own_slots;
                    }
                }
                }
            } else {
                worker = __shfl(h_worker, min(rec, 63), 64);
                ordinal = __shfl(h_ord, min(rec, 63), 64);
            }
            if (!draws) return;
            uint32_t seed_lo = (uint32_t)a.seed, seed_hi = (uint32_t)(a.seed >> 32);
            asm volatile("" : "+s"(seed_lo), "+s"(seed_hi));      // the round keys are rebuilt here: kept across the loop they are spilled
            const uint32_t id = batch_index(((uint64_t)seed_hi << 32) | seed_lo, (uint32_t)rep, (uint32_t)worker, (uint32_t)ordinal, (uint32_t)ver,
                                            (uint32_t)smp, a.N);
            if constexpr (!SPLIT) row_lab = reinterpret_cast<const float*>(a.y)[id];    // fp32 or int32: the word as it is
            row_id = (smp < m && rec < h_nrec) ? id : kNoRow;
        };
        // The tile described last becomes the one whose rows are gathered.
        auto adopt = [&]() {
            p_row_id = row_id;
            if constexpr (!SPLIT) p_row_lab = row_lab;
            p_K = n_K; p_nrec = n_nrec; p_nstale = n_nstale; p_stale = n_stale; p_stale_pos = n_stale_pos; p_rec_word = n_rec_word;
            p_rows = n_rows; p_flags = n_flags; p_ver = n_ver;
            if constexpr (SPLIT) p_row_lab = reinterpret_cast<const float*>(a.y)[p_row_id == kNoRow ? 0u : p_row_id];
            else asm volatile("" : "+v"(p_row_lab) : : "memory");
            if constexpr (chunked) asm volatile("" : "+v"(p_row_id) : : "memory");
            else asm volatile("" : "+v"(p_row_id), "+v"(p_stale), "+v"(p_stale_pos), "+v"(p_rec_word) : : "memory");
        };
        // Its gathers.  A wave's loads return in order, so what is asked for afterwards must not be needed before the rows are.
        auto gather = [&]() {
            int olw = lw;
            asm volatile("" : "+s"(olw));
            const int used = p_nrec * p_rows;      // a CU takes in about 16 bytes of gathers per cycle: rows past the records are left out
            __builtin_amdgcn_sched_barrier(0);
            if (!ONE || lane < 16 * nblk) {
#pragma unroll
                for (int i0 = 0; i0 < LLOADS; i0 += 4) {
                    if (4 * i0 >= used) break;
#pragma unroll
                    for (int i = i0; i < i0 + 4; ++i) {
                        // rows without a sample are zero: their delta is, but zero times an infinity is not
                        const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)p_row_id, olw + 4 * i);
                        const bool none = id == kNoRow;
                        pref[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, none ? (int)kPastMatrix : goff[i & 3],
                                                                                                  none ? 0 : (int)(id * row_bytes), kStream));
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto publish = [&]() {
            if (has_tail) {
#pragma unroll
                for (int i = 0; i < LLOADS; ++i) {
                    const f32x4 r = pref[i];
                    const f32x4 moved = {d_rem == 1 ? r.w : (d_rem == 2 ? r.z : r.y), d_rem == 1 ? 0.0f : (d_rem == 2 ? r.w : r.z),
                                         d_rem == 3 ? r.w : 0.0f, 0.0f};
                    pref[i] = tail[i & 3] ? moved : r;
                }
            }
            if (!ONE || lane < 16 * nblk) {
                // (rows past the records have no sample: whatever is there, their logits are not used)
                const int used = p_nrec * p_rows;
#pragma unroll
                for (int i0 = 0; i0 < LLOADS; i0 += 4) {
                    if (4 * i0 >= used) break;
#pragma unroll
                    for (int i = i0; i < i0 + 4; ++i) *reinterpret_cast<f32x4*>(my_tile + 4 * i * SL) = pref[i];
                }
            }
            if (lw == (SPLIT ? 3 : 0)) L.ylab[lane] = p_row_lab;
            if (lw == 0) {
                L.rowid[lane] = p_row_id;
                if (lane == 0) { L.ctl[4] = p_K; L.ctl[5] = p_nrec; L.ctl[6] = p_nstale; L.ctl[7] = p_flags | (p_rows << 8); }
                if (!chunked && p_stale_pos < kc) L.s_stale[p_stale_pos] = p_stale;
                if (lane < kc) L.s_rec[lane] = chunked ? 1 << 16 : p_rec_word;       // (only the first entry is read)
            }
            if constexpr (SPLIT) asm volatile("" : "+v"(q_sel), "+v"(q_tau), "+v"(q_ord) : : "memory");
            else asm volatile("" : "+v"(q_sel), "+v"(q_tau), "+v"(q_ord), "+v"(row_lab) : : "memory");     // lists and labels asked for behind the rows
        };

        // One loader wave (0; one slice: 3), between D and B: the column sums of the delta tile per record, i.e. the bias
        // gradient (classes 0..C-1) and the mean mini-batch loss (class 15), summed over the consume
        // list of update v like the weight gradients; then the bias step and the loss record.  (A team's compute waves take
        // these sums themselves.)
        float run_tot = 0.0f;      // sums of the earlier tiles of the same update
        auto bias_and_loss = [&](int64_t v, int flags) {
            const int Kv = __builtin_amdgcn_readfirstlane(L.ctl[4]);
            const int n_rec = __builtin_amdgcn_readfirstlane(L.ctl[5]);
            const int n_st = __builtin_amdgcn_readfirstlane(L.ctl[6]);
            // (a tile of one record that the update consumes: four parts, so that no lane idles)
            const int parts = chunked ? 4 : n_rec, rows = chunked ? flags >> 10 : flags >> 8;
            // lane = class + 16 * (record within a batch of four records)
            const int c = lane & 15, grp = lane >> 4;
            const int sidx = (c == 15) ? 16 : c;          // the slot record keeps the loss in word 16
            float tot = 0.0f;
            for (int i = 0; i < n_st; ++i) {
                const float was = L.small[__builtin_amdgcn_readfirstlane(L.s_stale[i]) * 17 + sidx];
                if (grp == 0) tot += was;
            }
            for (int r0 = 0; r0 < parts; r0 += 4) {
                const int r = r0 + grp;
                const bool have = r < parts;
                const float* zp = L.zbuf + (have ? r : 0) * rows * 16 + c;
                float p0 = 0.0f, p1 = 0.0f;
                int i0 = 0;
                for (; i0 + 16 <= rows; i0 += 16) {     // sixteen rows in flight
                    float t[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) t[i] = zp[(i0 + i) * 16];
#pragma unroll
                    for (int i = 0; i < 16; i += 2) { p0 += t[i]; p1 += t[i + 1]; }
                }
                for (; i0 < rows; i0 += 4) {
                    float t[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = zp[(i0 + i) * 16];
                    p0 += t[0] + t[2];
                    p1 += t[1] + t[3];
                }
                const float part = p0 + p1;
                const int word = have ? (chunked ? 1 << 16 : L.s_rec[r]) : 0;
                if (have) {
                    if (((word >> 16) & 1) != 0) tot += part;
                    else if (((word >> 18) & 1) != 0) L.small[(word & 0xFFFF) * 17 + sidx] += part;    // a later block of its record
                    else L.small[(word & 0xFFFF) * 17 + sidx] = part;
                }
            }
            tot += __shfl_xor(tot, 16, 64);
            tot += __shfl_xor(tot, 32, 64);
            if ((flags & 2) == 0) tot += run_tot;
            run_tot = tot;
            if ((flags & 1) != 0) {
                if (KIND == kSoftmax && lane < C) L.bias[lane] -= (a.lr / (float)Kv) * tot;
                if (lane == 15 && slice == 0) a.tr.loss[(int64_t)rep * cap + v] = tot * (1.0f / (float)Kv);
                // the averaged gradient of replica 0, when the caller asked for it: bias part
                if (KIND == kSoftmax && a.agg_out != nullptr && rep == 0 && slice == 0 && lane < C)
                    a.agg_out[(int64_t)C * d + lane] = tot * (1.0f / (float)Kv);
            }
        };

        lds_barrier();                               // the compute waves have set up the control words
        if (L.ctl[0] != 0) return;
        if ((async || BATCH) && a.v0 >= 1 && lane < Kcap) cur_sel = tr_sel[(a.v0 - 1) * Kcap + lane];
        if constexpr (TEAM) team = __builtin_amdgcn_readfirstlane(L.ctl[2]);
        if constexpr (TEAM && BATCH) {
            if (lw == 0)
                for (int q = lane; q < S; q += 64) L.own[q] = 0;
        }
        int64_t at = 0;                              // update and tile described last
        int at_tile = 0;
        issue_lists(a.v0);
        take_lists(a.v0);
        issue_lists(a.v0 + min((int64_t)1, a.nsteps - 1));
        describe_tile(a.v0, 0, true);
        asm volatile("" : "+v"(q_sel), "+v"(q_tau), "+v"(q_ord), "+v"(row_lab) : : "memory");
        bool more = true;                            // the tile described last is still to be gathered
        auto turn = [&]() {
            adopt();
            if constexpr (!LATE) gather();
            if (at_tile + 1 < h_tiles) {
                ++at_tile;
            } else if (at + 1 < a.nsteps) {
                ++at; at_tile = 0;
                take_lists(a.v0 + at);
            } else {
                more = false;
            }
            issue_lists(a.v0 + min(at + 1, a.nsteps - 1));
            if constexpr (!SPLIT) describe_tile(a.v0 + at, at_tile, true);       // past the last tile: that tile again, never gathered
            if constexpr (LATE) {
                if constexpr (!SPLIT) asm volatile("" : "+v"(row_id) : : "memory");
                gather();
            }
        };
        // the rest of the tile that the compute waves work on; false: the launch is aborted
        auto rest = [&](int64_t v, int flags, bool turned) -> bool {
            lmark(1);
            lds_barrier();                           // D
            if (L.ctl[0] != 0) return false;
            if (!TEAM && lw == (SPLIT ? 3 : 0)) bias_and_loss(v, flags);
            if constexpr (SPLIT) {
                if (turned) {
                    describe_tile(a.v0 + at, at_tile, false);
                    // for waves 0 and 3, from whom the next words of these places come; the compute waves are done with them
                    if (lw == 1) { L.rowid[lane] = row_id; L.ylab[lane] = __uint_as_float(row_id); }
                }
            }
            lmark(2);
            lds_barrier();                           // B
            if constexpr (SPLIT) {
                if (turned && lw == 0) row_id = L.rowid[lane];
                if (turned && lw == 3) row_id = __float_as_uint(L.ylab[lane]);
            }
            lmark(3);
            return true;
        };
        turn();
        if constexpr (SPLIT) describe_tile(a.v0 + at, at_tile, true);
        for (;;) {
            lmark(4);
            publish();
            lmark(0);
            const int64_t v = p_ver;
            const int flags = p_flags | (p_rows << 8);
            lds_barrier();                           // TU
            if (!more) {
                if (!rest(v, flags, false)) return;
                break;
            }
            turn();
            if (!rest(v, flags, true)) return;
        }
        if constexpr (PROF) {
            if (lprof && lane == 0 && member == 0) a.prof[(int64_t)a.prof_base + ((int64_t)rep * G + slice) * 2 + 1] += lp_acc;
        }
        lds_barrier();                               // the compute waves' last LDS writes
        return;
    }

    // ================================= compute waves =================================
    const int64_t nw = (KIND == kLsq) ? d : (int64_t)C * d + C;
    float* params = a.params + (int64_t)rep * nw;
    const int nt = ONE ? a.park_threads : NTC;            // threads in the layout of the parked gradients
    float* park = a.park + ((int64_t)rep * G + slice) * S * 16 * nt;
    float* small_g = a.park_small + ((int64_t)rep * G + slice) * S * 17;
    float* zpart = a.zpart + (int64_t)rep * 2 * G * a.maxrows * 16;
    unsigned int* arrive = a.arrive + kArriveStride * rep;   // fenced exchanges; word kArriveFast: shared-L2 exchanges
    const float inv_m = 1.0f / (float)m;
    const int nquad = (C + 3) / 4;

    // share of the parameters: classes own_cls .. own_cls+3, columns own_col .. own_col+3
    const int own_ch = 16 * wave + (lane & 15);
    const int own_col = col0 + 4 * own_ch;
    const int own_cls = 4 * (lane >> 4);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int cls = own_cls + v;
        if (cls < C) {
            f32x4 val;
#pragma unroll
            for (int c = 0; c < 4; ++c) val[c] = (own_col + c < d) ? params[(int64_t)cls * d + own_col + c] : 0.0f;
            *reinterpret_cast<f32x4*>(L.wlds + cls * SL + ((own_ch ^ cls) << 2)) = val;
        }
    }
    if (tid < 16) L.bias[tid] = (KIND == kSoftmax && tid < C) ? params[(int64_t)C * d + tid] : 0.0f;
    if constexpr (!TEAM)
        for (int q = tid; q < S * 17; q += NTC) L.small[q] = small_g[q];
    if (tid == 0) {
        L.ctl[0] = __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        L.ctl[1] = 0;   // fenced until the cluster is known to share an XCD
        L.ctl[2] = 0;
        L.ctl[3] = 0;
        // XCC_ID in the low byte (what the same-XCD check compares); HW_ID (CU, shader engine) above it, for diagnostics
        const int my_xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xF);
        const int hw_id = (int)__builtin_amdgcn_s_getreg((15 << 11) | 4);
        __hip_atomic_store(a.xcc_ids + (int64_t)crew * G + slice, my_xcc | (hw_id << 8), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (TEAM) {
            // The team meets once: where everyone has come and those who exchange through an L2 share one it goes on as a team; else
            // its first member goes on alone and the others leave.
            const int all = a.team * G;
            unsigned int* met = a.arrive + kArriveStride * rep + kArriveTeam;
            if ((a.debug_flags & 4) != 0) __hip_atomic_fetch_or(met, kMeetingClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(met, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t spins = 0;
            Meeting seen = kMeetingOpen;
            while (L.ctl[0] == 0) {
                uint32_t word = __hip_atomic_load(met, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                seen = meeting(word, (uint32_t)all);
                if (seen != kMeetingOpen) break;
                __builtin_amdgcn_s_sleep(8);
                ++spins;
                if (spins > a.spin_limit)
                    __hip_atomic_compare_exchange_strong(met, &word, word | kMeetingClosed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else if ((spins & 63u) == 0 && __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
                    L.ctl[0] = 1;
            }
            const bool together = seen == kMeetingComplete && team_shares_l2(a.team, G, a.spread != 0, [&](int q) {
                return __hip_atomic_load(a.xcc_ids + (int64_t)rep * all + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFF;
            });
            int same = a.allow_fast && together ? 1 : 0;
            if ((a.debug_flags & 1) != 0 && (rep & 1) != 0) same = 0;
            L.ctl[1] = same;
            L.ctl[2] = same ? a.team : 1;
            if (!same && member > 0) L.ctl[0] = 1;
        }
    }
    __syncthreads();
    if (L.ctl[0] != 0) return;

    const __amdgpu_buffer_rsrc_t zrsrc = make_rsrc(zpart, (uint32_t)(2u * G * a.maxrows * 16u * sizeof(float)));
    // shared-L2 exchange: three buffers of G x 64 x 16 words used in turn; a word is the sentinel until written
    const __amdgpu_buffer_rsrc_t ersrc = make_rsrc(a.zx + (int64_t)crew * 3 * G * 1024, (uint32_t)(3u * G * 4096u));
    constexpr uint32_t kSentinel = 0xFFFFFFFFu;
    // parked gradients of this workgroup: class own_cls + vv of slot s, 4 columns: 16 bytes at ((s*4 + vv)*nt + tid)*16
    // TEAM: slots of this member.  K-batch-async, where a worker's gradient can be added by one member in the update in which
    // another parks the worker's next one, and teams on several XCDs, whose L2s must not hold the same slot, park here and put
    // what is in flight at the end of a launch where everyone finds it.  Behind them one slot in which a record of several
    // tiles is summed, since several records of a worker may be under way.
    const int64_t own_base = (((int64_t)rep * G + slice) * a.team + member) * (a.own_slots + 1);
    float* park2 = TEAM && BATCH ? a.park2 + own_base * 16 * nt : nullptr;
    float* small2 = TEAM && BATCH ? a.park2_small + own_base * 17 : nullptr;
    auto small_of = [&](int word) {      // bias gradients and losses
        const bool own = (word & kOwnSlot) != 0;
        return make_rsrc(own ? small2 : small_g, (uint32_t)(own ? a.own_slots + 1 : S) * 68u);
    };
    auto park_of = [&](int word) {
        const bool own = (word & kOwnSlot) != 0;
        return make_rsrc(own ? park2 : park, (uint32_t)(own ? a.own_slots + 1 : S) * 16u * nt * 4u);
    };
    const int scratch = a.own_slots | kOwnSlot;
    const __amdgpu_buffer_rsrc_t prsrc = make_rsrc(park, (uint32_t)S * 16u * nt * 4u);
    // (TEAM: offsets are derived from an opaque copy of the thread's number where they are used: kept across the loop more of them are
    // spilled where 128 registers have to do, and a spilled word that is read back waits behind the gathers.)
    auto myself = [&]() { int t = tid; asm volatile("" : "+v"(t)); return t; };
    auto owner = [&]() { if constexpr (TEAM) return myself(); else return tid; };
    auto pk_off = [&](int t, int vv) { return (4 * ((t & 63) >> 4) + vv < C && (!ONE || t < nt)) ? (vv * nt + t) * 16 : kOutOfRange; };
    // forward: rows 16 wave .. 16 wave + 15; row / class index of this lane in the MFMA operands
    const int f_row = 16 * wave + (lane & 15);
    // lanes of classes that do not exist read the last class: their logits are never used
    const int f_key = min(lane & 15, C - 1);
    // k-block s covers 16-byte chunks 4 s + lane/16 of the row; with the swizzle key split as
    // key = 4 k2 + k0 its position is 16 (s / 4) + 4 ((s % 4) ^ k2) + ((lane / 16) ^ k0): four base
    // addresses per operand, which differ in two bits, the rest is a constant offset
    const int f_x0 = f_row * SL + ((4 * ((f_row & 15) >> 2) + ((lane >> 4) ^ (f_row & 3))) << 2);
    const int f_w0 = f_key * SL + ((4 * (f_key >> 2) + ((lane >> 4) ^ (f_key & 3))) << 2);
    auto f_xa = [&](int s) { return *reinterpret_cast<const f32x4*>(L.tile + (f_x0 ^ ((s & 3) << 4)) + (s >> 2) * 64); };
    auto f_wa = [&](int s) { return *reinterpret_cast<const f32x4*>(L.wlds + (f_w0 ^ ((s & 3) << 4)) + (s >> 2) * 64); };
    // exchange: this lane's 16 bytes (4 classes of one row) inside one slice's block
    const int z_store = (f_row * 16 + 4 * (lane >> 4)) * 4;
    const int z_store_off = ((lane >> 4) < nquad) ? z_store : kOutOfRange;
    const int z_row = tid >> 2, z_qd = tid & 3;             // row / class quad of the softmax phase
    const int z_load_off = (z_qd < nquad) ? (z_row * 16 + 4 * z_qd) * 4 : kOutOfRange;
    const int slice_bytes = a.maxrows * 16 * 4;

    uint32_t n_fenced = 0, n_fast = 0;       // exchanges of each kind so far in this launch
    uint32_t p_acc = 0, p_t0 = 0;            // diagnostics, as in the loader waves
    const bool profiling = PROF && wave == a.prof_wave;
    auto mark = [&](int phase) {
        if constexpr (PROF) {
            if (profiling) {
                if (phase == a.prof_a) p_t0 = (uint32_t)clock64();
                if (phase == a.prof_b) p_acc += (uint32_t)clock64() - p_t0;
            }
        }
    };

    // TEAM: exchange of the members' gradient sums, three buffers used in turn: member q's word of thread tid and class
    // own_cls + vv at (buffer * team + q) * kTeamWords + (vv * 256 + tid) * 4, its bias gradient and loss behind them
    const int team = TEAM ? __builtin_amdgcn_readfirstlane(L.ctl[2]) : 1;
    const __amdgpu_buffer_rsrc_t trsrc = make_rsrc(TEAM ? a.tx + ((int64_t)rep * G + slice) * 3 * a.team * kTeamWords : nullptr,
                                                   TEAM ? (uint32_t)(3 * a.team * kTeamWords * 4) : 0u);
    const int small_word = (lane & 15) == 15 ? 16 : (lane & 15);       // the slot record keeps the loss in word 16
    uint32_t n_team = 0;
    float gbias = 0.0f;      // TEAM: sum of the bias gradients (class 15: loss), class lane % 16

    constexpr int NV = KIND == kLsq ? 1 : 4;      // class rows of a thread that can exist
    float gsum[4 * NV];      // this thread's part of sum_l g_l of the update in progress: gsum[4 vv + c]
    // TEAM: gsum and gbias become the sums over the members, added in their order by everyone.  A word is a sentinel until its
    // member has written it, as in the exchange of the partial logits; a thread talks to the threads of its own number only.
    // (through to memory if the members sit on several XCDs; 0.45 to 0.57 us from store to sight between two XCDs, 0.39 through
    // the L2 of one)
    auto put = [&](u32x4 v, int off) {
        if (a.spread) __builtin_amdgcn_raw_buffer_store_b128(v, trsrc, off, 0, kAgentLoad);
        else __builtin_amdgcn_raw_buffer_store_b128(v, trsrc, off, 0, 0);
    };
    auto put1 = [&](uint32_t v, int off) {
        if (a.spread) __builtin_amdgcn_raw_buffer_store_b32((int)v, trsrc, off, 0, kAgentLoad);
        else __builtin_amdgcn_raw_buffer_store_b32((int)v, trsrc, off, 0, 0);
    };
    auto team_sum = [&]() {
        const int me = myself();
        auto tx_off = [&](int vv) { return 4 * ((me & 63) >> 4) + vv < C ? (vv * NTC + me) * 16 : kOutOfRange; };
        const int tx_bias = me < 16 ? (4 * NTC * 4 + me) * 4 : kOutOfRange;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the re-arming stores of the last exchange have arrived
        const int base = (int)(n_team % 3u) * team;
        const int mine = (base + member) * (kTeamWords * 4);
#pragma unroll
        for (int vv = 0; vv < NV; ++vv) {
            u32x4 ob;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t bits = __float_as_uint(gsum[4 * vv + c]);
                ob[c] = bits == kSentinel ? 0x7FC00000u : bits;
            }
            put(ob, tx_off(vv) + mine);
        }
        const uint32_t bias_bits = __float_as_uint(gbias);
        put1(bias_bits == kSentinel ? 0x7FC00000u : bias_bits, tx_bias + mine);
#pragma unroll
        for (int e = 0; e < 4 * NV; ++e) gsum[e] = 0.0f;
        gbias = 0.0f;
        uint32_t spins = 0;
        // the parts of members q0 .. q0 + N - 1
        auto take = [&](auto n, int q0) {
            constexpr int N = decltype(n)::value;
            u32x4 part[N][NV];
            uint32_t pb[N];
            for (;;) {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int soff = (base + q0 + i) * (kTeamWords * 4);
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv) part[i][vv] = __builtin_amdgcn_raw_buffer_load_b128(trsrc, tx_off(vv), soff, kAgentLoad);
                    pb[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(trsrc, tx_bias, soff, kAgentLoad);
                }
                asm volatile("" ::: "memory");
                uint32_t top = 0u;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    top = max(top, pb[i]);
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv) top = max(max(top, max(part[i][vv].x, part[i][vv].y)), max(part[i][vv].z, part[i][vv].w));
                }
                if (__ballot(top == kSentinel) == 0ull) break;
                __builtin_amdgcn_s_sleep(2);
                ++spins;
                if (spins > a.spin_limit ||
                    ((spins & 63u) == 0 && __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    if (lane == 0) {
                        __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        L.ctl[0] = 1;
                    }
                    break;         // give up: the launch is aborted at the next barrier D
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int vv = 0; vv < NV; ++vv)
#pragma unroll
                    for (int c = 0; c < 4; ++c) gsum[4 * vv + c] += __uint_as_float(part[i][vv][c]);
                gbias += __uint_as_float(pb[i]);
            }
        };
        constexpr int NB = KIND == kLsq ? 8 : (ROOMY ? 4 : 2);     // at most so many at a time
        for (int q0 = 0; q0 < team;) {
            const int left = team - q0;
            if (left >= NB) { take(std::integral_constant<int, NB>{}, q0); q0 += NB; }
            else if (NB > 4 && left >= 4) { take(std::integral_constant<int, 4>{}, q0); q0 += 4; }
            else if (NB > 3 && left == 3) { take(std::integral_constant<int, 3>{}, q0); q0 += 3; }
            else if (NB > 2 && left == 2) { take(std::integral_constant<int, 2>{}, q0); q0 += 2; }
            else { take(std::integral_constant<int, 1>{}, q0); q0 += 1; }
        }
        // everyone has read the exchange before this one: its words of this thread are armed again
        uint32_t sv = kSentinel;
        asm volatile("" : "+v"(sv));
        const u32x4 arm = {sv, sv, sv, sv};
        const int prev = ((int)((n_team + 2u) % 3u) * team + member) * (kTeamWords * 4);
#pragma unroll
        for (int vv = 0; vv < NV; ++vv) put(arm, tx_off(vv) + prev);
        put1(sv, tx_bias + prev);
        ++n_team;
    };
    for (int64_t step = 0; step < a.nsteps; ++step) {
      for (bool last_tile = false; !last_tile;) {           // the tiles of update a.v0 + step
        mark(14);
        lds_barrier();                                      // TU
        mark(0);
        const bool fast = L.ctl[1] != 0;
        const int4 ctl4 = *reinterpret_cast<const int4*>(L.ctl + 4);
        const int2 st01 = *reinterpret_cast<const int2*>(L.s_stale);
        const int2 rec01 = *reinterpret_cast<const int2*>(L.s_rec);     // records 0 and 1, read ahead of their use
        const int Kv = __builtin_amdgcn_readfirstlane(ctl4.x);
        const int n_rec = __builtin_amdgcn_readfirstlane(ctl4.y);
        const int n_stale = __builtin_amdgcn_readfirstlane(ctl4.z);
        const int tile_flags = __builtin_amdgcn_readfirstlane(ctl4.w);
        const int rows = tile_flags >> 8;                   // per record
        last_tile = (tile_flags & 1) != 0;
        const int par = (int)(n_fenced & 1u);               // buffer of a fenced exchange: a step may have several of them
        const bool work = !TEAM || n_rec > 0;               // an empty tile goes through the barriers alone
        // An opaque zero: addresses built from it are recomputed every step instead of being kept in
        // registers across the whole loop (they would be spilled to scratch memory).
        int opq = 0;
        asm volatile("" : "+s"(opq));

        f32x4 own_z = {0.f, 0.f, 0.f, 0.f};       // ONE: logits of row z_row
        // ---- partial logits of rows 16 wave ..: D[class][row] += W[class][k] X[row][k] over this slice;
        //      the operands of the next k-block are read from LDS before the MFMAs of this one are issued
        if (work) {
            f32x4 out;       // classes 4*(lane/16)+0..3 of row f_row
            if constexpr (KIND == kLsq) {
                // One class: on the matrix units fifteen sixteenths of the work would be padding (2350 cycles at 256 columns, one
                // slice; 900 so).  A quarter of the row per lane, the four quarters added across the lanes.
                f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < SL / 16; ++s) {
                    if (ONE && s > 0 && (s & 3) == 0 && s >= 4 * nblk) break;
                    const f32x4 wv = f_wa(s);
                    const f32x4 xv = f_xa(s);
#pragma unroll
                    for (int c = 0; c < 4; ++c) sum[c] = __builtin_fmaf(wv[c], xv[c], sum[c]);
                }
                float z = (sum.x + sum.y) + (sum.z + sum.w);
                z += across<16>(z, lane);
                z += across<32>(z, lane);
                out = f32x4{z, 0.f, 0.f, 0.f};
            } else {
            f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
            f32x4 wv = f_wa(0);
            f32x4 xv = f_xa(0);
#pragma unroll
            for (int s = 0; s < SL / 16; ++s) {
                if (ONE && s > 0 && (s & 3) == 0 && s >= 4 * nblk) break;
                f32x4 wn = wv, xn = xv;
                if (s + 1 < SL / 16) {
                    wn = f_wa(s + 1);
                    xn = f_xa(s + 1);
                }
                __builtin_amdgcn_sched_barrier(0);   // keep the reads ahead of the MFMAs
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.x, xv.x, acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.y, xv.y, acc1, 0, 0, 0);
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.z, xv.z, acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.w, xv.w, acc1, 0, 0, 0);
                wv = wn; xv = xn;
            }
            out = acc0 + acc1;
            }
            mark(8);
            if constexpr (ONE) {
                // thread tid takes class quad tid % 4 of row tid / 4, a row of this wave (one class: every lane of a row has it)
                const int from = KIND == kLsq ? (lane >> 2) * 4 : ((lane & 3) * 16 + (lane >> 2)) * 4;
#pragma unroll
                for (int c = 0; c < (KIND == kLsq ? 1 : 4); ++c)
                    own_z[c] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(out[c])));
            } else
            // 16-byte buffer stores carry their whole offset in the vector register: with the scalar offset in a
            // register, such a store has lost data here when the next instruction rewrote its source registers
            if (fast) {
                // the re-arming stores of the last exchange are in the L2 before this exchange's data can be seen
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                u32x4 ob = __builtin_bit_cast(u32x4, out);
#pragma unroll
                for (int c = 0; c < 4; ++c) ob[c] = (ob[c] == kSentinel) ? 0x7FC00000u : ob[c];   // a NaN that is not the sentinel
                __builtin_amdgcn_raw_buffer_store_b128(ob, ersrc, z_store_off + (int)((n_fast % 3u) * G + slice) * 4096, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out), zrsrc,
                                                       z_store_off + (par * G + slice) * slice_bytes, 0, 0);
            }
        }
        // ---- the part of update v that earlier steps parked: the first two such gradients are fetched
        //      while the exchange stores are on their way
        auto park_load = [&](int slot, f32x4 (&pv)[4]) {
            // classes that do not exist are out of range and read as zero
            const int word = __builtin_amdgcn_readfirstlane(slot);
            const int soff = (word & 0xFFFF) * 16 * nt * 4, me = owner();
            const __amdgpu_buffer_rsrc_t rs = TEAM && BATCH ? park_of(word) : prsrc;
#pragma unroll
            for (int vv = 0; vv < NV; ++vv)
                pv[vv] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, pk_off(me, vv), soff, 0));
        };
        // (TEAM: bias gradient and loss of a parked mini-batch, class lane % 16)
        auto park_bias = [&](int slot) {
            const int word = __builtin_amdgcn_readfirstlane(slot);
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(small_of(word), small_word * 4, (word & 0xFFFF) * 68, 0));
        };
        f32x4 pva[4], pvb[4];
        float ba = 0.0f, bb = 0.0f;
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) { pva[vv] = f32x4{0.f, 0.f, 0.f, 0.f}; pvb[vv] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        if (!chunked && n_stale > 0) park_load(st01.x, pva);
        if (!chunked && n_stale > 1) park_load(st01.y, pvb);
        if constexpr (TEAM && !chunked) {
            if (n_stale > 0) ba = park_bias(st01.x);
            if (n_stale > 1) bb = park_bias(st01.y);
        }
        mark(9);
        // ---- arrival.  Shared-L2 mode needs none: the readers poll the data words themselves.  Otherwise the
        //      wave's stores are released to the device and counted.
        if (!ONE && !fast && work && lane == 0) __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        mark(1);

        // (waited for whether this is the update's first tile or not: where the compiler takes them to be in flight still, it
        // puts a wait for everything in front of the softmax, and that is one for the re-arming store behind the gathers: 1600
        // cycles; K-async at the shape above 6.35 -> 5.48 us per update)
        if constexpr (!chunked && !ONE) {
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) asm volatile("" : "+v"(pva[vv]), "+v"(pvb[vv]));
        }
        if ((tile_flags & 2) != 0) {
#pragma unroll
            for (int e = 0; e < 4 * NV; ++e) gsum[e] = pva[e >> 2][e & 3] + pvb[e >> 2][e & 3];
            if constexpr (TEAM) gbias = ba + bb;
        }
        for (int i = 2; !chunked && i < n_stale; ++i) {     // further parked gradients (K > 2)
            park_load(L.s_stale[i], pva);
#pragma unroll
            for (int e = 0; e < 4 * NV; ++e) gsum[e] += pva[e >> 2][e & 3];
            if constexpr (TEAM) gbias += park_bias(L.s_stale[i]);
        }
        mark(2);

        // ---- wave 0 polls the counter in the L2 (all 4 G compute waves of the cluster have arrived) and
        //      relays the result through an LDS word, which the other waves poll
        if (!ONE && !fast && work) {
            const uint32_t target = (n_fenced + 1u) * (uint32_t)(4 * G);
            const int want = (int)(n_fenced + 1u);
            if (wave == 0) {
                uint32_t spins = 0;
                for (;;) {
                    uint32_t got = __hip_atomic_load(arrive, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("" ::: "memory");   // the load is repeated every turn
                    got = (uint32_t)__builtin_amdgcn_readfirstlane((int)got);
                    if ((int32_t)(got - target) >= 0) break;
                    __builtin_amdgcn_s_sleep(8);
                    ++spins;
                    if (spins > a.spin_limit ||
                        ((spins & 63u) == 0 && __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                        if (lane == 0) {
                            __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            L.ctl[0] = 1;
                        }
                        break;
                    }
                }
                if (lane == 0) __hip_atomic_store(&L.ctl[3], want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&L.ctl[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < want)
                    __builtin_amdgcn_s_sleep(1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            if (!TEAM && a.allow_fast && tid == 0) {
                // first exchange of the launch: do all slices of this cluster share an XCD (one L2)?
                const int32_t* ids = a.xcc_ids + (int64_t)rep * G;
                int same = 1;
                const int mine = __hip_atomic_load(ids + slice, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFF;
                for (int g = 0; g < G; ++g)
                    if ((__hip_atomic_load(ids + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFF) != mine) same = 0;
                L.ctl[2] = same;
            }
            ++n_fenced;
        }
        mark(3);

        // ---- full logits of row z_row (sum of the G partials in slice order), then residual / softmax
        if (work) {
            f32x4 zz = {0.f, 0.f, 0.f, 0.f};
            if constexpr (ONE) {
                zz = own_z;
            } else if (fast) {
                // Poll the partial logits themselves: a batch of slices has arrived for this wave when none of
                // the words its lanes need is the sentinel, i.e. when the largest word read is not all ones.
                // A round re-reads the whole batch; the slices are added in order once it is complete.
                const int xbase = (int)((n_fast % 3u) * G) * 4096;
                uint32_t spins = 0;
                for (int g0 = 0; g0 < G; g0 += 12) {
                    u32x4 part[12];
                    for (;;) {
#pragma unroll
                        for (int i = 0; i < 12; ++i)
                            part[i] = __builtin_amdgcn_raw_buffer_load_b128(ersrc, z_load_off, xbase + min(g0 + i, G - 1) * 4096, kAgentLoad);
                        asm volatile("" ::: "memory");   // the loads are repeated every round
                        uint32_t top = 0u;
#pragma unroll
                        for (int i = 0; i < 12; ++i) top = max(max(top, max(part[i].x, part[i].y)), max(part[i].z, part[i].w));
                        if (__ballot(top == kSentinel) == 0ull) break;
                        // with another workgroup on this CU, re-reading at once would slow its memory operations
                        if (a.shared_cus) __builtin_amdgcn_s_sleep(32); else __builtin_amdgcn_s_sleep(2);
                        ++spins;
                        if (spins > a.spin_limit ||
                            ((spins & 63u) == 0 && __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                            if (lane == 0) {
                                __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                L.ctl[0] = 1;
                            }
                            break;         // give up: the launch is aborted at the next barrier
                        }
                    }
                    if (g0 + 12 <= G) {
#pragma unroll
                        for (int i = 0; i < 12; ++i) zz += __builtin_bit_cast(f32x4, part[i]);
                    } else {
                        // the last, partial batch re-read its final slice in the unused places
#pragma unroll
                        for (int i = 0; i < 12; ++i)
                            if (g0 + i < G) zz += __builtin_bit_cast(f32x4, part[i]);
                    }
                }
                // Every slice of this exchange has been written, so every workgroup has finished reading the one
                // before it: this wave's rows of that buffer are re-armed for their next use.
                uint32_t sv = kSentinel;
                asm volatile("" : "+v"(sv));      // built here, not kept in registers across the loop
                const u32x4 arm = {sv, sv, sv, sv};
                __builtin_amdgcn_raw_buffer_store_b128(arm, ersrc, z_store_off + (int)(((n_fast + 2u) % 3u) * G + slice) * 4096, 0, 0);
                ++n_fast;
            } else {
                const int zbase = par * G * slice_bytes;
                for (int g0 = 0; g0 < G; g0 += 12) {
                    // straight-line batch: slices past the end re-read the last one and are not added
                    f32x4 part[12];
#pragma unroll
                    for (int i = 0; i < 12; ++i)
                        part[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                            zrsrc, z_load_off, zbase + min(g0 + i, G - 1) * slice_bytes, kAgentLoad));
#pragma unroll
                    for (int i = 0; i < 12; ++i) {
                        const float keep = (g0 + i < G) ? 1.0f : 0.0f;
                        zz += part[i] * keep;
                    }
                }
            }
            mark(4);
            const bool ok = L.rowid[z_row] != kNoRow;
            f32x4 dl = {0.f, 0.f, 0.f, 0.f};
            float loss = 0.0f;
            if constexpr (KIND == kLsq) {
                const float z0 = quad_lane0(zz.x);
                const float r = z0 - L.ylab[z_row];
                if (ok) loss = 0.5f * r * r;
                if (z_qd == 0 && ok) dl.x = r * inv_m;
            } else {
                const int lab = __float_as_int(L.ylab[z_row]);
                float zmax = -3.0e38f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    zz[e] += L.bias[4 * z_qd + e];
                    if (4 * z_qd + e < C) zmax = fmaxf(zmax, zz[e]);
                }
                zmax = fmaxf(zmax, quad_xor1(zmax));
                zmax = fmaxf(zmax, quad_xor2(zmax));
                float den = 0.0f, lt_ = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ex = (4 * z_qd + e < C) ? expf(zz[e] - zmax) : 0.0f;
                    den += ex;
                    if (4 * z_qd + e == lab) lt_ = -(zz[e] - zmax);
                    dl[e] = ex;
                }
                den += quad_xor1(den);
                den += quad_xor2(den);
                lt_ += quad_xor1(lt_);
                lt_ += quad_xor2(lt_);
                loss = ok ? lt_ + logf(den) : 0.0f;
                const float inv = 1.0f / den;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float pr = dl[e] * inv - ((4 * z_qd + e == lab) ? 1.0f : 0.0f);
                    dl[e] = (ok && 4 * z_qd + e < C) ? pr * inv_m : 0.0f;
                }
            }
            // the unused class 15 carries the row loss: the column sums of the delta tile (taken by a
            // loader wave) then hold the bias gradient and the loss sum
            if (z_qd == 3) dl.w = loss * inv_m;
            *reinterpret_cast<f32x4*>(L.zbuf + z_row * 16 + 4 * z_qd) = dl;
        }
        mark(13);
        lds_barrier();                                      // D
        if (L.ctl[0] != 0) return;   // uniform: every thread reads the same LDS word
        mark(5);

        // ---- per record: the gradient slice delta^T X, in k-steps of four rows
        {
            const bool has_cols = !ONE || wave < nblk;      // a wave without columns contracts nothing
            const int n_own = has_cols ? n_rec : 0;
            f32x4 acc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            // record r is complete: add it to the aggregate of update v, or park it in its slot
            float bsum = 0.0f;      // TEAM: column sums of delta, class lane % 16, rows lane / 16 modulo 4
            auto whole_bias = [&]() {
                bsum += across<16>(bsum, lane);
                bsum += across<32>(bsum, lane);
                return bsum;
            };
            auto finish = [&](int rec_word) {         // its entry in the compute list
                const int me = owner();
                if constexpr (PROF) { asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])); mark(11); }
                const int word = __builtin_amdgcn_readfirstlane(rec_word);
                bool to_sum = ((word >> 16) & 1) != 0;
                if constexpr (BATCH) {
                    // A record of several tiles is summed in its worker's slot (free by now: what it held was consumed
                    // by an earlier update or with the first tile of this one): later blocks add what is there, and
                    // only the last one goes to the aggregate if the update consumes the record itself.
                    if (((word >> 18) & 1) != 0) {
                        const int from = TEAM ? scratch : word;
                        const int soff = (from & 0xFFFF) * 16 * nt * 4;
                        const __amdgpu_buffer_rsrc_t rs = TEAM ? park_of(from) : prsrc;
#pragma unroll
                        for (int vv = 0; vv < NV; ++vv) {
                            const f32x4 pv = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, pk_off(me, vv), soff, 0));
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[c][vv] += pv[c];
                        }
                    }
                    if (((word >> 17) & 1) != 0) to_sum = false;
                }
                const int dest = TEAM && ((word >> 17) & 1) != 0 ? scratch : word;
                if constexpr (TEAM) {
                    float b = whole_bias();
                    const int off = tid < 16 ? small_word * 4 : kOutOfRange;
                    if (((word >> 18) & 1) != 0)
                        b += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(small_of(scratch), off, (scratch & 0xFFFF) * 68, 0));
                    if (to_sum) gbias += b;
                    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, b), small_of(dest), off + (dest & 0xFFFF) * 68, 0, 0);
                    bsum = 0.0f;
                }
                if (to_sum) {
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv)
#pragma unroll
                        for (int c = 0; c < 4; ++c) gsum[vv * 4 + c] += acc[c][vv];
                } else {
                    const int soff = (dest & 0xFFFF) * 16 * nt * 4;
                    const __amdgpu_buffer_rsrc_t rs = TEAM && BATCH ? park_of(dest) : prsrc;
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv) {
                        const f32x4 gv = {acc[0][vv], acc[1][vv], acc[2][vv], acc[3][vv]};
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, gv), rs, pk_off(me, vv) + soff, 0, 0);
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
                mark(12);
            };
            const int ome = myself(), olo = (ome & 63) >> 4, ocl = ome & 15, och = 16 * wave + ocl;
            const float* bz = L.zbuf + olo * 16 + ocl;
            if constexpr (KIND == kLsq) {
                // One class: a lane adds up its four columns over every fourth row, the four lanes of a column are added at the
                // end of a record (two records of 16 rows, 256 columns, one slice: 3500 cycles on the matrix units, 2400 so).
                const float* dz = L.zbuf + olo * 16;
                const float* xr = L.tile + olo * SL;
                const int key = och ^ olo, kpr = rows >> 2;
                int k = opq;
#pragma unroll 1
                for (int r = 0; r < n_own; ++r) {
                    const int rec_word = L.s_rec[r];      // read ahead of its use
                    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
                    auto add = [&](auto n, int k0) {
                        constexpr int N = decltype(n)::value;
                        float dv[N], lv[N];
                        f32x4 xv[N];
#pragma unroll
                        for (int u = 0; u < N; ++u) {
                            dv[u] = dz[(k0 + u) * 64];
                            if constexpr (TEAM) lv[u] = dz[(k0 + u) * 64 + ocl];
                            xv[u] = *reinterpret_cast<const f32x4*>(xr + (k0 + u) * 4 * SL + ((key ^ (4 * ((k0 + u) & 3))) << 2));
                        }
#pragma unroll
                        for (int u = 0; u < N; ++u) {
                            if constexpr (TEAM) bsum += lv[u];
#pragma unroll
                            for (int c = 0; c < 4; ++c) sum[c] = __builtin_fmaf(dv[u], xv[u][c], sum[c]);
                        }
                    };
                    const int end = k + kpr;
#pragma unroll 1
                    for (; k + 8 <= end; k += 8) add(std::integral_constant<int, 8>{}, k);
                    if (k + 4 <= end) { add(std::integral_constant<int, 4>{}, k); k += 4; }
#pragma unroll 1
                    for (; k < end; ++k) add(std::integral_constant<int, 1>{}, k);
                    // (two columns at a time: after the swaps of halves and of rows each row of lanes has one column's sum; the
                    // owners are the first row's lanes)
                    auto halves = [](float& x, float& y) {
                        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
                        x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
                    };
                    auto rows16 = [](float& x, float& y) {
                        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
                        x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
                    };
                    float s0 = sum.x, s1 = sum.y, s2 = sum.z, s3 = sum.w;
                    halves(s0, s1);
                    halves(s2, s3);
                    float lo = s0 + s1, hi = s2 + s3;                  // columns 0 | 1 and 2 | 3 in the two halves
                    rows16(lo, hi);
                    float t0 = lo + hi;                                // rows of lanes: columns 0, 2, 1, 3
                    float t1 = t0;
                    rows16(t0, t1);                                    // t1: columns 2 and 3 in the first row and the third
                    acc[0][0] = t0;
                    float u0 = t0, u1 = t1, v0 = t0, v1 = t1;
                    halves(u0, v0);                                    // v0: the third row's column 1
                    halves(u1, v1);                                    // v1: its column 3
                    acc[1][0] = v0; acc[2][0] = t1; acc[3][0] = v1;
                    finish(rec_word);
                }
            } else if constexpr (WHOLE) {
                // Whole groups of 16 rows only, at most four of them: two register sets take turns, one being read from LDS while the MFMAs of the other are issued.
                // half-group h: k-steps 2 h and 2 h + 1, i.e. rows 8 h .. 8 h + 7
                const float* bx[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) bx[u] = L.tile + (4 * u + olo) * SL + ((och ^ (4 * u + olo)) << 2);
                auto fetch = [&](int h, float (&dv)[2], f32x4 (&xv)[2]) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        dv[u] = bz[(8 * h + 4 * u) * 16];
                        xv[u] = *reinterpret_cast<const f32x4*>(bx[2 * (h & 1) + u] + 16 * (h >> 1) * SL);
                    }
                };
                auto mac = [&](bool first, const float (&dv)[2], const f32x4 (&xv)[2]) {
                    if constexpr (TEAM) bsum = (first ? 0.0f : bsum) + (dv[0] + dv[1]);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const f32x4 init = (first && u == 0) ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[c];
                            acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[u], xv[u][c], init, 0, 0, 0);
                        }
                    }
                };
                auto done = [&](int r) {
                    const int me = owner();
                    if constexpr (PROF) { asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])); mark(11); }
                    const int word = __builtin_amdgcn_readfirstlane(r == 0 ? rec01.x : rec01.y);
                    if constexpr (TEAM) {
                        const float b = whole_bias();
                        const int off = tid < 16 ? small_word * 4 : kOutOfRange;
                        if (((word >> 16) & 1) != 0) gbias += b;
                        else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, b), small_of(word), off + (word & 0xFFFF) * 68, 0, 0);
                    }
                    if (((word >> 16) & 1) != 0) {
#pragma unroll
                        for (int vv = 0; vv < NV; ++vv)
#pragma unroll
                            for (int c = 0; c < 4; ++c) gsum[vv * 4 + c] += acc[c][vv];
                    } else {
                        const int soff = (word & 0xFFFF) * 16 * nt * 4;
                        const __amdgpu_buffer_rsrc_t rs = TEAM && BATCH ? park_of(word) : prsrc;
#pragma unroll
                        for (int vv = 0; vv < NV; ++vv) {
                            const f32x4 gv = {acc[0][vv], acc[1][vv], acc[2][vv], acc[3][vv]};
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, gv), rs, pk_off(me, vv) + soff, 0, 0);
                        }
                    }
                    mark(12);
                };
                float da[2], db[2];
                f32x4 xa[2], xb[2];
                const int H = n_own * (rows >> 3);         // half-groups in the tile: 0, 4 or 8
                if (H > 0) {
                    fetch(0, da, xa);
                    fetch(1, db, xb);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(true, da, xa);
                    fetch(2, da, xa);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(false, db, xb);
                    fetch(3, db, xb);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(false, da, xa);
                    if (H > 4) fetch(4, da, xa);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(false, db, xb);
                    if (H > 4) {
                        const bool two = rows == 32;         // the second record starts with half-group 4
                        if (two) done(0);
                        fetch(5, db, xb);
                        __builtin_amdgcn_sched_barrier(0);
                        if (two) mac(true, da, xa); else mac(false, da, xa);
                        fetch(6, da, xa);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(false, db, xb);
                        fetch(7, db, xb);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(false, da, xa);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(false, db, xb);
                        done(two ? 1 : 0);
                    } else {
                        done(0);
                    }
                }
            } else if constexpr (!BATCH) {
                // Records of any multiple of four rows, one behind the other, 16 rows a turn: a record ends where its rows do.
                // Four register sets, each read again for the next turn as soon as its MFMAs are issued.
                const int kpr = rows >> 2, steps = n_own * kpr;
                const float* bx[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) bx[u] = L.tile + (4 * u + olo) * SL + ((och ^ (4 * u + olo)) << 2);
                float dv[4];
                f32x4 xv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { dv[u] = bz[4 * u * 16]; xv[u] = *reinterpret_cast<const f32x4*>(bx[u]); }
                int r = opq, end = kpr;
                for (int g0 = 0; g0 < steps; g0 += 4) {
                    const int nx = min(g0 + 4, ROWS / 4 - 4);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (g0 + u < steps) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[u], xv[u][c], acc[c], 0, 0, 0);
                            if (g0 + u + 1 == end) { finish(r == 0 ? rec01.x : (r == 1 ? rec01.y : L.s_rec[r])); ++r; end += kpr; }
                        }
                        dv[u] = bz[4 * (nx + u) * 16];
                        xv[u] = *reinterpret_cast<const f32x4*>(bx[u] + 4 * nx * SL);
                    }
                }
            } else {
                // The same where records are described one by one and their ends are more code: two register sets take turns,
                // one being read from LDS while the MFMAs of the other are issued, and the loops are kept rolled.  (Unrolled over
                // the sixteen k-steps that a tile can have, with the end of a record behind each, they are 25 KB of code:
                // softmax, P = 20, K = 5, m = 25, d = 785, 8 replicas 4 % more per update.  Without that code the unrolled loop is the
                // better one: P = 11, K = 5, m = 12, d = 2420, one replica 7.4 us, 7.6 rolled.)
                const int kpr = rows >> 2, last = n_own * kpr - 1;
                const float* xr = L.tile + olo * SL;
                const int key = och ^ olo;
                auto fetch = [&](int k, float& dv, f32x4& xv) {
                    dv = bz[64 * k];
                    xv = *reinterpret_cast<const f32x4*>(xr + 4 * k * SL + ((key ^ (4 * (k & 3))) << 2));
                };
                auto mac = [&](float dv, const f32x4& xv) {
                    if constexpr (TEAM) bsum += dv;
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, xv[c], acc[c], 0, 0, 0);
                };
                float da, db;
                f32x4 xa, xb;
                int k = opq;
                fetch(0, da, xa);
#pragma unroll 1
                for (int r = 0; r < n_own; ++r) {
                    const int rec_word = L.s_rec[r];      // read ahead of its use
                    const int end = k + kpr;
#pragma unroll 1
                    for (; k + 2 <= end; k += 2) {
                        fetch(k + 1, db, xb);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(da, xa);
                        fetch(min(k + 2, last), da, xa);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(db, xb);
                    }
                    if (k < end) {
                        fetch(min(k + 1, last), db, xb);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(da, xa);
                        da = db; xa = xb;
                        ++k;
                    }
                    finish(rec_word);
                }
            }
        }
        mark(6);
        lds_barrier();                                      // B: the loader waves may rewrite the tile and the lists
        // ---- update v: each compute thread owns its weights; nobody reads them before TU
        if constexpr (TEAM) {
            if (last_tile && team > 1) team_sum();
        }
        if (last_tile) {
            const float scale = a.lr / (float)Kv;
            const int me = myself(), och = 16 * wave + (me & 15), ocl = 4 * ((me & 63) >> 4);
#pragma unroll
            for (int vv = 0; vv < NV; ++vv) {
                const int cls = ocl + vv;
                if (cls < C) {
                    f32x4* wp = reinterpret_cast<f32x4*>(L.wlds + cls * SL + ((och ^ cls) << 2));
                    f32x4 w = *wp;
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[c] -= scale * gsum[vv * 4 + c];
                    *wp = w;
                }
            }
            if constexpr (TEAM) {
                if (tid < 16) {
                    if (KIND == kSoftmax && tid < C) L.bias[tid] -= scale * gbias;
                    if (tid == 15 && slice == 0 && member == 0) a.tr.loss[(int64_t)rep * cap + a.v0 + step] = gbias * (1.0f / (float)Kv);
                    if (KIND == kSoftmax && a.agg_out != nullptr && rep == 0 && slice == 0 && member == 0 && tid < C)
                        a.agg_out[(int64_t)C * d + tid] = gbias * (1.0f / (float)Kv);
                }
            }
            if (a.agg_out != nullptr && rep == 0 && member == 0) {
                // the averaged gradient of replica 0, when the caller asked for it
                const float invK = 1.0f / (float)Kv;
#pragma unroll
                for (int vv = 0; vv < NV; ++vv) {
                    const int cls = own_cls + vv;
                    if (cls < C)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (own_col + c < d) a.agg_out[(int64_t)cls * d + own_col + c] = gsum[vv * 4 + c] * invK;
                }
            }
        }
        if (!TEAM && tid == 0 && L.ctl[2] != 0) L.ctl[1] = 1;   // later exchanges of this launch use the shared L2
        mark(7);
      }
    }
    if constexpr (PROF) {
        if (profiling && lane == 0 && member == 0) a.prof[(int64_t)a.prof_base + ((int64_t)rep * G + slice) * 2] += p_acc;
    }
    lds_barrier();

    // ---- leave the state in HBM for the next launch
    if constexpr (TEAM && BATCH) {
        // (Written through: a line may hold bias gradients of several members.  Four gradients at a time: one after the other, a trip to
        // memory each, they made short calls longer than without a team.  Softmax, K-batch-async, P = 30, K = 7, m = 14, d = 40,
        // 5 replicas, calls of one, two and five updates 49, 67, 117 -> 44, 59, 102 us, without a team 46, 59, 99; eight at a time 45, 59, 104.)
        constexpr int AT_ONCE = 4;
        for (int q0 = 0; a.own_slots > 0 && q0 < S; q0 += 64) {
            unsigned long long left = __ballot(q0 + lane < S && L.own[min(q0 + lane, S - 1)] != 0);
            while (left != 0) {
                u32x4 g[AT_ONCE][NV];
                int b[AT_ONCE], slot[AT_ONCE], none[AT_ONCE];
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) {
                    slot[i] = left != 0 ? q0 + __builtin_ctzll(left) : 0;
                    none[i] = left != 0 ? 0 : kOutOfRange;
                    left &= left - 1;
                }
                const int off = tid < 16 ? small_word * 4 : kOutOfRange;
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) {
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv)
                        g[i][vv] = __builtin_amdgcn_raw_buffer_load_b128(park_of(kOwnSlot), pk_off(tid, vv) | none[i], slot[i] * 16 * nt * 4, 0);
                    b[i] = __builtin_amdgcn_raw_buffer_load_b32(small_of(kOwnSlot), off | none[i], slot[i] * 68, 0);
                }
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) {
#pragma unroll
                    for (int vv = 0; vv < NV; ++vv)
                        __builtin_amdgcn_raw_buffer_store_b128(g[i][vv], prsrc, (pk_off(tid, vv) | none[i]) + slot[i] * 16 * nt * 4, 0, kAgentLoad);
                    __builtin_amdgcn_raw_buffer_store_b32(b[i], small_of(0), (off | none[i]) + slot[i] * 68, 0, kAgentLoad);
                }
            }
        }
    }
    if (TEAM && member > 0) return;
#pragma unroll
    for (int vv = 0; vv < 4; ++vv) {
        const int cls = own_cls + vv;
        if (cls < C) {
            const f32x4 w = *reinterpret_cast<const f32x4*>(L.wlds + cls * SL + ((own_ch ^ cls) << 2));
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (own_col + c < d) params[(int64_t)cls * d + own_col + c] = w[c];
        }
    }
    if (KIND == kSoftmax && slice == 0 && tid < C) params[(int64_t)C * d + tid] = L.bias[tid];
    if constexpr (!TEAM)
        for (int q = tid; q < S * 17; q += NTC) small_g[q] = L.small[q];
}

template <int KIND, bool PROF, bool WHOLE, bool CHUNKED, bool BATCH, bool ONE, bool ROOMY, bool LATE, bool TEAM = false>
hipError_t launch_r(const LinArgs& a, size_t lds, hipStream_t s) {
    constexpr auto kernel = linear_tile_kernel<KIND, PROF, WHOLE, CHUNKED, BATCH, ONE, ROOMY, LATE, TEAM>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int groups = (a.replicas + 7) / 8;
    const int blocks = TEAM ? (a.spread ? (a.replicas * a.team + 7) / 8 : groups * a.team) * 8 * a.G : (a.pair_cus > 0 ? 8 * a.pair_cus * a.pair_layers : groups * 8 * a.G);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(512), lds, s, a);
    return hipGetLastError();
}

template <int KIND, bool PROF, bool WHOLE, bool CHUNKED, bool BATCH>
hipError_t launch_w(const LinArgs& a, size_t lds, hipStream_t s) {
    if constexpr (CHUNKED || BATCH)
        if (a.team > 1) {
            if (a.G == 1) return a.whole_cus ? launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, true, true, true, true>(a, lds, s)
                                             : launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, true, false, true, true>(a, lds, s);
            return a.whole_cus ? launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, false, true, true, true>(a, lds, s)
                               : launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, false, false, true, true>(a, lds, s);
        }
    if (a.G == 1) return a.shared_cus ? launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, true, false, !CHUNKED>(a, lds, s)
                                      : launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, true, true, !CHUNKED>(a, lds, s);
    if (a.whole_cus) return launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, false, true, true>(a, lds, s);
    if constexpr (CHUNKED)
        if (a.shared_cus) return launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, false, false, false>(a, lds, s);
    return launch_r<KIND, PROF, WHOLE, CHUNKED, BATCH, false, false, true>(a, lds, s);
}

// K-async whose versions may have more records than a tile holds; version 0, at which all P workers start, is one.
bool records_one_by_one(const LinArgs& a) { return a.variant == kBatchAsync || (a.variant == kAsync && (a.v0 < 1 || a.mp * a.tr.Kcap > ROWS)); }

// WHOLE: every record is a whole number of 32-row blocks, so the gradient contraction is fully unrolled;
// CHUNKED: a synchronous variant, one record per tile; BATCH: records described one by one; neither: K-async, one tile
template <int KIND, bool PROF>
hipError_t launch_k(const LinArgs& a, size_t lds, hipStream_t s) {
    if (a.chunked) return launch_w<KIND, PROF, true, true, false>(a, lds, s);
    const bool whole = a.mp == 32 || a.mp == 64;
    if (records_one_by_one(a)) return whole ? launch_w<KIND, PROF, true, false, true>(a, lds, s) : launch_w<KIND, PROF, false, false, true>(a, lds, s);
    return whole ? launch_w<KIND, PROF, true, false, false>(a, lds, s) : launch_w<KIND, PROF, false, false, false>(a, lds, s);
}

}  // namespace

#ifdef SSGD_TILE_LSQ
hipError_t launch_linear_tile_lsq(const LinArgs& a, hipStream_t s) {
    const size_t lds = linear_tile_lds_bytes(a.C, a.S, a.tr.Kcap, a.team > 1);
    return a.prof != nullptr ? launch_k<kLsq, true>(a, lds, s) : launch_k<kLsq, false>(a, lds, s);
}
#else
size_t linear_tile_lds_bytes(int C, int S, int Kcap, bool team) {
    const size_t words = (size_t)ROWS * SL + (size_t)C * SL + ROWS * 16 + 2 * ROWS + 16 + 8 + 2 * (Kcap > 32 ? 64 : 32) + (team ? ((size_t)S + 3) / 4 : (size_t)S * 17);
    return sizeof(float) * words;
}

bool linear_tile_supports(const LinArgs& a, int max_records) {
    // the consume list and the restarts of an update sit in one lane each; the last chunk of a row is read as its last four columns
    if (a.C > 15 || a.d < 4 || a.tr.Kcap > KC || max_records > KC) return false;
    const bool synchronous = a.variant == kSync || a.variant == kBatchSync;
    if (synchronous != (a.chunked != 0)) return false;
    if (!one_descriptor_spans(a.N, (uint64_t)a.d)) return false;
    return linear_tile_lds_bytes(a.C, a.S, a.tr.Kcap, false) <= 160 * 1024;
}

int linear_tile_resident_groups(size_t lds_bytes) {
    int dev = 0, per_cu = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(linear_tile_kernel<kSoftmax, false, false, false, false, false, false, true, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, linear_tile_kernel<kSoftmax, false, false, false, false, false, false, true, false>, 512, lds_bytes) != hipSuccess) return 0;
    return per_cu * cus;
}

hipError_t launch_linear_tile(const LinArgs& a, hipStream_t s) {
    const size_t lds = linear_tile_lds_bytes(a.C, a.S, a.tr.Kcap, a.team > 1);
    if (a.kind == kLsq) return launch_linear_tile_lsq(a, s);
    return a.prof != nullptr ? launch_k<kSoftmax, true>(a, lds, s) : launch_k<kSoftmax, false>(a, lds, s);
}
#endif

}  // namespace ssgd
