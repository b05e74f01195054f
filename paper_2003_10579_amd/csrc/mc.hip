// Monte-Carlo estimate of the runtime per iteration T (Sec. 2.3; Lemma 1: K-sync
// T = X_{K:P}; Lemma 2: K-batch-sync; Lemma 3: K-async; the simulation of Fig. 6).
//
// One wavefront owns a trial and a share of the values of K.  For every K it runs the variant's event process for
// chain_len updates, the P finish times in registers (fp64, NQ per lane).  Bound: plain ALU issue; what it is spent on
// and how each part is kept small:
//   * Drawing delays (counter-based generator and logarithm, about 280 SIMD cycles for 64 of them).  Which delays a
//     chain needs does not depend on its outcome, so they are drawn densely, 64 at a time, into a window in LDS and
//     taken from there (drawing the K restarts of an update in place leaves 64 - K lanes idle).
//   * Selecting.  An update needs the K-th smallest finish time and the set of the K earliest, not their order: the
//     process only depends on the multiset of finish times, so any one-to-one assignment of the K fresh delays to the K
//     restarting workers gives the same chain, bit for bit.  select_kth narrows a set of candidates held as lane masks
//     in scalar registers: two cuts around a guess (the previous T), then pivots, a ballot each; about five rounds at
//     P = 128 where sorting took 28 exchanges of both registers.
//   * K-batch-async: the renewals of all workers up to a bound are listed unsorted in LDS, lane by lane in parallel, and
//     a list is sorted in registers (the push sequence is the same for every K); one argmin per push is kept for lists
//     that do not fit.
// 10^5 trials, P = 128, all K, chains of 8 (K-async, Exp(1)): 35.6 ms a call, 110 ms with sorted arrays and restarts
// drawn in place (15 of them host additions of the blocks' sums); 169 vector instructions per update, issued 85 % of the
// time; K-batch-async, P = 64, K = 32, chains of 8: 0.4 ms, 6 with an argmin and a draw per push.
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "../../include/ssgd.h"
#include "common.hpp"

namespace ssgd {
namespace {

constexpr int kWindow = 512;      // delays drawn ahead per wavefront (fp32, LDS)
constexpr int kFew = 32;          // candidates that are ranked against each other instead of narrowed further
constexpr int kList = 512;        // K-batch-async: renewals listed before they are sorted (fp64, LDS)

struct McArgs {
    Dist dist;
    uint64_t seed;
    int32_t variant, P, Kmin, Kmax, chain_len;
    int32_t nslices;     // block b takes the values K = Kmin + b % nslices, + nslices, ...: small accumulators, many waves per CU
    int64_t trial0, trials;
    double mean_delay;   // a rough value: first guess of a selection, size of the K-batch-async lists
    double* partial;     // [blocks][nK*chain_len][2]
    double* per_trial;   // nullable
    int32_t one_by_one;  // K-batch-async: delays may be below zero, so that a push can be earlier than the one before it
};

typedef unsigned long long u64;

__device__ __forceinline__ double inf64() { return __longlong_as_double(0x7FF0000000000000LL); }

// Orders the LDS accesses of one wavefront (its lanes read what other lanes of it wrote).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int rank_in(u64 mask) {      // set bits below this lane
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const u64 b = (u64)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), lane));
}

// ---- exchanges between lanes without LDS: data-parallel-primitive moves inside a row of 16, swaps across rows
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false); }

// value of lane ^ MASK, for the masks the sorting network uses: 1, 2, 4, 8, 16, 32 and 3, 7, 15, 31, 63
template <int MASK>
__device__ __forceinline__ uint32_t exchange(uint32_t v, int lane) {
    constexpr int in_row = MASK & 15;
    if constexpr (in_row == 1) v = dpp<0xB1>(v);            // quad_perm [1,0,3,2]
    if constexpr (in_row == 2) v = dpp<0x4E>(v);            // quad_perm [2,3,0,1]
    if constexpr (in_row == 3) v = dpp<0x1B>(v);            // quad_perm [3,2,1,0]
    if constexpr (in_row == 4) v = dpp<0x141>(dpp<0x1B>(v));
    if constexpr (in_row == 7) v = dpp<0x141>(v);           // row_half_mirror
    if constexpr (in_row == 8) v = dpp<0x128>(v);           // row_ror:8
    if constexpr (in_row == 15) v = dpp<0x140>(v);          // row_mirror
    if constexpr ((MASK & 16) != 0) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);    // even rows twice, odd rows twice
        v = (lane & 16) ? r[0] : r[1];
    }
    if constexpr ((MASK & 32) != 0) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = (lane & 32) ? r[0] : r[1];
    }
    return v;
}
template <int MASK>
__device__ __forceinline__ float exchange(float v, int lane) { return __uint_as_float(exchange<MASK>(__float_as_uint(v), lane)); }
template <int MASK>
__device__ __forceinline__ double exchange(double v, int lane) {
    const u64 b = (u64)__double_as_longlong(v);
    const u64 lo = exchange<MASK>((uint32_t)b, lane), hi = exchange<MASK>((uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)((hi << 32) | lo));
}

__device__ __forceinline__ double lesser(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double greater(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ float lesser(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float greater(float a, float b) { return __builtin_fmaxf(a, b); }

// One compare-exchange step of all positions p = lane * NQ + q with p ^ (D * NQ) or, MIRROR, with the position that
// mirrors it in a block of 2 D lanes.
template <int NQ, int D, bool MIRROR, typename T>
__device__ __forceinline__ void lane_step(T (&key)[NQ], int lane) {
    constexpr int MASK = MIRROR ? 2 * D - 1 : D;
    T other[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) other[q] = exchange<MASK>(key[MIRROR ? NQ - 1 - q : q], lane);
    const bool low = (lane & D) == 0;
    // Compared and selected: fmin and fmax cost another instruction for every operand that the compiler does not know to be
    // no signalling NaN, and a flag that says so for the whole file takes the NaN checks out of host code (10^5 trials at
    // P = 64, K = 32: 431 us, 516 with fmin and fmax, 459 with fmin, fmax and the flag; all K up to 64: 3.51, 4.23, 3.39 ms).
#pragma unroll
    for (int q = 0; q < NQ; ++q) key[q] = (key[q] < other[q]) == low ? key[q] : other[q];
}
template <int NQ, int K, typename T>
__device__ __forceinline__ void register_merge(T (&key)[NQ]) {       // xor steps K/2 .. 1 inside a lane
#pragma unroll
    for (int j = K / 2; j > 0; j >>= 1)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if ((q & j) == 0) { const T a = key[q], b = key[q | j]; key[q] = lesser(a, b); key[q | j] = greater(a, b); }
}
template <int NQ, int D, typename T>
__device__ __forceinline__ void lane_merge(T (&key)[NQ], int lane) { // xor steps D .. 1 lanes, then inside a lane
    if constexpr (D >= 1) { lane_step<NQ, D, false>(key, lane); lane_merge<NQ, D / 2>(key, lane); }
    else register_merge<NQ, NQ>(key);
}
// Ascending sort of 64 NQ keys, position p = lane * NQ + q: every block is merged with its mirror image, so that all
// steps order upwards and steps shorter than NQ stay inside a lane.
template <int NQ, int K = 2, typename T>
__device__ __forceinline__ void sort_keys(T (&key)[NQ], int lane) {
    if constexpr (K <= NQ) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int m = q ^ (K - 1);
            if (q < m) { const T a = key[q], b = key[m]; key[q] = lesser(a, b); key[m] = greater(a, b); }
        }
        register_merge<NQ, K / 2>(key);
        sort_keys<NQ, 2 * K>(key, lane);
    } else if constexpr (K <= 64 * NQ) {
        constexpr int D = K / (2 * NQ);
        lane_step<NQ, D, true>(key, lane);
        if constexpr (D > 1) lane_merge<NQ, D / 2>(key, lane); else register_merge<NQ, NQ>(key);
        sort_keys<NQ, 2 * K>(key, lane);
    }
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v, int lane) {
    v = min(v, exchange<1>(v, lane));
    v = min(v, exchange<2>(v, lane));
    v = min(v, exchange<7>(v, lane));
    v = min(v, exchange<15>(v, lane));
    v = min(v, exchange<16>(v, lane));
    v = min(v, exchange<32>(v, lane));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
// Smallest of the lanes' values: the high words decide as integers (in the order of the numbers: the sign bit turned over,
// all bits of a negative one), the low words only where several lanes have the same high word.  (An exchange and a
// minimum of 32 bits per step instead of 64, and no instruction against signalling NaN: K-batch-sync, P = 64, all K, chains of
// 4, 20000 trials: 11.6 ms, 14.9 with fmin, 13.2 with fmin and the flag named at lane_step.)
__device__ __forceinline__ double wave_min(double v, int lane) {
    const u64 b = (u64)__double_as_longlong(v);
    const uint32_t turn = (uint32_t)((int32_t)(b >> 32) >> 31);              // all ones below zero
    const uint32_t hi = (uint32_t)(b >> 32) ^ (turn | 0x80000000u);
    const uint32_t top = wave_min(hi, lane);
    const u64 m = __ballot(hi == top);
    if ((m & (m - 1)) == 0) return lane_value(v, __builtin_ctzll(m));
    const uint32_t lo = hi == top ? (uint32_t)b ^ turn : 0xFFFFFFFFu;
    const uint32_t low = wave_min(lo, lane);
    return lane_value(v, __builtin_ctzll(m & __ballot(lo == low)));
}

template <int NQ>
__device__ __forceinline__ int count(const u64 (&m)[NQ]) {
    int c = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) c += __popcll(m[q]);
    return c;
}

__device__ __forceinline__ bool in_mask(u64 mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }
template <typename T> __device__ __forceinline__ T unbounded();
template <> __device__ __forceinline__ double unbounded<double>() { return inf64(); }
template <> __device__ __forceinline__ float unbounded<float>() { return __uint_as_float(0x7F800000u); }

// The K-th smallest key (K from 1, wave-uniform) of all 64 NQ.  [lo, hi): where it is expected, extended by w, 2 w, 4 w ...
// until it holds the key wanted (w > 0); few: kFew keys of LDS.  The mask arithmetic is scalar work, which a CU issues
// once per cycle for all its waves, so it ends as soon as at most kFew candidates are left; those go to LDS and each is
// counted against all.  (With pivots to the end an update took 198 scalar and 165 vector instructions at P = 128, and the
// scalar unit was what the kernel waited for.)  Every comparison is exact, so the result does not depend on the guess.
template <int NQ, typename T>
__device__ __forceinline__ T select_kth(const T (&key)[NQ], int K, T lo, T hi, T w, T* few, int lane) {
    u64 below[NQ], upto[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) { below[q] = __ballot(key[q] < lo); upto[q] = __ballot(key[q] < hi); }
    int cl = count(below), ch = count(upto);
    for (int it = 0; it < 100 && (K <= cl || K > ch); ++it) {
        if (K <= cl) {
            ch = cl; lo -= w;
#pragma unroll
            for (int q = 0; q < NQ; ++q) { upto[q] = below[q]; below[q] = __ballot(key[q] < lo); }
            cl = count(below);
        } else {
            cl = ch; hi += w;
#pragma unroll
            for (int q = 0; q < NQ; ++q) { below[q] = upto[q]; upto[q] = __ballot(key[q] < hi); }
            ch = count(upto);
        }
        w += w;
    }
    if (K <= cl || K > ch) {                   // an infinite finish time
        cl = 0; ch = 64 * NQ;
#pragma unroll
        for (int q = 0; q < NQ; ++q) { below[q] = 0; upto[q] = ~0ull; }
    }
    u64 act[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) act[q] = upto[q] & ~below[q];
    int n = ch - cl, r = K - cl;
    while (n > kFew) {
        // the first candidate by position as the pivot if the one wanted is in the lower half, else the last: fresh
        // delays lie in no order, what is left of a sorted list lies in ascending order
        T pivot = key[0];
        if (2 * r <= n) {
            bool found = false;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (!found && act[q] != 0) { found = true; const int l = __builtin_ctzll(act[q]); pivot = lane_value(key[q], l); act[q] &= ~(1ull << l); }
        } else {
            bool found = false;
#pragma unroll
            for (int q = NQ - 1; q >= 0; --q)
                if (!found && act[q] != 0) { found = true; const int l = 63 - __builtin_clzll(act[q]); pivot = lane_value(key[q], l); act[q] &= ~(1ull << l); }
        }
        u64 lt[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) lt[q] = __ballot(key[q] < pivot) & act[q];
        const int c = count(lt);
        if (r == c + 1) return pivot;
        if (r <= c) {
            n = c;
#pragma unroll
            for (int q = 0; q < NQ; ++q) act[q] = lt[q];
        } else {                               // the pivot and everything below it go
            r -= c + 1; n -= c + 1;
#pragma unroll
            for (int q = 0; q < NQ; ++q) act[q] &= ~lt[q];
        }
    }
    wave_fence();
    if (lane < kFew) few[lane] = unbounded<T>();
    wave_fence();
    int at = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (in_mask(act[q])) few[at + rank_in(act[q])] = key[q];
        at += __popcll(act[q]);
    }
    wave_fence();
    const T v = few[lane & (kFew - 1)];
    int rank = 0;
    for (int j = 0; j < n; j += 4) {
        T c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = few[j + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += (c[u] < v) ? 1 : 0;
    }
    for (;; --r) {                             // equal keys have the rank of the first of them; rank 0 is always there
        const u64 m = __ballot(rank == r - 1);
        if (m != 0) return lane_value(v, __builtin_ctzll(m));
        if (r <= 1) return v;
    }
}

struct Best { double key; int32_t id; };
template <int NQ>
__device__ __forceinline__ Best wave_argmin(const double (&key)[NQ], int lane) {
    double v = key[0];
#pragma unroll
    for (int q = 1; q < NQ; ++q) v = lesser(v, key[q]);
    Best b{wave_min(v, lane), 0};
    bool found = false;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {             // ties: the lowest worker
        const u64 m = __ballot(key[q] == b.key);
        if (!found && m != 0) { found = true; b.id = q * 64 + __builtin_ctzll(m); }
    }
    return b;
}

template <int NQ>
__device__ __forceinline__ void sort_list(const double* list, int cnt, double* out, int keep, int lane) {
    double v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = (lane * NQ + q < cnt) ? list[lane * NQ + q] : inf64();
    sort_keys<NQ>(v, lane);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (lane * NQ + q < keep) out[lane * NQ + q] = v[q];
}

template <int NQ, int VARIANT>
__global__ __launch_bounds__(64, VARIANT == kBatchAsync ? 4 : 8) void mc_kernel(McArgs a) {
    extern __shared__ double acc[];   // [values of K of this block][chain_len][2]
    const int lane = threadIdx.x;
    const int P = a.P, L = a.chain_len, nK = a.Kmax - a.Kmin + 1;
    const int slice = blockIdx.x % a.nslices, group = blockIdx.x / a.nslices, groups = gridDim.x / a.nslices;
    const int mineK = (nK - slice + a.nslices - 1) / a.nslices;
    const int cells = mineK * L;
    const int cells_max = ((nK + a.nslices - 1) / a.nslices) * L;
    for (int c = lane; c < 2 * cells; c += 64) acc[c] = 0.0;
    wave_fence();

    for (int64_t q0 = group; q0 < a.trials; q0 += groups) {
        const uint32_t trial = (uint32_t)(a.trial0 + q0);
        auto fresh_delay = [&](uint32_t aux, int worker, uint32_t ordinal, uint32_t version) -> float {
            return delay_from_bits(a.dist, draw(a.seed, kMonteCarlo, aux, trial, worker, ordinal, version).x);
        };
        if constexpr (VARIANT == kBatchAsync) {
            // No worker ever waits, whatever K is: the pushes of all workers merged in time order are one sequence
            // shared by every K, and update l happens at push l K (the superposition of renewal processes behind
            // Lemma 5).  The sequence goes to LDS; worker w's n-th delay is keyed by (worker w, version n).
            double* list = acc + 2 * cells_max;
            double* push = list + kList;
            const int npush = L * a.Kmax;
            double key[NQ];
            uint32_t started[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int w = q * 64 + lane;
                key[q] = (w < P) ? (double)fresh_delay(0, w, 0, 0) : inf64();
                started[q] = 0;
            }
            if (lane == 0) push[0] = 0.0;
            int n = 0, halvings = a.one_by_one ? 40 : 0;
            double t = 0.0, span = 0.0;
            while (n < npush && halvings < 40) {
                // renewals up to t + span, meant to be the ones still needed or the 300 next
                if (halvings == 0) span = (double)min(npush - n + 8 + (npush - n) / 8, 300) * a.mean_delay / (double)P;
                double soonest = key[0];
#pragma unroll
                for (int q = 1; q < NQ; ++q) soonest = lesser(soonest, key[q]);
                const double bound = greater(t + span, wave_min(soonest, lane));      // at least one push per list
                double key0[NQ];
                uint32_t started0[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) { key0[q] = key[q]; started0[q] = started[q]; }
                int cnt = 0;
                for (;;) {
                    int added = 0;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const bool mine = key[q] <= bound;
                        const u64 m = __ballot(mine);
                        if (m == 0) continue;
                        const int at = cnt + added + rank_in(m);
                        added += __popcll(m);
                        if (mine) {
                            if (at < kList) list[at] = key[q];
                            started[q] += 1;
                            key[q] = key[q] + (double)fresh_delay(0, q * 64 + lane, 0, started[q]);
                        }
                    }
                    cnt += added;
                    if (added == 0 || cnt > kList) break;
                }
                if (cnt == 0) break;           // no finish time compares with the bound (delays that are no numbers): one by one below
                if (cnt > kList) {             // the list does not hold them: once more with a shorter span
#pragma unroll
                    for (int q = 0; q < NQ; ++q) { key[q] = key0[q]; started[q] = started0[q]; }
                    span *= 0.5; ++halvings;
                    continue;
                }
                halvings = 0;
                t = bound;
                wave_fence();
                const int keep = min(cnt, npush - n);
                double* out = push + n + 1;
                if (cnt > 256) sort_list<8>(list, cnt, out, keep, lane);
                else if (cnt > 128) sort_list<4>(list, cnt, out, keep, lane);
                else if (cnt > 64) sort_list<2>(list, cnt, out, keep, lane);
                else if (cnt > 0) sort_list<1>(list, cnt, out, keep, lane);
                n += keep;
                wave_fence();
            }
            for (; n < npush; ++n) {           // more pushes at one instant than a list holds, or no lists: one by one
                const Best b = wave_argmin<NQ>(key, lane);
                if (lane == 0) push[n + 1] = b.key;
                if ((b.id & 63) == lane) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        if ((b.id >> 6) == q) {
                            started[q] += 1;
                            key[q] = key[q] + (double)fresh_delay(0, b.id, 0, started[q]);
                        }
                }
            }
            wave_fence();
            for (int c = lane; c < cells; c += 64) {       // one lane per (K, update) cell of this block
                const int kk = c / L, l = c - kk * L;
                const int K = a.Kmin + slice + kk * a.nslices;
                const double T = push[(l + 1) * K] - push[l * K];
                acc[2 * c] += T;
                acc[2 * c + 1] += T * T;
                if (a.per_trial) a.per_trial[(q0 * nK + (K - a.Kmin)) * L + l] = T;
            }
            wave_fence();
        } else {
        // fresh launch: P delays, shared by every K.  Sorted if enough values of K use the order (K-batch-sync needs the
        // workers, and a single K is selected for less); worker of a key = q * 64 + lane before sorting.
        float base[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int w = q * 64 + lane;
            base[q] = (w < P) ? fresh_delay(0, w, 0, 0) : __uint_as_float(0x7F800000u);
        }
        const bool sorted = VARIANT != kBatchSync && mineK > 2;
        if (sorted) sort_keys<NQ>(base, lane);

        double* few = acc + 2 * cells_max;
        float* window = reinterpret_cast<float*>(few + kFew);
        for (int K = a.Kmin + slice, kk = 0; K <= a.Kmax; K += a.nslices, ++kk) {
            // The chain's delays in the order it takes them: per update from the second on K restarts (K-async) or P
            // fresh ones (K-sync); K-batch-sync: P fresh ones, then the K - 1 restarts, from the first update on (whose
            // fresh ones are `base`).  Element i of that sequence is element i % per of update i / per.
            const int per = VARIANT == kAsync ? K : (VARIANT == kSync ? P : P + K - 1);
            const int total = per * (VARIANT == kBatchSync ? L : L - 1);
            const float recip = __builtin_amdgcn_rcpf((float)per);      // (i + 1/2) / per rounds down to the quotient for i < 1024, per < 512
            int win_lo = 0, win_hi = 0, next = VARIANT == kBatchSync ? P : 0;
            auto need = [&](int n) {           // the next n elements are in the window (n <= kWindow)
                if (next + n <= win_hi) return;
                win_lo = next;
                win_hi = min(total, win_lo + kWindow);
                const uint32_t u0 = (uint32_t)(win_lo / per);
                const int r0 = win_lo - (int)u0 * per;
                wave_fence();
                for (int i0 = 0; i0 < win_hi - win_lo; i0 += 64) {
                    const int i = r0 + i0 + lane;
                    const uint32_t u = per < 512 ? (uint32_t)(((float)i + 0.5f) * recip) : (i >= per ? 1u : 0u);
                    const int r = i - (int)u * per;
                    const uint32_t upd = u0 + u;
                    const bool restart = VARIANT == kBatchSync && r >= P;
                    const float x = fresh_delay((uint32_t)K, restart ? r - P : r, restart ? 1u : 0u, VARIANT == kBatchSync ? upd : upd + 1u);
                    if (i0 + lane < kWindow) window[i0 + lane] = x;
                }
                wave_fence();
            };
            // expected relative spread of T, roughly (a guess)
            const float narrow = 1.3f * __builtin_amdgcn_sqrtf((1.02f - (float)K * __builtin_amdgcn_rcpf((float)(P + 1))) * __builtin_amdgcn_rcpf((float)K));
            const int cell0 = kk * L;

            double t = 0.0, T = 0.0, kept = 0.0;
            double key[NQ];
            u64 gone[NQ];                      // K-async: the workers whose mini-batches the last update consumed
            for (int l = 0; l < L; ++l) {
                double t_new;
                if constexpr (VARIANT == kAsync) {
                    if (l == 0) {
#pragma unroll
                        for (int q = 0; q < NQ; ++q) key[q] = (double)base[q];
                    } else {
                        need(K);
                        const float* x = window + (next - win_lo);
                        int first = 0;
#pragma unroll
                        for (int q = 0; q < NQ; ++q) {
                            const bool mine = in_mask(gone[q]);
                            const double restart = t + (double)x[mine ? first + rank_in(gone[q]) : 0];
                            key[q] = mine ? restart : key[q];
                            first += __popcll(gone[q]);
                        }
                        next += K;
                    }
                    if (l == 0 && sorted) {
                        const int p = K - 1;
                        t_new = key[0];
#pragma unroll
                        for (int q = 0; q < NQ; ++q)
                            if (p % NQ == q) t_new = lane_value(key[q], p / NQ);
                    } else {
                        const double w = T * (double)narrow, at = t + T;
                        t_new = select_kth<NQ>(key, K, at - w, at + w, l == 0 ? 0.125 * a.mean_delay : w + w, few, lane);
                    }
                    if (l + 1 < L) {
#pragma unroll
                        for (int q = 0; q < NQ; ++q) gone[q] = __ballot(key[q] <= t_new);
                        int extra = count(gone) - K;
                        if (extra > 0) {       // several workers finish at t_new: only as many of them go as are wanted
#pragma unroll
                            for (int q = 0; q < NQ; ++q) {
                                u64 same = __ballot(key[q] == t_new);
                                while (extra > 0 && same != 0) { gone[q] &= ~(same & (0ull - same)); same &= same - 1; --extra; }
                            }
                        }
                    }
                } else if constexpr (VARIANT == kSync) {
                    float f[NQ];
                    if (l == 0) {
#pragma unroll
                        for (int q = 0; q < NQ; ++q) f[q] = base[q];
                    } else {
                        need(P);
                        const float* x = window + (next - win_lo);
#pragma unroll
                        for (int q = 0; q < NQ; ++q) f[q] = (q * 64 + lane < P) ? x[q * 64 + lane] : __uint_as_float(0x7F800000u);
                        next += P;
                    }
                    float s;
                    if (l == 0 && sorted) {
                        const int p = K - 1;
                        s = f[0];
#pragma unroll
                        for (int q = 0; q < NQ; ++q)
                            if (p % NQ == q) s = lane_value(f[q], p / NQ);
                    } else {
                        const float Tf = (float)T, w = Tf * narrow;
                        s = select_kth<NQ>(f, K, Tf - w, Tf + w, l == 0 ? 0.125f * (float)a.mean_delay : w + w, reinterpret_cast<float*>(few), lane);
                    }
                    t_new = t + (double)s;
                } else {
                    if (l == 0) {
#pragma unroll
                        for (int q = 0; q < NQ; ++q) key[q] = (double)base[q];
                    } else {
                        need(P);
                        const float* x = window + (next - win_lo);
#pragma unroll
                        for (int q = 0; q < NQ; ++q) key[q] = (q * 64 + lane < P) ? (double)x[q * 64 + lane] : inf64();
                        next += P;
                    }
                    double last = 0.0;
                    for (int pop0 = 0; pop0 < K; pop0 += 64) {
                        const int here = min(64, K - pop0), draws = min(64, K - 1 - pop0);
                        float x = 0.0f;        // lane i: the delay of the restart after pop pop0 + i
                        if (draws > 0) {
                            need(draws);
                            if (lane < draws) x = window[(next - win_lo) + lane];
                            next += draws;
                        }
                        for (int i = 0; i < here; ++i) {
                            const Best b = wave_argmin<NQ>(key, lane);
                            last = b.key;
                            const double restart = b.key + (double)lane_value(x, i);
#pragma unroll
                            for (int q = 0; q < NQ; ++q)
                                if (b.id == q * 64 + lane) key[q] = restart;
                        }
                    }
                    t_new = t + last;
                }
                T = t_new - t;
                t = t_new;
                // lane l % 64 keeps the T of update l; they are added up 64 at a time
                if (lane == (l & 63)) kept = T;
                if (l + 1 == L || (l & 63) == 63) {
                    const int c = cell0 + (l & ~63) + lane;
                    if (lane <= (l & 63)) {
                        acc[2 * c] += kept;
                        acc[2 * c + 1] += kept * kept;
                        if (a.per_trial) a.per_trial[(q0 * nK + (K - a.Kmin)) * L + (l & ~63) + lane] = kept;
                    }
                }
            }
        }
        }
    }
    wave_fence();
    for (int c = lane; c < 2 * cells; c += 64) a.partial[(int64_t)blockIdx.x * 2 * cells_max + c] = acc[c];
}

// Sums of the blocks' accumulators: out[2 cell], out[2 cell + 1].  A workgroup takes `width` (a power of two up to 64)
// words of one slice's accumulators; its 1024 / width groups of threads take consecutive runs of the slice's blocks, eight
// loads in flight, and the runs' sums are added in order, pairs first.  (A single value of K has 16 words and 8192 blocks:
// 64 words wide and four runs this took 120 us, as long as a small estimate itself.)
constexpr int kReduceThreads = 1024;
constexpr int64_t kReduceGroups = 32;      // workgroups wanted
__global__ __launch_bounds__(kReduceThreads) void mc_reduce_kernel(McArgs a, int groups, int cells_max, int width, double* out) {
    __shared__ double runs[kReduceThreads];
    const int w = threadIdx.x & (width - 1), part = threadIdx.x / width, parts = kReduceThreads / width;
    const int slice = blockIdx.y, c = blockIdx.x * width + w;
    const int nK = a.Kmax - a.Kmin + 1, L = a.chain_len;
    const int words = 2 * ((nK - slice + a.nslices - 1) / a.nslices) * L;
    const int per = (groups + parts - 1) / parts, g0 = part * per, g1 = min(groups, g0 + per);
    const int64_t step = (int64_t)a.nslices * 2 * cells_max;
    double sum = 0.0;
    if (c < words) {
        const double* src = a.partial + (int64_t)slice * 2 * cells_max + c;
        int g = g0;
        for (; g + 8 <= g1; g += 8) {
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = src[(g + i) * step];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += v[i];
        }
        for (; g < g1; ++g) sum += src[g * step];
    }
    runs[threadIdx.x] = sum;
    for (int stride = 1; stride < parts; stride *= 2) {
        __syncthreads();
        if (part % (2 * stride) == 0) runs[threadIdx.x] += runs[threadIdx.x + stride * width];
    }
    if (part == 0 && c < words) {
        const int local = c >> 1, kk = local / L, l = local - kk * L;
        out[2 * ((int64_t)(slice + kk * a.nslices) * L + l) + (c & 1)] = runs[w];
    }
}

template <int NQ, int VARIANT>
hipError_t launch_mc_variant(const McArgs& a, unsigned blocks, size_t lds, hipStream_t s) {
    const hipError_t e = hipFuncSetAttribute((const void*)mc_kernel<NQ, VARIANT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mc_kernel<NQ, VARIANT>), dim3(blocks), dim3(64), lds, s, a);
    return hipGetLastError();
}
template <int NQ>
hipError_t launch_mc(const McArgs& a, unsigned blocks, size_t lds, hipStream_t s) {
    switch (a.variant) {
    case kSync: return launch_mc_variant<NQ, kSync>(a, blocks, lds, s);
    case kBatchSync: return launch_mc_variant<NQ, kBatchSync>(a, blocks, lds, s);
    case kAsync: return launch_mc_variant<NQ, kAsync>(a, blocks, lds, s);
    default: return launch_mc_variant<NQ, kBatchAsync>(a, blocks, lds, s);
    }
}

}  // namespace
}  // namespace ssgd

using namespace ssgd;

namespace {
void mc_fail(const std::string& m) { set_global_error(m); }
}  // namespace

extern "C" __attribute__((visibility("default"))) ssgd_status ssgd_runtime_mc(int32_t variant, int32_t P, int32_t Kmin, int32_t Kmax,
                                       const ssgd_delay_dist* dist, int64_t trial0, int64_t trials,
                                       int32_t chain_len, uint64_t seed, void* hip_stream, double* mean,
                                       double* var, double* sum, double* sumsq, double* per_trial) {
    if (!dist || dist->kind == SSGD_TABLE || dist->kind < 0 || dist->kind > SSGD_PARETO) { mc_fail("invalid distribution"); return SSGD_EINVAL; }
    if ((dist->kind != SSGD_PARETO && !(dist->rate > 0)) || (dist->kind == SSGD_PARETO && (!(dist->alpha > 0) || !(dist->scale > 0))) ||
        (dist->kind == SSGD_SHIFTED_EXP && std::isnan(dist->shift))) { mc_fail("invalid distribution parameters"); return SSGD_EINVAL; }
    if (variant < SSGD_K_SYNC || variant > SSGD_K_BATCH_ASYNC) { mc_fail("unknown variant"); return SSGD_EINVAL; }
    if (P < 1 || P > kMaxWorkers || Kmin < 1 || Kmax < Kmin || chain_len < 1 || trials < 1 || trial0 < 0 || trial0 + trials > (1ll << 32)) { mc_fail("P, K range, chain_len or trials out of range"); return SSGD_EINVAL; }
    if (variant != SSGD_K_BATCH_SYNC && variant != SSGD_K_BATCH_ASYNC && Kmax > P) { mc_fail("K must not exceed P"); return SSGD_EINVAL; }
    if (Kmax > 65535) { mc_fail("K too large"); return SSGD_EINVAL; }
    const int nK = Kmax - Kmin + 1;
    const int64_t cells = (int64_t)nK * chain_len;
    // Accumulators of at most 2.5 KB per wavefront, so that with the window of delays 32 of them fit a CU.  The limit on
    // chain_len is stated in accumulators and pushes alone.
    int nslices = 1;
    while (nslices < nK && (int64_t)((nK + nslices - 1) / nslices) * chain_len * 16 > 2560) ++nslices;
    const int64_t cells_max = (int64_t)((nK + nslices - 1) / nslices) * chain_len;
    size_t lds = sizeof(double) * 2 * cells_max;
    if (variant == SSGD_K_BATCH_ASYNC) lds += sizeof(double) * ((size_t)chain_len * Kmax + 1);   // the push sequence of a trial
    if (lds > 64 * 1024) { mc_fail("chain_len (K-batch-async: chain_len * Kmax) too large for one launch"); return SSGD_EINVAL; }
    lds += variant == SSGD_K_BATCH_ASYNC ? sizeof(double) * kList : sizeof(double) * kFew + sizeof(float) * kWindow;
    if (per_trial && trials * cells > (1ll << 27)) { mc_fail("per_trial output limited to 2^27 values"); return SSGD_EINVAL; }
    hipStream_t st = (hipStream_t)hip_stream;
    McArgs a{};
    a.dist.kind = dist->kind; a.dist.shift = (float)dist->shift; a.dist.rate = (float)dist->rate;
    a.dist.alpha = (float)dist->alpha; a.dist.scale = (float)dist->scale; a.dist.table = nullptr; a.dist.table_len = 0;
    a.dist.inv_div = quotient_reciprocal(dist->kind == SSGD_PARETO ? a.dist.alpha : a.dist.rate);
    a.seed = seed; a.variant = variant; a.P = P; a.Kmin = Kmin; a.Kmax = Kmax; a.chain_len = chain_len;
    a.trial0 = trial0; a.trials = trials; a.nslices = nslices;
    switch (dist->kind) {
    case SSGD_EXP: a.mean_delay = 1.0 / dist->rate; break;
    case SSGD_SHIFTED_EXP: a.mean_delay = dist->shift + 1.0 / dist->rate; break;
    default: a.mean_delay = dist->alpha > 1.5 ? dist->scale * dist->alpha / (dist->alpha - 1.0) : 3.0 * dist->scale; break;
    }
    a.one_by_one = dist->kind == SSGD_SHIFTED_EXP && dist->shift < 0.0 ? 1 : 0;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) { mc_fail("no device"); return SSGD_EDEVICE; }
    const int64_t groups = std::max<int64_t>(1, std::min<int64_t>(trials, (int64_t)cus * 32 / nslices));
    const int64_t blocks = groups * nslices;
    void *d_partial = nullptr, *d_pt = nullptr;
    ssgd_status rc = SSGD_OK;
    std::vector<double> host((size_t)(2 * cells));
    const int64_t partial_words = blocks * 2 * cells_max;
    do {
        if (hipMalloc(&d_partial, sizeof(double) * (partial_words + 2 * cells)) != hipSuccess) { mc_fail("hipMalloc"); rc = SSGD_ENOMEM; break; }
        if (per_trial && hipMalloc(&d_pt, sizeof(double) * trials * cells) != hipSuccess) { mc_fail("hipMalloc"); rc = SSGD_ENOMEM; break; }
        a.partial = (double*)d_partial; a.per_trial = (double*)d_pt;
        double* d_sums = a.partial + partial_words;
        hipError_t e = P <= 64 ? launch_mc<1>(a, (unsigned)blocks, lds, st) : (P <= 128 ? launch_mc<2>(a, (unsigned)blocks, lds, st) : launch_mc<4>(a, (unsigned)blocks, lds, st));
        if (e == hipSuccess) {
            // (narrower where that leaves too few workgroups to keep enough loads in flight: 8192 blocks of 16 words 16 -> 12 us)
            int width = 2;
            while (width < 64 && width < 2 * cells_max && (2 * cells_max / (2 * width)) * nslices >= kReduceGroups) width *= 2;
            hipLaunchKernelGGL(mc_reduce_kernel, dim3((unsigned)((2 * cells_max + width - 1) / width), (unsigned)nslices), dim3(kReduceThreads), 0, st,
                               a, (int)groups, (int)cells_max, width, d_sums);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(host.data(), d_sums, sizeof(double) * host.size(), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess && per_trial) e = hipMemcpyAsync(per_trial, d_pt, sizeof(double) * trials * cells, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) { mc_fail(std::string("mc kernel: ") + hipGetErrorString(e)); rc = SSGD_EDEVICE; break; }
        for (int64_t c = 0; c < cells; ++c) {
            const double s = host[2 * c], s2 = host[2 * c + 1];
            if (sum) sum[c] = s;
            if (sumsq) sumsq[c] = s2;
            if (mean) mean[c] = s / (double)trials;
            if (var) var[c] = trials > 1 ? (s2 - s * s / (double)trials) / (double)(trials - 1) : 0.0;
        }
    } while (0);
    if (d_partial) (void)hipFree(d_partial);
    if (d_pt) (void)hipFree(d_pt);
    return rc;
}
