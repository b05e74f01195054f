// Event process of the parameter server (Sec. 2.2) on the device: random delays
// (Sec. 3.1), K-of-P selection of the earliest finishers, staleness bookkeeping.
//
// One wavefront simulates one replica; each lane owns up to four of the P <= 256
// workers.  The delays do not depend on the data, so a whole segment of updates is
// scheduled before any gradient is taken; the gradient kernels then read the trace.
#include <algorithm>

#include "common.hpp"

namespace ssgd {
namespace {


struct Best { double key; int32_t id; };

__device__ __forceinline__ bool before(double ka, int32_t ia, double kb, int32_t ib) {
    return ka < kb || (ka == kb && ia < ib);   // ties go to the lower worker id
}

// Smallest (key, id) over the first `width` lanes (a power of two covering every worker), known to every
// lane afterwards.  The butterfly carries the key only; the owner is found with a ballot, and the rare
// tie between lanes goes to the lowest worker id.
template <int CTRL>
__device__ __forceinline__ double dpp_fetch(double k) {
    const long long b = __double_as_longlong(k);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((unsigned long long)b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ Best wave_min(Best b, int width) {
    double k = b.key;
    // inside a row of 16 lanes the exchange is a data-parallel-primitive move (no LDS round trip):
    // lane ^ 1, lane ^ 2, then the mirrored lane of the other half of 8, then of 16
    if (width > 1) { const double o = dpp_fetch<0xB1>(k); k = o < k ? o : k; }     // quad_perm [1,0,3,2]
    if (width > 2) { const double o = dpp_fetch<0x4E>(k); k = o < k ? o : k; }     // quad_perm [2,3,0,1]
    if (width > 4) { const double o = dpp_fetch<0x141>(k); k = o < k ? o : k; }    // row_half_mirror
    if (width > 8) { const double o = dpp_fetch<0x140>(k); k = o < k ? o : k; }    // row_mirror
    for (int off = 16; off < width; off <<= 1) {
        const double ok = __shfl_xor(k, off, 64);
        k = ok < k ? ok : k;
    }
    const long long kb = __double_as_longlong(k);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)kb);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((unsigned long long)kb >> 32));
    const double kmin = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    unsigned long long mask = __ballot(b.key == kmin && b.id != 0x7FFFFFFF);
    int best = 0x7FFFFFFF;
    while (mask) {
        const int l = __builtin_ctzll(mask);
        mask &= mask - 1;
        const int id = __builtin_amdgcn_readlane(b.id, l);
        best = id < best ? id : best;
    }
    return Best{kmin, best};
}

template <int NQ>
__device__ __forceinline__ Best local_min(const double (&key)[NQ], uint32_t skip, int lane, int P) {
    Best b{__longlong_as_double(0x7FF0000000000000LL), 0x7FFFFFFF};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int w = lane + 64 * q;
        if (w < P && !((skip >> q) & 1u) && before(key[q], w, b.key, b.id)) { b.key = key[q]; b.id = w; }
    }
    return b;
}

// Update j of a synchronous variant (K-sync, K-batch-sync): every worker starts a fresh mini-batch at t_j with w_j, so
// the contributors do not depend on earlier updates.  One wavefront; writes the lists, returns t_{j+1} - t_j.
template <int NQ, class Draw>
__device__ __forceinline__ double sync_update(const Draw& draw_delay, bool batch, int P, int K, int width, int lane, int64_t j,
                                              int32_t* sel, int32_t* tau, int32_t* order) {
    const uint32_t ver = (uint32_t)j;
    double key[NQ];
    int32_t ord[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int w = lane + 64 * q;
        ord[q] = 0;
        key[q] = (w < P) ? (double)draw_delay(w, 0, ver) : 0.0;
    }
    uint32_t taken = 0;
    double last = 0.0;
    for (int l = 0; l < K; ++l) {
        const Best b = wave_min(local_min(key, taken, lane, P), width);
        last = b.key;
        if ((b.id & 63) == lane) {
            const int q = b.id >> 6;
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) {
                if (qq != q) continue;
                sel[l] = b.id; tau[l] = (int32_t)j; order[l] = ord[qq];
                if (!batch) {
                    taken |= 1u << qq;
                } else {
                    // K-batch-sync: the worker starts its next mini-batch at the same w_j
                    ord[qq] += 1;
                    if (l + 1 < K) key[qq] = key[qq] + (double)draw_delay(b.id, ord[qq], ver);
                }
            }
        }
    }
    return last;
}

// The updates of a synchronous segment side by side, one wavefront each; the time between updates is left in the trace
// for sync_clock_kernel to add up.  (One wavefront per replica took them one after the other, K argmin rounds of 0.4 us
// each; that stays for segments so short that a second launch, about 5 us, costs more.)
template <int NQ, bool TABLE>
__global__ __launch_bounds__(64 * kSyncWaves) void sync_schedule_kernel(SchedArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * kSyncWaves + wave;
    if (q >= a.count) return;
    const int rep = a.replica0 + blockIdx.y, P = a.P, Kcap = a.tr.Kcap;
    const int64_t row = (int64_t)rep * a.tr.cap + a.j0 + q;
    auto draw_delay = [&](uint32_t worker, uint32_t ordinal, uint32_t version) -> float {
        if constexpr (TABLE) return delay(a.dist, a.seed, kDelay, 0, rep, P, a.table_ord, worker, ordinal, version);
        else return delay_from_bits(a.dist, draw(a.seed, kDelay, 0, rep, worker, ordinal, version).x);
    };
    int width = 1;
    while (width < P && width < 64) width <<= 1;
    const int K = a.ws.curK[rep];
    int32_t *sel = a.tr.sel + row * Kcap, *tau = a.tr.tau + row * Kcap, *ord = a.tr.ord + row * Kcap;
    for (int l = K + lane; l < Kcap; l += 64) { sel[l] = -1; tau[l] = -1; ord[l] = -1; }
    const double dt = sync_update<NQ>(draw_delay, a.variant == kBatchSync, P, K, width, lane, a.j0 + q, sel, tau, ord);
    if (lane == 0) { a.tr.t[row] = dt; a.tr.K[row] = K; }
}

// Clock of a synchronous segment: t_{j+1} = t_j + the difference left in the trace, in the order of the updates.
__global__ __launch_bounds__(64) void sync_clock_kernel(SchedArgs a) {
    const int lane = threadIdx.x, rep = a.replica0 + blockIdx.x;
    double* t = a.tr.t + (int64_t)rep * a.tr.cap + a.j0;
    double clock = a.ws.clock[rep];
    double next = lane < a.count ? t[lane] : 0.0;
    for (int64_t base = 0; base < a.count; base += 64) {
        const long long bits = __double_as_longlong(next);
        double mine = 0.0;
        next = base + 64 + lane < a.count ? t[base + 64 + lane] : 0.0;
#pragma unroll
        for (int l = 0; l < 64; ++l) {         // past the end: + 0
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, l);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)bits >> 32), l);
            clock = clock + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
            mine = lane == l ? clock : mine;
        }
        if (base + lane < a.count) t[base + lane] = mine;
    }
    if (lane == 0) { a.ws.clock[rep] = clock; a.ws.n_done[rep] = a.count; a.ws.crossed[rep] = 0; }
}

// NQ: workers per lane (1 while P <= 64).  TABLE: delays come from a table in memory; kept out of the common
// instantiation, whose loop then holds no load and never waits for its own trace stores.
template <int NQ, bool TABLE>
__global__ __launch_bounds__(64) void schedule_kernel(SchedArgs a) {
    const int lane = threadIdx.x;
    const int rep = a.replica0 + blockIdx.x;
    const int P = a.P, Kcap = a.tr.Kcap;
    const int64_t cap = a.tr.cap;
    double* tr_t = a.tr.t + (int64_t)rep * cap;
    int32_t* tr_K = a.tr.K + (int64_t)rep * cap;
    int32_t* tr_sel = a.tr.sel + (int64_t)rep * cap * Kcap;
    int32_t* tr_tau = a.tr.tau + (int64_t)rep * cap * Kcap;
    int32_t* tr_ord = a.tr.ord + (int64_t)rep * cap * Kcap;

    auto draw_delay = [&](uint32_t worker, uint32_t ordinal, uint32_t version) -> float {
        if constexpr (TABLE) return delay(a.dist, a.seed, kDelay, 0, rep, P, a.table_ord, worker, ordinal, version);
        else return delay_from_bits(a.dist, draw(a.seed, kDelay, 0, rep, worker, ordinal, version).x);
    };
    int width = 1;
    while (width < P && width < 64) width <<= 1;
    const int K = a.ws.curK[rep];
    double clock = a.ws.clock[rep];
    double key[NQ];
    int32_t tau[NQ], ord[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int w = lane + 64 * q;
        key[q] = 0.0; tau[q] = 0; ord[q] = 0;
        if (w < P && a.variant >= kAsync) {
            key[q] = a.ws.finish[(int64_t)rep * P + w];
            tau[q] = a.ws.tau[(int64_t)rep * P + w];
            ord[q] = a.ws.ord[(int64_t)rep * P + w];
        }
    }

    int64_t done = 0;
    int crossed = 0;
    if (NQ == 1 && !TABLE && a.variant == kAsync && !(a.interval_t > 0.0)) {
        // K-async with a worker per lane, in a loop of its own: every lane ranks its worker's finish time against all
        // P of them, which gives the K earliest in consume-list order at once.  The delay a worker would draw if
        // it restarted now depends on (worker, version) only: the 64 lanes draw it for 64 / width versions in one go.
        const int wmask = width - 1, per = 64 / width;
        const int me = lane & wmask;
        float ahead = 0.0f;
        int64_t ahead_base = a.j0 + 1 - per;         // refilled before the first use
        double mine = key[0];
        int32_t mytau = tau[0];
        for (; done < a.count; ++done) {
            const int64_t j = a.j0 + done;
            const int slot = (int)(j + 1 - ahead_base);
            if (slot >= per) {
                ahead_base = j + 1;
                ahead = 0.0f;
                if (me < P) ahead = draw_delay((uint32_t)me, 0, (uint32_t)(ahead_base + lane / width));
            }
            const float restart = __shfl(ahead, me + width * (slot >= per ? 0 : slot), 64);
            const long long bits = __double_as_longlong(mine);
            int rank = 0;
            for (int w = 0; w < P; ++w) {
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, w);
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)bits >> 32), w);
                const double other = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                rank += before(other, w, mine, lane) ? 1 : 0;
            }
            const int last = __builtin_ctzll(__ballot(lane < P && rank == K - 1));
            const uint32_t tlo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, last);
            const uint32_t thi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)bits >> 32), last);
            const double t_new = __longlong_as_double((long long)(((unsigned long long)thi << 32) | tlo));
            if (lane < P && rank < K) {
                tr_sel[j * Kcap + rank] = lane; tr_tau[j * Kcap + rank] = mytau; tr_ord[j * Kcap + rank] = 0;
                mytau = (int32_t)(j + 1);
                mine = t_new + (double)restart;
            }
            for (int l = K + lane; l < Kcap; l += 64) {
                tr_sel[j * Kcap + l] = -1; tr_tau[j * Kcap + l] = -1; tr_ord[j * Kcap + l] = -1;
            }
            if (lane == 0) { tr_t[j] = t_new; tr_K[j] = K; }
            clock = t_new;
        }
        key[0] = mine; tau[0] = mytau;
    }
    if (!TABLE && a.variant == kAsync && NQ > 1 && K >= 8 && 18 * K >= P * NQ && !(a.interval_t > 0.0)) {
        // K-async with many contributors per update: K rounds of a wave-wide argmin (0.4 us each) cost more than
        // ranking every worker's finish time against all P of them (one pass over the workers, whatever K is: 22 us
        // at P = 256), which also gives the K earliest in consume-list order.
        for (; done < a.count; ++done) {
            const int64_t j = a.j0 + done;
            double nd[NQ];
            int rank[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int w = lane + 64 * q;
                nd[q] = (w < P) ? (double)draw_delay(w, 0, (uint32_t)j + 1u) : 0.0;
                rank[q] = 0;
            }
#pragma unroll
            for (int qo = 0; qo < NQ; ++qo) {
                const long long bits = __double_as_longlong(key[qo]);
                const int lim = min(64, P - 64 * qo);                  // workers held in register qo
                for (int l = 0; l < lim; ++l) {
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, l);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)bits >> 32), l);
                    const double other = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                    const int wo = l + 64 * qo;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) rank[q] += before(other, wo, key[q], lane + 64 * q) ? 1 : 0;
                }
            }
            // the K-th earliest finish time is the time of the update
            double t_new = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const unsigned long long m = __ballot(lane + 64 * q < P && rank[q] == K - 1);
                if (m != 0ull) {
                    const int l = __builtin_ctzll(m);
                    const long long bits = __double_as_longlong(key[q]);
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, l);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)bits >> 32), l);
                    t_new = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                }
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int w = lane + 64 * q;
                if (w < P && rank[q] < K) {
                    tr_sel[j * Kcap + rank[q]] = w; tr_tau[j * Kcap + rank[q]] = tau[q]; tr_ord[j * Kcap + rank[q]] = 0;
                    tau[q] = (int32_t)(j + 1);
                    key[q] = t_new + nd[q];
                }
            }
            for (int l = K + lane; l < Kcap; l += 64) {
                tr_sel[j * Kcap + l] = -1; tr_tau[j * Kcap + l] = -1; tr_ord[j * Kcap + l] = -1;
            }
            if (lane == 0) { tr_t[j] = t_new; tr_K[j] = K; }
            clock = t_new;
        }
    }
    for (; done < a.count; ++done) {
        const int64_t j = a.j0 + done;
        const uint32_t ver = (uint32_t)j;
        for (int l = lane; l < Kcap; l += 64) {
            tr_sel[j * Kcap + l] = -1; tr_tau[j * Kcap + l] = -1; tr_ord[j * Kcap + l] = -1;
        }
        double t_new = clock;
        if (a.variant == kSync || a.variant == kBatchSync) {
            const double last = sync_update<NQ>(draw_delay, a.variant == kBatchSync, P, K, width, lane, j, tr_sel + j * Kcap,
                                                tr_tau + j * Kcap, tr_ord + j * Kcap);
            t_new = clock + last;
        } else if (a.variant == kBatchAsync) {
            // K-batch-async: the K earliest mini-batches contribute, whoever computed them.  A worker that pushes
            // one of the first K-1 re-reads the parameters (still w_j) and starts its next mini-batch at once; the
            // K-th push triggers update j, and that worker reads w_{j+1}.
            for (int l = 0; l < K; ++l) {
                const Best b = wave_min(local_min(key, 0u, lane, P), width);
                t_new = b.key;
                if ((b.id & 63) == lane) {
                    const int q = b.id >> 6;
#pragma unroll
                    for (int qq = 0; qq < NQ; ++qq) {
                        if (qq != q) continue;
                        tr_sel[j * Kcap + l] = b.id; tr_tau[j * Kcap + l] = tau[qq]; tr_ord[j * Kcap + l] = ord[qq];
                        if (l + 1 < K) {
                            if (tau[qq] == (int32_t)j) ord[qq] += 1; else { tau[qq] = (int32_t)j; ord[qq] = 0; }
                            key[qq] = key[qq] + (double)draw_delay(b.id, ord[qq], ver);
                        } else {
                            tau[qq] = (int32_t)(j + 1); ord[qq] = 0;
                            key[qq] = t_new + (double)draw_delay(b.id, 0, ver + 1u);
                        }
                    }
                }
            }
        } else {
            // K-async: the K earliest finishers contribute; only they restart, at t_{j+1}.  The delay a
            // worker would draw if it restarted now depends on (worker, version) only, so every lane
            // draws it up front, off the selection's dependency chain.
            double nd[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int w = lane + 64 * q;
                nd[q] = 0.0;
                if (w < P) nd[q] = (double)draw_delay(w, 0, ver + 1u);
            }
            uint32_t taken = 0;
            for (int l = 0; l < K; ++l) {
                const Best b = wave_min(local_min(key, taken, lane, P), width);
                t_new = b.key;
                if ((b.id & 63) == lane) {
                    const int q = b.id >> 6;
#pragma unroll
                    for (int qq = 0; qq < NQ; ++qq) {
                        if (qq != q) continue;
                        tr_sel[j * Kcap + l] = b.id; tr_tau[j * Kcap + l] = tau[qq]; tr_ord[j * Kcap + l] = 0;
                        taken |= 1u << qq;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if (!((taken >> q) & 1u)) continue;
                tau[q] = (int32_t)(j + 1);
                key[q] = t_new + nd[q];
            }
        }
        if (lane == 0) { tr_t[j] = t_new; tr_K[j] = K; }
        const double t_prev = clock;
        clock = t_new;
        if (a.interval_t > 0.0 && floor(t_new / a.interval_t) > floor(t_prev / a.interval_t)) {
            crossed = 1; ++done; break;
        }
    }

#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int w = lane + 64 * q;
        if (w < P && a.variant >= kAsync) {
            a.ws.finish[(int64_t)rep * P + w] = key[q];
            a.ws.tau[(int64_t)rep * P + w] = tau[q];
            a.ws.ord[(int64_t)rep * P + w] = ord[q];
        }
    }
    if (lane == 0) { a.ws.clock[rep] = clock; a.ws.n_done[rep] = done; a.ws.crossed[rep] = crossed; }
}

// AdaSync controller (Sec. 6): one thread per replica, run after the gradient kernels of a segment.
__global__ void adasync_kernel(AdaArgs a, int replicas) {
    const int rep = blockIdx.x * blockDim.x + threadIdx.x;
    if (rep >= replicas) return;
    const float* loss = a.tr.loss + (int64_t)rep * a.tr.cap;
    int K = a.ws.curK[rep];
    if (a.j_end >= 1 && a.ws.F0[rep] < 0.0) a.ws.F0[rep] = (double)loss[0];
    if (a.mode == 1) {
        if (!a.window_closed) return;
        double s = 0.0;
        for (int64_t j = a.j_end - a.window; j < a.j_end; ++j) s += (double)loss[j];
        const double mean = s / (double)a.window;
        if (a.ws.win_index[rep] >= 1 && mean > (1.0 - a.rel_tol) * a.ws.win_prev[rep]) {
            K = 2 * K; if (K > a.Kmax) K = a.Kmax;
        }
        a.ws.win_prev[rep] = mean;
        a.ws.win_index[rep] += 1;
    } else {
        if (!a.ws.crossed[rep]) return;
        double s = 0.0;
        const int64_t j0 = a.ws.int_start[rep];
        for (int64_t j = j0; j < a.j_end; ++j) s += (double)loss[j];
        const double Fstart = s / (double)(a.j_end - j0);
        a.ws.int_start[rep] = a.j_end;
        if (K < a.Kmax && Fstart > 0.0) {
            const double ratio = a.ws.F0[rep] / Fstart;
            double Knew;
            if (a.mode == 2) {
                Knew = (double)a.K0 * sqrt(ratio);                       // Algorithm 1
            } else {
                const double q = (double)a.K0 * a.K0 / (double)(a.P - a.K0) * ratio;   // App. D, K-sync
                Knew = 0.5 * (-q + sqrt(q * q + 4.0 * q * (double)a.P));
            }
            int Ki = (int)floor(Knew + 0.5);
            if (Ki < K) Ki = K;
            if (Ki > a.Kmax) Ki = a.Kmax;
            K = Ki;
        }
    }
    a.ws.curK[rep] = K;
}

}  // namespace

void launch_schedule(const SchedArgs& a, int replicas, hipStream_t s) {
    const bool table = a.dist.kind == 3;
    // (a segment that ends where the clock crosses an interval is found update by update; a grid has 65535 rows)
    if ((a.variant == kSync || a.variant == kBatchSync) && !(a.interval_t > 0.0) && a.count * (int64_t)a.tr.Kcap >= 16 && replicas <= 65535) {
        for (int64_t off = 0; off < a.count; off += kSyncUpdatesPerLaunch) {
            SchedArgs b = a;
            b.j0 = a.j0 + off; b.count = std::min(kSyncUpdatesPerLaunch, a.count - off);
            const dim3 grid(sync_schedule_blocks(b.count), (unsigned)replicas), block(64 * kSyncWaves);
            if (a.P <= 64) {
                if (table) hipLaunchKernelGGL((sync_schedule_kernel<1, true>), grid, block, 0, s, b);
                else hipLaunchKernelGGL((sync_schedule_kernel<1, false>), grid, block, 0, s, b);
            } else {
                if (table) hipLaunchKernelGGL((sync_schedule_kernel<kMaxWorkers / 64, true>), grid, block, 0, s, b);
                else hipLaunchKernelGGL((sync_schedule_kernel<kMaxWorkers / 64, false>), grid, block, 0, s, b);
            }
        }
        hipLaunchKernelGGL(sync_clock_kernel, dim3(replicas), dim3(64), 0, s, a);
        return;
    }
    if (a.P <= 64) {
        if (table) hipLaunchKernelGGL((schedule_kernel<1, true>), dim3(replicas), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((schedule_kernel<1, false>), dim3(replicas), dim3(64), 0, s, a);
    } else {
        if (table) hipLaunchKernelGGL((schedule_kernel<kMaxWorkers / 64, true>), dim3(replicas), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((schedule_kernel<kMaxWorkers / 64, false>), dim3(replicas), dim3(64), 0, s, a);
    }
}

void launch_adasync(const AdaArgs& a, int replicas, hipStream_t s) {
    hipLaunchKernelGGL(adasync_kernel, dim3((replicas + 63) / 64), dim3(64), 0, s, a, replicas);
}

}  // namespace ssgd
