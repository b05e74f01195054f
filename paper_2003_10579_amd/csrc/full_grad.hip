// Gradient of the objective over the whole data set, grad F(w) = (1/N) sum_n grad f(w, xi_n) (Eq. (1)), for the
// linear models: the quantity in which the staleness bound (fifth assumption of Sec. 4.1) is stated
// (E||grad F(w_j) - grad F(w_tau)||^2 <= gamma E||grad F(w_j)||^2).
//
// full_grad_fused_kernel reads the sample matrix once; the read is what bounds it.  A workgroup owns a run of rows and
// takes 16 of them at a time, wave w the columns of its share (up to 384: 24 blocks of 16, held in 96 registers in the
// layout of the MFMA operand).  Logits: fp32 MFMA 16x16x4 with the weights from LDS, the waves' partial sums meet in LDS
// (one barrier per 16 rows), every wave takes softmax or residual itself.  Gradient: delta^T X needs the rows with the
// lane on the column where the forward pass had it on the row; a block of 16 x 16 is turned over through a buffer of the
// wave's own in LDS (one 16-byte store and four 4-byte loads per lane, all in different banks), one block ahead of its
// contraction.  (By four MFMA steps with a selector of ones instead, matrix time was 18 000 cycles per 16 rows of d = 3072 and
// CU where it is 12 000, and the pass took 197 us where it takes 165.)  The registers of a block are refilled with the next 16
// rows as soon as it has been turned over, so the loads travel behind the rest of the gradient pass and the next forward pass.
// The gradient stays in registers (96 more) until the run of rows ends.  The rows take 23 000 cycles to arrive.
// full_grad_reduce_kernel adds the workgroups' partial gradients in order in fp64.
// N = 50000, d = 3072, 10 classes: 165 us (3.7 TB/s) + 10 us for the reduction, where the two passes below took 518 +
// 297 + 35; N = 4096, d = 256, least squares: 5 + 3 us where they took 5 + 40 + 6 (32 workgroups in the second pass).
//
// Shapes whose weights do not fit the LDS beside that (more than about 11 classes at d = 3072, or d > 3072) take two
// passes: deltas to memory (16 floats per sample), then G[c][col] = sum_n delta[n][c] X[n][col] with a thread per column.
#include <mutex>

#include "common.hpp"

namespace ssgd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Scratch memory of the entry point that allocates nothing: every GPU the library runs on holds one copy of this
// array for the life of the process (36 MiB: one partial gradient per workgroup, at most 256 of 34 k floats).  In host code the name stands for the symbol, not for a device
// address: the address on the current device comes from hipGetSymbolAddress, once per device, and only that pointer
// is handed to kernels.
constexpr int64_t kStaticScratchFloats = 9ll << 20;
constexpr int64_t kStaticLimitFloats = 4ll << 20;      // what the entry point accepts, in the floats of full_grad_scratch_floats
static __device__ __align__(256) float scratch[kStaticScratchFloats];
constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

struct FullGradArgs {
    const float* X;
    const void* y;
    const float* w;      // parameters of one replica, standard layout
    int64_t N;
    int32_t d, C, kind;
    int32_t chunks;      // the samples are split into this many runs of chunk_rows rows
    int64_t chunk_rows;
    int32_t stride;      // fused kernel: words per weight row in LDS
    float* delta;        // [N][16], two-pass kernels
    float* partial;      // [chunks][C][d + 1]
    float* out;          // [C * d (+ C)], device memory or mapped host memory
    Done done;
};

constexpr int FG_TSTRIDE = 20;    // words per sample in a wave's buffer for turning delta over: 16-byte rows in different banks

// Orders the LDS accesses of one wavefront for the compiler.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// BL: 16-column blocks of a wave's share (even); columns past d have zero weights in LDS and their loads are sent out
// of range, so that no step is behind a branch (behind one the compiler waits for every load in flight).
template <int KIND, int WAVES, int BL>
__global__ __launch_bounds__(64 * WAVES, BL <= 8 ? 4 : 2) void full_grad_fused_kernel(FullGradArgs a) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d, C = a.C, stride = a.stride;
    float* wl = smem;                                                    // [C][stride], zero past column d
    f32x4* part = reinterpret_cast<f32x4*>(smem + (size_t)C * stride);   // [2][WAVES][64]
    float* turn = reinterpret_cast<float*>(part + 2 * WAVES * 64) + wave * 16 * FG_TSTRIDE;

    const int j = lane & 15, quarter = lane >> 4;
    const int s_lo = wave * BL;                                          // first block of this wave's share
    const int mine = (d - 16 * s_lo - 4 * quarter + 15) >> 4;            // this lane's blocks inside the row (<= 0: none); d % 4 == 0
    const uint32_t row_bytes = (uint32_t)d * 4u;
    const int lane_off = (int)(j * row_bytes) + (16 * s_lo + 4 * quarter) * 4;
    const int64_t r0 = (int64_t)blockIdx.x * a.chunk_rows, r1 = min(a.N, r0 + a.chunk_rows);
    auto rows_at = [&](int64_t r) -> __amdgpu_buffer_rsrc_t {       // 16 rows from r on; rows past the run read as zeros
        const int64_t rows = (r < r1) ? min<int64_t>(16, r1 - r) : 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.X + (rows > 0 ? r : 0) * (int64_t)d), 0, (int)(rows * row_bytes), 0x00020000);
    };
    auto load = [&](const __amdgpu_buffer_rsrc_t& rs, int u) -> f32x4 {
        const int off = (u < mine) ? lane_off : (int)0x80000000;
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 64 * u, 0));
    };
    f32x4 xq[BL], g[BL];
    {
        const __amdgpu_buffer_rsrc_t rs = rows_at(r0);
#pragma unroll
        for (int u = 0; u < BL; ++u) { g[u] = f32x4{0.f, 0.f, 0.f, 0.f}; xq[u] = load(rs, u); }
    }
    for (int c = 0; c < C; ++c)
        for (int col = tid; col < stride; col += 64 * WAVES) wl[c * stride + col] = (col < d) ? a.w[(int64_t)c * d + col] : 0.0f;
    const float* wrow = wl + min(j, C - 1) * stride + 4 * quarter + 16 * s_lo;   // classes past C read the last one; never used
    float bias[4] = {0.f, 0.f, 0.f, 0.f};
    if (KIND == kSoftmax)
        for (int v = 0; v < 4; ++v)
            if (4 * quarter + v < C) bias[v] = a.w[(int64_t)C * d + 4 * quarter + v];
    __syncthreads();

    f32x4 gb = {0.f, 0.f, 0.f, 0.f};   // bias gradient: classes 4 quarter .. + 3 of row j
    int buf = 0;
    for (int64_t r = r0; r < r1; r += 16, buf ^= 1) {
        const int64_t row = r + j;
        const bool valid = row < r1;
        float target = 0.0f;
        int lab = 0;
        if constexpr (KIND == kLsq) target = valid ? reinterpret_cast<const float*>(a.y)[row] : 0.0f;
        else lab = valid ? reinterpret_cast<const int32_t*>(a.y)[row] : 0;
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const f32x4 wv = *reinterpret_cast<const f32x4*>(wrow + 16 * u);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.x, xq[u].x, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.y, xq[u].y, acc1, 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.z, xq[u].z, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.w, xq[u].w, acc1, 0, 0, 0);
            if (u % 2 == 1) __builtin_amdgcn_sched_barrier(0);      // no more weights fetched ahead than registers are left
        }
        f32x4 z4 = acc0 + acc1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WAVES > 1) {
            part[(buf * WAVES + wave) * 64 + lane] = z4;
            __syncthreads();
            z4 = part[buf * WAVES * 64 + lane];
#pragma unroll 1
            for (int w = 1; w < WAVES; ++w) z4 += part[(buf * WAVES + w) * 64 + lane];    // (unrolled, its reads push the rows out of the registers)
        }
        // this lane: classes 4 quarter .. + 3 of row j
        f32x4 dl = {0.f, 0.f, 0.f, 0.f};
        if constexpr (KIND == kLsq) {
            dl.x = (valid && quarter == 0) ? z4.x - target : 0.0f;
        } else {
            float z[4], zmax = -3.0e38f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                z[v] = z4[v] + bias[v];
                if (4 * quarter + v < C) zmax = fmaxf(zmax, z[v]);
            }
            zmax = fmaxf(zmax, __shfl_xor(zmax, 16, 64));
            zmax = fmaxf(zmax, __shfl_xor(zmax, 32, 64));
            float den = 0.0f;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * quarter + v < C) { dl[v] = expf(z[v] - zmax); den += dl[v]; }
            den += __shfl_xor(den, 16, 64);
            den += __shfl_xor(den, 32, 64);
            const float inv = 1.0f / den;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                dl[v] = (valid && 4 * quarter + v < C) ? dl[v] * inv - (4 * quarter + v == lab ? 1.0f : 0.0f) : 0.0f;
            gb += dl;
        }
        // delta with the lane on the class (the buffer is the wave's own: no barrier)
        *reinterpret_cast<f32x4*>(turn + j * FG_TSTRIDE + 4 * quarter) = dl;
        wave_fence();
        float dv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) dv[v] = turn[(4 * quarter + v) * FG_TSTRIDE + j];

        const __amdgpu_buffer_rsrc_t rs = rows_at(r + 16);
        __builtin_amdgcn_sched_barrier(0);
        // A block is turned over through the same buffer: a wave's LDS accesses happen in order, so nothing is waited for but
        // the turned block, and that one is on its way while the block before it is contracted.
        auto turn_over = [&](int u) {
            wave_fence();
            *reinterpret_cast<f32x4*>(turn + j * FG_TSTRIDE + 4 * quarter) = xq[u];
            wave_fence();
            f32x4 t;
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = turn[(4 * quarter + v) * FG_TSTRIDE + j];
            return t;
        };
        f32x4 t = turn_over(0);
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            f32x4 next = t;
            if (u + 1 < BL) next = turn_over(u + 1);
            __builtin_amdgcn_sched_barrier(0);
            xq[u] = load(rs, u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 4; ++v) g[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[v], t[v], g[u], 0, 0, 0);
            t = next;
        }
        wave_fence();
    }

    float* dst = a.partial + (int64_t)blockIdx.x * C * (d + 1);
#pragma unroll
    for (int u = 0; u < BL; ++u) {
        const int col = 16 * (s_lo + u) + j;
        if (col < d) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * quarter + v < C) dst[(int64_t)(4 * quarter + v) * (d + 1) + col] = g[u][v];
        }
    }
    if (KIND == kSoftmax && wave == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float s = gb[v];
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (j == 0 && 4 * quarter + v < C) dst[(int64_t)(4 * quarter + v) * (d + 1) + d] = s;
        }
    }
}

// 16 samples per workgroup and turn; thread -> (sample tid / 16, columns 4 (tid % 16) + 64 k .. + 3)
template <int KIND>
__global__ __launch_bounds__(256) void full_grad_delta_kernel(FullGradArgs a) {
    const int tid = threadIdx.x, part = tid & 15, rl = tid >> 4;
    const int d = a.d, C = a.C;
    for (int64_t n0 = (int64_t)blockIdx.x * 16; n0 < a.N; n0 += (int64_t)gridDim.x * 16) {
        const int64_t n = n0 + rl;
        const bool have = n < a.N;
        float z[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) z[c] = 0.0f;
        if (have) {
            const float* xr = a.X + n * d;
            for (int col = 4 * part; col < d; col += 64) {
                const f32x4 xv = *reinterpret_cast<const f32x4*>(xr + col);
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    if (c < C) {
                        const float* wp = a.w + (int64_t)c * d + col;      // a replica's parameters need not be 16-byte aligned
                        z[c] += (xv.x * wp[0] + xv.y * wp[1]) + (xv.z * wp[2] + xv.w * wp[3]);
                    }
                }
            }
        }
        // the 16 parts of a sample sit in 16 neighbouring lanes
#pragma unroll
        for (int c = 0; c < 16; ++c)
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) z[c] += __shfl_xor(z[c], o, 64);
        if (have && part == 0) {
            float dl[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) dl[c] = 0.0f;
            if (KIND == kLsq) {
                dl[0] = z[0] - reinterpret_cast<const float*>(a.y)[n];
            } else {
                const int lab = reinterpret_cast<const int32_t*>(a.y)[n];
                float zmax = -3.0e38f;
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (c < C) { z[c] += a.w[(int64_t)C * d + c]; zmax = fmaxf(zmax, z[c]); }
                float den = 0.0f;
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (c < C) { dl[c] = expf(z[c] - zmax); den += dl[c]; }
                const float inv = 1.0f / den;
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (c < C) dl[c] = dl[c] * inv - (c == lab ? 1.0f : 0.0f);
            }
            f32x4* dst = reinterpret_cast<f32x4*>(a.delta + n * 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[q] = f32x4{dl[4 * q], dl[4 * q + 1], dl[4 * q + 2], dl[4 * q + 3]};
        }
    }
}

// workgroup = (block of 256 columns, chunk of samples); column d is the bias column (x = 1)
__global__ __launch_bounds__(256) void full_grad_partial_kernel(FullGradArgs a) {
    __shared__ float ds[64][16];
    const int tid = threadIdx.x;
    const int col = blockIdx.x * 256 + tid;
    const int d = a.d, C = a.C;
    const int64_t r0 = (int64_t)blockIdx.y * a.chunk_rows, r1 = min(a.N, r0 + a.chunk_rows);
    float acc[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[c] = 0.0f;
    for (int64_t b0 = r0; b0 < r1; b0 += 64) {
        const int cnt = (int)min<int64_t>(64, r1 - b0);
        __syncthreads();
        for (int q = tid; q < cnt * 16; q += 256) ds[q >> 4][q & 15] = a.delta[b0 * 16 + q];
        __syncthreads();
        if (col <= d) {
            for (int s = 0; s < cnt; ++s) {
                const float x = (col < d) ? a.X[(b0 + s) * d + col] : 1.0f;
#pragma unroll
                for (int c = 0; c < 16; ++c) acc[c] += ds[s][c] * x;
            }
        }
    }
    if (col <= d)
        for (int c = 0; c < C; ++c) a.partial[((int64_t)blockIdx.y * C + c) * (d + 1) + col] = acc[c];
}

// 64 outputs per workgroup; each of the sixteen waves adds a sixteenth of the partial gradients (fp64, in order), their sums
// are added in order.  What bounds it is the chain of loads of a wave, eight in flight at a time: with four waves and 256
// partial gradients it was eight round trips to memory deep, now it is two (256 partial gradients of 4096 x 256 least
// squares: 5.3 -> 3.3 us; those of d = 3072, 10 classes, 31 MB: 10 us either way).
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(64 * kReduceWaves) void full_grad_reduce_kernel(FullGradArgs a) {
    __shared__ double parts[kReduceWaves][64];
    const int d = a.d, C = a.C, lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int total = C * (d + 1);
    const int q = blockIdx.x * 64 + lane;
    const int per = (a.chunks + kReduceWaves - 1) / kReduceWaves, ch0 = part * per, ch1 = min(a.chunks, ch0 + per);
    double sum = 0.0;
    if (q < total) {
        const float* src = a.partial + q;
        int ch = ch0;
        for (; ch + 8 <= ch1; ch += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = src[(int64_t)(ch + i) * total];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += (double)v[i];
        }
        for (; ch < ch1; ++ch) sum += (double)src[(int64_t)ch * total];
    }
    parts[part][lane] = sum;
    __syncthreads();
    if (part == 0 && q < total) {
        sum = parts[0][lane];
#pragma unroll
        for (int p = 1; p < kReduceWaves; ++p) sum += parts[p][lane];
        const int c = q / (d + 1), col = q - c * (d + 1);
        const float gr = (float)(sum / (double)a.N);
        if (col < d) store_result(a.out + (int64_t)c * d + col, gr);
        else if (a.kind == kSoftmax) store_result(a.out + (int64_t)C * d + c, gr);
    }
    // (one wave has written)
    if (part == 0) {
        results_arrived();
        if (lane == 0) signal_done(a.done, gridDim.x);
    }
}

// Launch shape of the fused kernel for one data set: waves per workgroup and blocks per wave (waves = 0 if it does not
// take the shape), workgroups, LDS.  As many workgroups as row blocks until every CU has one, more, up to what is
// resident, only where each has at least four row blocks (every workgroup costs the reduction a partial gradient).
struct FusedShape { int waves, bl, groups; int64_t rows; size_t lds; int stride; };
FusedShape fused_shape(int64_t N, int d, int C, int cus) {
    FusedShape f{};
    f.waves = d <= 64 ? 2 : (d <= 128 ? 4 : 8);
    f.bl = d <= 256 ? 2 : (d <= 512 ? 4 : (d <= 768 ? 6 : (d <= 1024 ? 8 : (d + 511) / 512 * 4)));
    f.stride = 16 * f.waves * f.bl + 4;     // stride % 64 == 4 or 36: the 16 class rows of a fetch hit different bank groups
    f.lds = sizeof(float) * ((size_t)C * f.stride + (size_t)f.waves * (2 * 64 * 4 + 16 * FG_TSTRIDE));
    if (f.bl > 24 || f.lds > 160 * 1024) { f.waves = 0; return f; }
    const int64_t nrb = (N + 15) / 16;
    const int64_t waves_per_cu = f.bl <= 8 ? 16 : 8;       // by registers
    int64_t resident = std::min<int64_t>(waves_per_cu / f.waves, (int64_t)(160 * 1024 / f.lds)) * cus;
    resident = std::max<int64_t>(1, std::min(resident, kStaticScratchFloats / ((int64_t)C * (d + 1))));
    const int64_t groups = std::min(std::min(nrb, std::max<int64_t>(cus, nrb / 4)), resident);
    f.rows = (N + groups - 1) / groups;
    f.groups = (int)((N + f.rows - 1) / f.rows);
    return f;
}

template <int KIND, int WAVES, int BL>
hipError_t launch_fused(const FullGradArgs& a, const FusedShape& f, hipStream_t s) {
    const hipError_t e = hipFuncSetAttribute((const void*)full_grad_fused_kernel<KIND, WAVES, BL>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)f.lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((full_grad_fused_kernel<KIND, WAVES, BL>), dim3(f.groups), dim3(64 * WAVES), f.lds, s, a);
    return hipGetLastError();
}
template <int KIND>
hipError_t launch_fused(const FullGradArgs& a, const FusedShape& f, hipStream_t s) {
    if (f.waves == 2) return launch_fused<KIND, 2, 2>(a, f, s);
    if (f.waves == 4) return launch_fused<KIND, 4, 2>(a, f, s);
    switch (f.bl) {
    case 2: return launch_fused<KIND, 8, 2>(a, f, s);
    case 4: return launch_fused<KIND, 8, 4>(a, f, s);
    case 6: return launch_fused<KIND, 8, 6>(a, f, s);
    case 8: return launch_fused<KIND, 8, 8>(a, f, s);
    case 12: return launch_fused<KIND, 8, 12>(a, f, s);
    case 16: return launch_fused<KIND, 8, 16>(a, f, s);
    case 20: return launch_fused<KIND, 8, 20>(a, f, s);
    default: return launch_fused<KIND, 8, 24>(a, f, s);
    }
}

}  // namespace

bool full_grad_supports(int kind, int d, int C) {
    return (kind == kLsq || kind == kSoftmax) && d % 4 == 0 && C >= 1 && C <= 16;
}

int64_t full_grad_scratch_floats(int64_t N, int d, int C, int* chunks_out) {
    const int chunks = (int)std::max<int64_t>(1, std::min<int64_t>(64, (N + 255) / 256));
    if (chunks_out) *chunks_out = chunks;
    return N * 16 + (int64_t)chunks * C * (d + 1);
}

// What launch_full_grad writes to its work area.
int64_t full_grad_work_floats(int64_t N, int d, int C, int cus) {
    const FusedShape f = fused_shape(N, d, C, cus);
    return f.waves > 0 ? (int64_t)f.groups * C * (d + 1) : full_grad_scratch_floats(N, d, C, nullptr);
}

int64_t full_grad_static_scratch_floats() { return kStaticLimitFloats; }

// Looks up, once per device, where that device keeps its copy of the static scratch array.  Called with the device
// current (ssgd_create does, for every context of a linear model), so that the entry point itself only reads the table.
hipError_t full_grad_static_scratch_prepare() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] != nullptr) return hipSuccess;
    float* p = nullptr;
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
    return hipSuccess;
}

// The current device's copy of the static scratch array, nullptr before full_grad_static_scratch_prepare ran there.
float* full_grad_static_scratch() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[dev];
}

// `work`: full_grad_work_floats floats of device memory; `out`: |w| floats the device can write
hipError_t launch_full_grad(int kind, const float* X, const void* y, int64_t N, int d, int C, const float* w,
                            float* work, float* out, int cus, hipStream_t s, const Done& done) {
    FullGradArgs a{};
    a.done = done;
    a.X = X; a.y = y; a.w = w; a.N = N; a.d = d; a.C = C; a.kind = kind; a.out = out;
    const FusedShape f = fused_shape(N, d, C, cus);
    if (f.waves > 0) {
        a.partial = work; a.chunks = f.groups; a.chunk_rows = f.rows; a.stride = f.stride;
        const hipError_t e = kind == kLsq ? launch_fused<kLsq>(a, f, s) : launch_fused<kSoftmax>(a, f, s);
        if (e != hipSuccess) return e;
    } else {
        (void)full_grad_scratch_floats(N, d, C, &a.chunks);
        a.chunk_rows = ((N + a.chunks - 1) / a.chunks + 63) / 64 * 64;
        a.delta = work; a.partial = work + N * 16;
        const int blocks = (int)std::min<int64_t>((N + 15) / 16, (int64_t)std::max(1, cus) * 8);
        if (kind == kLsq) hipLaunchKernelGGL(full_grad_delta_kernel<kLsq>, dim3(blocks), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(full_grad_delta_kernel<kSoftmax>, dim3(blocks), dim3(256), 0, s, a);
        hipLaunchKernelGGL(full_grad_partial_kernel, dim3((d + 1 + 255) / 256, a.chunks), dim3(256), 0, s, a);
    }
    hipLaunchKernelGGL(full_grad_reduce_kernel, dim3((C * (d + 1) + 63) / 64), dim3(64 * kReduceWaves), 0, s, a);
    return hipGetLastError();
}

}  // namespace ssgd
