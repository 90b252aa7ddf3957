// Offline outlier-threshold profiling (Oaken Sec. 4.3, "offline outlier threshold
// profiling"; ratios of Sec. 6.1).
//
// The paper takes topK boundaries per profiling run and averages them.  Here every
// boundary is an exact order statistic of fp16 data, found without sorting: fp16 bit
// patterns map to 16-bit keys whose integer order is the value order, a 4096-bin LDS
// histogram over the keys' high 12 bits finds the bin of a given rank, and a second pass
// over the values counts the low 4 bits of that bin's few members.
#include "oaken_internal.h"

#include <hip/hip_fp16.h>

namespace oaken {
namespace {

constexpr int kCalThreads = 1024;
constexpr int kCalWaves = kCalThreads / 64;
constexpr int kBins = 4096;       // key >> 4
constexpr int kHalf = kBins / 2;  // bins of one sign

// Monotone key for value order: negative patterns are reversed below positive ones.
__device__ inline uint32_t value_key(uint32_t b) {
    return (b & 0x8000u) ? (~b & 0xffffu) : (b | 0x8000u);
}
__device__ inline uint16_t value_key_inverse(uint32_t k) {
    return (k & 0x8000u) ? (uint16_t)(k & 0x7fffu) : (uint16_t)(~k & 0xffffu);
}

// Calls f(bits) for every value of the set [T][d] that starts at src, rows H * d apart.
// VEC: d is a multiple of 8 with at most 8 * kCalThreads values and src is 16-byte aligned:
// a lane takes eight values per load, d / 8 lanes per row.  Other sets: one value per load, all
// lanes busy whatever d (eight runs of 512 tokens x 40 heads x 128, two bytes off an aligned
// address: 104 us, 610 with one row at a time and d lanes busy).
template <bool VEC, class F>
__device__ inline void each_value(const uint16_t* src, int T, int d, int64_t row_stride, F f) {
    if constexpr (VEC) {
        const int cpr = d / 8, rows = kCalThreads / cpr;
        const int r = (int)threadIdx.x / cpr, c = (int)threadIdx.x % cpr;
        if (r >= rows) return;
#pragma unroll 4
        for (int t = r; t < T; t += rows) {
            const uint4 w = *reinterpret_cast<const uint4*>(src + t * row_stride + 8 * c);
            const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                f(x[k] & 0xffffu);
                f(x[k] >> 16);
            }
        }
    } else {
        // value i of the set on lane i mod kCalThreads, whatever d: a step of kCalThreads values is
        // dt rows and dj values
        const int dt = kCalThreads / d, dj = kCalThreads % d;
        int j = (int)threadIdx.x % d;
#pragma unroll 4
        for (int64_t t = (int)threadIdx.x / d; t < T;) {
            f((uint32_t)src[t * row_stride + j]);
            t += dt;
            j += dj;
            if (j >= d) {
                j -= d;
                ++t;
            }
        }
    }
}

// Exclusive prefix sum over the workgroup's threads.
__device__ inline uint64_t block_excl_scan(uint64_t v, uint64_t* s_wave) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o, 64);
        x += lane >= o ? y : 0;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    uint64_t before = 0;
    for (int k = 0; k < wave; ++k) before += s_wave[k];
    __syncthreads();
    return before + x - v;
}

// Three selections per (run, head, K|V): ranks k_o and n-1-k_o in value order, rank k_i-1
// in magnitude order.  A value's magnitude bin m holds the value bins 2048 + m and 2047 - m,
// so one histogram serves all three.
// Bound: LDS atomics (one per value).  With the 256-bin histograms of the high key byte
// (two per value) the bulk of a layer's values falls into some twenty bins, whose lanes
// queue; the 4096 bins spread them over hundreds.  Eight runs of 512 tokens x 40 heads x
// 128 (84 MB): 190 us with those, 2-byte loads and a 64-bit division per value, 46 us now.
template <bool VEC>
__global__ __launch_bounds__(kCalThreads) void calib_select_kernel(CalibArgs a) {
    const int r = blockIdx.x, h = blockIdx.y, which = blockIdx.z;
    const uint16_t* src = (which ? a.v : a.k) + ((int64_t)r * a.T * a.H + h) * a.d;
    const int64_t row_stride = (int64_t)a.H * a.d;

    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t low[3][16];
    __shared__ uint64_t s_wave[kCalWaves];
    __shared__ uint32_t sel[3];
    __shared__ uint64_t rest[3];   // rank within the selected bin

    const int tid = threadIdx.x;
    for (int i = tid; i < kBins; i += kCalThreads) hist[i] = 0;
    if (tid < 48) low[tid / 16][tid % 16] = 0;
    if (tid < 3) sel[tid] = 0, rest[tid] = 0;
    __syncthreads();
    each_value<VEC>(src, a.T, a.d, row_stride, [&](uint32_t b) { atomicAdd(&hist[value_key(b) >> 4], 1u); });
    __syncthreads();

    // the bin of each rank: the thread whose bins [excl, excl + sum) hold it
    constexpr int PER = kBins / kCalThreads;
    {
        uint32_t c[PER];
        uint64_t sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += c[k] = hist[tid * PER + k];
        const uint64_t excl = block_excl_scan(sum, s_wave);
        const uint64_t rank[2] = {(uint64_t)a.k_o, (uint64_t)(a.n - 1 - a.k_o)};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint64_t at = excl;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (rank[q] >= at && rank[q] < at + c[k]) {
                    sel[q] = (uint32_t)(tid * PER + k);
                    rest[q] = rank[q] - at;
                }
                at += c[k];
            }
        }
    }
    {
        constexpr int PERM = kHalf / kCalThreads;
        uint32_t c[PERM];
        uint64_t sum = 0;
#pragma unroll
        for (int k = 0; k < PERM; ++k) {
            const int m = tid * PERM + k;
            sum += c[k] = hist[kHalf + m] + hist[kHalf - 1 - m];
        }
        uint64_t at = block_excl_scan(sum, s_wave);
        const uint64_t rank = a.k_i > 0 ? (uint64_t)(a.k_i - 1) : 0u;
#pragma unroll
        for (int k = 0; k < PERM; ++k) {
            if (rank >= at && rank < at + c[k]) {
                sel[2] = (uint32_t)(tid * PERM + k);
                rest[2] = rank - at;
            }
            at += c[k];
        }
    }
    __syncthreads();
    const uint32_t b0 = sel[0], b1 = sel[1], b2 = sel[2];
    each_value<VEC>(src, a.T, a.d, row_stride, [&](uint32_t b) {
        const uint32_t kv = value_key(b), km = b & 0x7fffu;
        if ((kv >> 4) == b0) atomicAdd(&low[0][kv & 15u], 1u);
        if ((kv >> 4) == b1) atomicAdd(&low[1][kv & 15u], 1u);
        if ((km >> 4) == b2) atomicAdd(&low[2][km & 15u], 1u);
    });
    __syncthreads();
    if (tid < 3) {
        uint64_t at = 0;
        uint32_t bin = 15;
        for (int k = 0; k < 16; ++k) {
            if (at + low[tid][k] > rest[tid]) {
                bin = (uint32_t)k;
                break;
            }
            at += low[tid][k];
        }
        const uint32_t key = (sel[tid] << 4) | bin;
        const uint16_t bits = tid < 2 ? value_key_inverse(key) : (uint16_t)key;
        float* o = a.per_run + (((int64_t)r * a.H + h) * 2 + which) * 3;
        o[tid] = (tid < 2 || a.k_i > 0) ? __half2float(__ushort_as_half(bits)) : 0.0f;
    }
}

// fp64 mean over runs in run order, one fp32 rounding, ordering repair, -0 -> +0.
__global__ void calib_average_kernel(CalibArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;   // (head, which)
    if (i >= a.H * 2) return;
    double s_lo = 0.0, s_hi = 0.0, s_t = 0.0;
#pragma unroll 8
    for (int r = 0; r < a.R; ++r) {
        const float* o = a.per_run + ((int64_t)r * a.H * 2 + i) * 3;
        s_lo += (double)o[0];
        s_hi += (double)o[1];
        s_t += (double)o[2];
    }
    const float lo_o = (float)(s_lo / (double)a.R);
    const float hi_o = (float)(s_hi / (double)a.R);
    const float t = (float)(s_t / (double)a.R);
    float lo_i = fminf(fmaxf(-t, lo_o), hi_o);
    float hi_i = fmaxf(fminf(t, hi_o), lo_i);
    float v[4] = {lo_o, lo_i, hi_i, hi_o};
    for (int k = 0; k < 4; ++k) a.thr_out[i * 4 + k] = (v[k] == 0.0f) ? 0.0f : v[k];
}

}  // namespace

hipError_t launch_calibrate(const CalibArgs& a, hipStream_t st) {
    // sixteen-byte loads where rows are whole chunks and every row is aligned to them
    const bool vec = a.d % 8 == 0 && a.d <= 8 * kCalThreads &&
                     ((reinterpret_cast<uintptr_t>(a.k) | reinterpret_cast<uintptr_t>(a.v)) & 15) == 0;
    if (vec)
        hipLaunchKernelGGL(calib_select_kernel<true>, dim3(a.R, a.H, 2), dim3(kCalThreads), 0, st, a);
    else
        hipLaunchKernelGGL(calib_select_kernel<false>, dim3(a.R, a.H, 2), dim3(kCalThreads), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(calib_average_kernel, dim3((a.H * 2 + 63) / 64), dim3(64), 0, st, a);
    return hipGetLastError();
}

}  // namespace oaken
