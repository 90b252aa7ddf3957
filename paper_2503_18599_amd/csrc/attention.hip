// Batched decode attention over the Oaken-quantized paged cache (Oaken Sec. 2.1): the plan
// that cuts sequences into page ranges, the launch of the kernel that serves a head shape
// (attention_mfma.hip at head_dim 128, attention_rows.hip at 64) and the log-sum-exp
// combine of the ranges.
#include "oaken_internal.h"
#include "prefill_internal.h"

#include <hip/hip_fp16.h>

namespace oaken {
namespace {

constexpr int kMaxG = 8;            // query heads per KV head

// Log-sum-exp merge of the page ranges' partials (m, l, o) of one (sequence, query head)
// row.  NW waves share the row's ranges (wave w takes ranges w, w + NW, ...), each lane
// D / 64 channels, with a running maximum (the sums are rescaled when it grows), unrolled
// so that several ranges' loads are in flight together; ranges with l = 0 are skipped.
// Decode rows (seq_lens given) read only the ranges that hold keys of their sequence:
// those starting before its last page (the others are empty by construction), so a batch
// of mixed lengths reads no partials of the empty ranges.  The waves' (M, den, num) then
// meet in LDS.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_combine_kernel(AttnArgs a) {
    constexpr int V = D / 64;
    const int64_t row = blockIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const float* pp = a.partial + row * a.n_splits * (D + 2);
    int n_used = a.n_splits;
    if (a.seq_lens) {
        // the page ranges of the attention kernels: range k starts at page lo / P + k * pps
        const int s = (int)(row / a.Hq);
        const int L = max(0, min(a.seq_lens[s], min(a.max_seq_len, a.max_blocks * kPage)));
        const int n_pages = (L + kPage - 1) / kPage;
        const int lo = (a.window > 0 && L > a.window) ? L - a.window : 0;
        n_used = min(a.n_splits, (n_pages - lo / kPage + a.pages_per_split - 1) / a.pages_per_split);
    }
    float M = -INFINITY, den = 0.0f, num[V];
#pragma unroll
    for (int v = 0; v < V; ++v) num[v] = 0.0f;
#pragma unroll 4
    for (int k = w; k < n_used; k += NW) {
        const float* pk = pp + (int64_t)k * (D + 2);
        const float m = pk[D], l = pk[D + 1];
        float o[V];
        if constexpr (V == 2) {
            const float2 t = *reinterpret_cast<const float2*>(pk + 2 * lane);   // (D + 2) * 4 is a multiple of 8
            o[0] = t.x;
            o[1] = t.y;
        } else {
            o[0] = pk[lane];
        }
        if (l > 0.0f) {
            const float Mn = fmaxf(M, m);
            const float r = __expf(M - Mn), e = __expf(m - Mn);
#pragma unroll
            for (int v = 0; v < V; ++v) num[v] = fmaf(num[v], r, e * o[v]);
            den = fmaf(den, r, e * l);
            M = Mn;
        }
    }
    if constexpr (NW > 1) {
        __shared__ float s_md[NW][2];
        __shared__ float s_num[NW][D];
        if (lane == 0) {
            s_md[w][0] = M;
            s_md[w][1] = den;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) s_num[w][V * lane + v] = num[v];
        __syncthreads();
        if (w != 0) return;
        float Mx = -INFINITY;
#pragma unroll
        for (int x = 0; x < NW; ++x)
            if (s_md[x][1] > 0.0f) Mx = fmaxf(Mx, s_md[x][0]);
        den = 0.0f;
#pragma unroll
        for (int v = 0; v < V; ++v) num[v] = 0.0f;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float r = s_md[x][1] > 0.0f ? __expf(s_md[x][0] - Mx) : 0.0f;
            den = fmaf(s_md[x][1], r, den);
#pragma unroll
            for (int v = 0; v < V; ++v) num[v] = fmaf(s_num[x][V * lane + v], r, num[v]);
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) a.out[row * D + V * lane + v] = (den > 0.0f) ? num[v] / den : 0.0f;
}

}  // namespace

SplitPlan plan_splits(int32_t n_seqs, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                      int32_t max_seq_len) {
    const int G = n_q_heads / n_kv_heads;
    const bool mfma = mfma_attention_supported(head_dim, G);
    const int max_pages = (max_seq_len + kPage - 1) / kPage;
    const int64_t units = (int64_t)n_seqs * n_kv_heads * (mfma ? G / mfma_wave_heads(G) : 1);
    const int64_t target = 4096;   // workgroups that keep 256 CUs busy
    int want = (int)((target + units - 1) / units);
    // Ranges of at least eight pages where the chip is full of them, fewer where it is not: at
    // head_dim 128 one group of four pages (one sequence of 1237 keys over 8 KV heads: 28.2 us
    // with eight pages, 21.5 with four), at 64 two pages.
    const int fit = max((max_pages + want - 1) / want, mfma ? (short_range(units, max_pages, 4, 8) + 3) / 4 * 4
                                                            : short_range(units, max_pages, 2, 8));
    auto plan = [&](int pps) { return SplitPlan{pps, (max_pages + pps - 1) / pps}; };
    if (mfma) return plan(max(min(fit, mfma_score_cap(mfma_wave_heads(G)) / kPage), 1));
    // Head dimension 64: ranges of at most 32 pages even out batches of mixed lengths, as long
    // as their partials stay small beside the 32 MiB that the allocation-free call has for them.
    const SplitPlan even = plan(min(fit, 32));
    if ((int64_t)n_seqs * n_q_heads * even.n_splits * (head_dim + 2) * 4 <= (16 << 20)) return even;
    // Larger calls: ranges of 8192 / G keys.  No kernel needs that limit; it keeps the partials, and
    // with them the calls that the allocation-free entry point takes, what they have always been
    // (256 sequences of 512-8192 keys, 32 query / 8 KV heads: 866 us in its 128 pages, 752 in
    // 32 with 34 MiB of partials; 64 query heads 797 and 763).
    constexpr int kLongRange = 8192;
    return plan(max(min(fit, kLongRange / (kPage * G)), 1));
}

// Waves per row of the combine: about eight ranges per wave, at most eight waves.
template <int D>
hipError_t launch_combine_d(const AttnArgs& a, hipStream_t st) {
    const dim3 grid((uint32_t)((int64_t)a.n_seqs * a.Hq));
    if (a.n_splits <= 8)
        hipLaunchKernelGGL((attn_combine_kernel<D, 1>), grid, dim3(64), 0, st, a);
    else if (a.n_splits <= 16)
        hipLaunchKernelGGL((attn_combine_kernel<D, 2>), grid, dim3(128), 0, st, a);
    else if (a.n_splits <= 32)
        hipLaunchKernelGGL((attn_combine_kernel<D, 4>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((attn_combine_kernel<D, 8>), grid, dim3(512), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_combine(const AttnArgs& a, int d, hipStream_t st) {
    if (d == 64) return launch_combine_d<64>(a, st);
    if (d == 128) return launch_combine_d<128>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_attention(const AttnArgs& args, int d, hipStream_t st) {
    AttnArgs a = args;
    const int G = a.Hq / a.H;
    if (G < 1 || G > kMaxG) return hipErrorInvalidValue;
    const bool mfma = mfma_attention_supported(d, G);
    a.wave_heads = mfma ? mfma_wave_heads(G) : G;
    a.head_parts = G / a.wave_heads;
    const uint32_t grid = attn_grid(a);
    if (grid == 0) return hipErrorInvalidValue;
    if (mfma) {
        hipError_t e = launch_attention_mfma(a, st);
        if (e != hipSuccess || a.n_splits == 1) return e;
        return launch_combine(a, d, st);
    }
    if (d != 64) return hipErrorInvalidValue;
    PrefillArgs r{};
    r.pool = a.pool;
    r.thr = a.thr;
    r.q = a.q;
    r.block_table = a.block_table;
    r.seq_lens = a.seq_lens;
    r.out = a.out;
    r.partial = a.partial;
    r.stride = a.stride;
    r.num_blocks = a.num_blocks;
    r.H = a.H;
    r.Hq = a.Hq;
    r.max_blocks = a.max_blocks;
    r.n_seqs = r.n_tokens = r.max_row_blocks = a.n_seqs;
    r.max_seq_len = a.max_seq_len;
    r.tokens_per_block = r.row_tiles = 1;
    r.pages_per_split = a.pages_per_split;
    r.n_splits = a.n_splits;
    r.window = a.window;
    r.scale = a.scale;
    hipError_t e = launch_rows(r, d, st);
    if (e != hipSuccess || a.n_splits == 1) return e;
    return launch_combine(a, d, st);
}

}  // namespace oaken
