// Chunked-prefill attention over the quantized cache (the prefill stage also reads the KV
// cache, Sec. 2.1; the sliding window of Sec. 6.1 applies per query), for chunks of more than
// 64 rows (query token, query head) per KV head; attention_rows.hip takes the shorter ones
// and prompts of a few pages (prefill_row_tiles).
//
// A workgroup of eight waves takes a block of up to 256 rows, or 128: consecutive query tokens
// of one sequence's chunk times the query heads of one KV head.  It reads every page of the
// keys those rows can see once, four pages (64 keys) a step: the pages are dequantized by
// all threads into LDS tiles of high and low fp16 parts under a power of two per step (x = hi + lo
// to about 2^-22 |x|, and 2^-35 of the step's largest element),
// middle readings from the nibbles first, then every COO entry overwrites its element with
// its true value (the engine's zero-insert and merge of Sec. 5.2), and each wave contracts
// the tiles with its own 32 rows on v_mfma_f32_32x32x16_f16:
//   S^T = K_hi Q^T + K_lo Q^T (the query is fp16 already)
//   O^T += V_hi P_hi + V_hi P_lo + V_lo P_hi, accumulated in fp32.
// Blocks of 256 rows: a wave takes both halves (32 keys) of a step.  Blocks of 128: waves w
// and w + 4 share 32 rows and take a half each; their sums meet in LDS at the end.
// Both products are formed transposed, so a row's scores, probabilities, softmax state and
// outputs stay on two lanes: lane q + 32 f holds rows 8 b + 4 f + r (b, r < 4) of column q of
// a result, and those keys are exactly the k-slots it owes the value product, because the
// value tiles are stored in that order.
//
// The tiles are double-buffered: while the waves contract a step's pages, they dequantize the
// next step's, so a step needs two barriers:
//   half 0 of step s, dense readings of s + 1, loads of s + 2 |
//   half 1 of step s, COO entries of s + 1, token constants of s + 2 |
// Of the two waves that share a SIMD one contracts first and the other dequantizes first, so
// that matrix and vector work overlap.
// Long prefixes are split into page ranges whose partials the log-sum-exp combine merges.
//
// Bound: vector issue beside the matrix cores.  A step of four pages takes a CU about 15.2 K
// cycles for 256 rows: on each SIMD 8.7 K of vector issue (dequantization 40 %, softmax 25 %)
// and 5.1 K of matrix work, which together leave little (two waves a SIMD overlap them only in
// part), the LDS active 5.6 K.  Measured, against 128-row blocks that walked 16-key pages
// through four barriers on v_mfma_f32_16x16x16_f16: 16 chunks of 64 tokens at 32K keys, 32 query
// / 8 KV heads, 3030 -> 1670 us (1870 over a cold card's first ten calls); eight prompts of
// 200-4096 tokens 2605 -> 1400 us; one prompt of 1000 tokens at head_dim 64 172 -> 70 us.
#include "coo_walk.h"
#include "oaken_internal.h"
#include "prefill_internal.h"

#include <hip/hip_fp16.h>

namespace oaken {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int P = kPage;
constexpr int kStage = 512;   // staged COO bytes per record (longer streams: read from HBM)

__device__ __forceinline__ f16v mfma(u4 a, u4 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// (x0, x1) as fp16 pairs: hi nearest, lo the nearest fp16 of the exact rest.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    const h2 h = __builtin_convertvector((f2{x0, x1}), h2);
    const h2 l = __builtin_convertvector((f2{x0 - (float)h[0], x1 - (float)h[1]}), h2);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// Workgroup barrier for data handed over through LDS: waits for the wave's LDS operations
// only.  (__syncthreads also waits for every global load in flight, which exposed a step's
// whole memory latency twice: 2650 us instead of 1940 for 16 chunks of 256 rows at 32K keys.)
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value of lane l ^ 32.
__device__ __forceinline__ float other_half(float v) {
    const int x = __float_as_int(v);
    const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return __int_as_float((threadIdx.x & 32) ? a[0] : a[1]);
}

// Four pages (64 tokens), dequantized.  Keys: D / 8 blocks of eight channels, each [token] 16
// bytes (16 bytes of padding per block spread the writers over the banks).  Values: D / 32
// tiles of [page][half f][channel] 16 bytes = the tokens 4 f .. 4 f + 3 and 8 + 4 f .. + 3.
constexpr int SP = 4;         // pages per step
constexpr int NW = 8, NT = 64 * NW;
template <int D>
struct PfTiles {
    static constexpr int KB = SP * P * 16 + 16, KP = (D / 8) * KB, VP = D * SP * 32;
    __align__(16) uint8_t k[2][KP];   // high, low parts
    __align__(16) uint8_t v[2][VP];
};
template <int D>
struct PfSmem {
    PfTiles<D> tl[2];
    __align__(16) uint8_t dense[2][SP * P * D / 2];   // nibbles of the pages' keys, values
    __align__(16) uint8_t coo[2][SP][kStage];         // COO bytes of keys, values, by page
    __align__(16) float4 kc[SP * P];                  // key tokens: base, Delta, Gp / 8
    __align__(16) float vc[SP][3][P];                 // value tokens: the same, by page
    __align__(8) int ex[4][2];                                     // exponents of a step's keys, values (step mod 4)
};

// KH = 1: 32 rows per wave; KH = 2: waves w and w + 4 share 32 rows, a half of the keys each.
template <int D, bool PG, int KH>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void prefill_kernel(PrefillArgs a) {
    constexpr Layout LY = PG ? make_layout_paged(P, D) : make_layout(P, D);
    constexpr int UP = 2 * D;                         // dwords of a page's keys (or values)
    constexpr int IT = SP * UP / NT;
    constexpr int NC = D / 64, KST = D / 16, VT = D / 32;
    constexpr int SPCAP = P * D;
    static_assert(SP * UP % NT == 0 && UP % 64 == 0, "whole passes, a wave's units in one page");

    __shared__ PfSmem<D> S;
    const int tid = threadIdx.x, lane = tid & 63, q32 = tid & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int type = wave & 1;        // COO work: even waves the keys, odd waves the values
    const bool late = wave >= 4;      // (waves w and w + 4 share a SIMD)

    // the KV head fastest: the row blocks of one head, which read the same pages, then share
    // an XCD's L2 when the heads are a multiple of eight
    const int h = (int)(blockIdx.x % (uint32_t)a.H);
    const uint32_t rest = blockIdx.x / (uint32_t)a.H;
    const int blk = (int)(rest % (uint32_t)a.max_row_blocks), split = (int)(rest / (uint32_t)a.max_row_blocks);
    const int4 rb = a.row_blocks[blk];                // (both loads at once: the list has room for every blk)
    if (blk >= *a.n_row_blocks) return;               // (uniform)
    const int s = rb.x, tok = rb.y, n_tok = rb.z, pos = rb.w, G = a.Hq / a.H;   // sequence, first token, tokens, position
    const int n_rows = n_tok * G;
    const int end = pos + n_tok;                      // keys any row sees
    const int lo_first = a.window > 0 ? max(0, pos + 1 - a.window) : 0;
    const int pg0 = lo_first / P + split * a.pages_per_split;
    const int pg_end = min((end + P - 1) / P, pg0 + a.pages_per_split);
    const int n_pages = max(0, pg_end - pg0), n_steps = (n_pages + SP - 1) / SP;

    // the range's block ids, one per lane, in two tables of 64 pages (even and odd ones)
    // (loaded whatever the range's end: no wait to merge a loaded and a default value)
    auto ld_blocks = [&](int k64) {
        return a.block_table[(int64_t)s * a.max_blocks + max(0, min(pg0 + 64 * k64 + lane, pg_end - 1))];
    };
    int ids0 = ld_blocks(0), ids1 = ld_blocks(1);
    // page k's key record and valid slots (an absent page reads record 0, whose bytes are
    // masked by its zero valid slots)
    auto record = [&](int k, int& nv) {
        const int b = (k >> 6) & 1 ? __builtin_amdgcn_readlane(ids1, k & 63) : __builtin_amdgcn_readlane(ids0, k & 63);
        const bool ok = k < n_pages && b >= 0 && b < a.num_blocks;
        nv = ok ? max(0, min(P, end - (pg0 + k) * P)) : 0;
        return a.pool + (ok ? ((int64_t)b * a.H + h) * 2 * a.stride : 0);
    };
    float th[4];                      // thresholds of the wave's record type
#pragma unroll
    for (int k = 0; k < 4; ++k) th[k] = fin(a.thr[(h * 2 + type) * 4 + k]);

    // ---- loads of a step ------------------------------------------------------------------
    // Every thread: dwords of the dense nibbles.  Lane = token (page lane >> 4, slot lane & 15)
    // of the wave's record type: counts and metadata.  Waves 0-3: 16 COO bytes of page
    // 2 (wave / 2) + (lane >> 5) of the type.
    struct Step {
        const uint8_t *tok, *str;     // the lane's token's record; that of its COO stream
        const uint8_t* dn[IT];        // the dense nibbles' key records
        int nv4, nv;                  // valid slots of the four pages (a byte each), of the lane's
        uint32_t counts;              // the dword of the lane's token's
        int2 tab;                     // first sparse pages of the stream
    };
    const int slot = lane & 15, pgl = lane >> 4;
    auto open_step = [&](int st) {
        Step x;
        int n0, n1, n2, n3;
        const uint8_t *r0 = record(SP * st, n0), *r1 = record(SP * st + 1, n1);
        const uint8_t *r2 = record(SP * st + 2, n2), *r3 = record(SP * st + 3, n3);
        const int64_t own = type ? a.stride : 0;
        const int64_t ga = (pgl & 1) ? r1 - r0 : 0, gb = (pgl & 1) ? r3 - r0 : r2 - r0;
        x.tok = r0 + own + ((pgl & 2) ? gb : ga);
        const bool up = (wave & 2) != 0;              // (uniform)
        const int64_t sa = up ? r2 - r0 : 0, sb = up ? r3 - r0 : r1 - r0;
        x.str = r0 + own + (hf ? sb : sa);
        x.nv4 = n0 | (n1 << 8) | (n2 << 16) | (n3 << 24);
        x.nv = (x.nv4 >> (8 * pgl)) & 0xff;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            int n;
            x.dn[it] = record(SP * st + (wave * 64 + NT * it) / UP, n);
        }
        // (a whole dword: nothing to extend, so nothing waits for it before its use)
        x.counts = *reinterpret_cast<const uint32_t*>(x.tok + LY.counts + (NC * slot & ~3));
        x.tab = int2{0, 0};
        if constexpr (PG) x.tab = *reinterpret_cast<const int2*>(x.str + LY.sparse);
        return x;
    };
    auto sparse_page = [&](int32_t entry) -> const uint8_t* {
        const int id = entry - 1;     // (clamped: a stale entry can only misread)
        return a.spool + (int64_t)((id >= 0 && id < a.spages) ? id : 0) * kSparsePage;
    };
    uint32_t kd[IT], vd[IT], run = 0;
    uint4 coo = make_uint4(0, 0, 0, 0);
    Meta meta{0, 0, 0};
    bool fit = true;
    // (every load is issued whatever the wave: the compiler's wait counts then stay exact, and no
    // wait for one load drains the others)
    auto ld_step = [&](const Step& x) {
        const uint32_t cw = slot < x.nv ? x.counts >> (8 * (NC * slot & 3)) : 0u;
        const int c0 = (int)(cw & 0xffu), c1 = NC == 2 ? (int)((cw >> 8) & 0xffu) : 0;
        const int incl = row_scan16(c0 + c1);
        // a 64-value chunk has at most 64 entries; larger counts are not a valid record
        Run r;
        r.st = min(incl - c0 - c1, SPCAP);
        r.c0 = min(c0, 64);
        r.cnt = max(0, min(r.c0 + min(c1, 64), SPCAP - r.st));
        run = pack_run(r);
        const int u0 = __builtin_amdgcn_readlane(incl, 15), u1 = __builtin_amdgcn_readlane(incl, 31);
        const int u2 = __builtin_amdgcn_readlane(incl, 47), u3 = __builtin_amdgcn_readlane(incl, 63);
        fit = max(max(u0, u1), max(u2, u3)) <= kStage;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const uint8_t* p = x.dn[it] + LY.dense + 4 * ((wave * 64 + NT * it) % UP + lane);
            kd[it] = *reinterpret_cast<const uint32_t*>(p);
            vd[it] = *reinterpret_cast<const uint32_t*>(p + a.stride);
        }
        const uint32_t* m = reinterpret_cast<const uint32_t*>(x.tok + LY.meta + 12 * slot);
        meta = Meta{m[0], m[1], m[2]};
        const int o = q32 * 16, ua = (wave & 2) ? u2 : u0, ub = (wave & 2) ? u3 : u1;
        const bool in = wave < 4 && o < (hf ? ub : ua);           // (past the stream: its first bytes again)
        if constexpr (PG) {
            const uint8_t* sp = sparse_page(o < kSparsePage || !in ? x.tab.x : x.tab.y);
            coo = ld16(sp + (in ? o & (kSparsePage - 1) : 0));
        } else {
            coo = ld16(x.str + LY.sparse + (in ? o : 0));
        }
    };

    // ---- token constants -------------------------------------------------------------------
    // A step's keys (values) x enter the tiles as x 2^(15 - e), |x| < 2^e for all of them: no part
    // reaches fp16's largest value (a stored 65504 reads back as up to 65536), and the low parts
    // of small values are not lost below its smallest.  e follows the step's largest bound; it
    // stays while that lies within five bits below, so that the outputs, in units of
    // 2^(e - 15), are rescaled rarely.  Waves 0 and 1 form it (in every wave, for its own
    // entries, the eight prompts of 200-4096 tokens took 1474 us instead of 1397).
    float i_m = 0.0f, i_d = 0.0f, o_m = 0.0f, o_d = 0.0f;   // the lane's token's Min, Delta (inner, outer)
    int ex = 15;                      // (waves 0, 1)
    auto within = [](float t) { return fabsf(t) < 65536.0f ? fabsf(t) : 0.0f; };   // (no value lies past others)
    const float th_m = fmaxf(within(th[1]), within(th[2])), th_o = fmaxf(within(th[0]), within(th[3]));
    uint32_t run_c = 0;
    bool fit_c = true;
    const uint8_t* mine_c = a.pool;   // the record of the lane's token
    auto token_phase = [&](const Step& x, int st) {
        const bool vt = slot < x.nv;                  // (other slots read as zeros)
        const Tok T = token_consts(meta, th);
        i_m = h2f(meta.w0 & 0xffffu);
        i_d = h2f(meta.w0 >> 16);
        o_m = h2f(meta.w2 & 0xffffu);
        o_d = h2f(meta.w2 >> 16);
        run_c = run;
        fit_c = fit;
        mine_c = x.tok;
        if (wave >= 2) return;
        // (non-negative floats, ordered as integers; the maximum itself only where e moves)
        auto bits = [](float v) { return __float_as_int(v); };
        int most = max(max(bits(fmaf(15.0f, i_d, i_m)), bits(th_o + fmaf(15.0f, o_d, o_m))),
                       bits(th_m + fmaf(7.0f, T.dm, h2f(meta.w1 & 0xffffu))));
        most = vt ? most : 0;
        if (__builtin_amdgcn_ballot_w64(most >= (127 + ex) << 23) ||
            !__builtin_amdgcn_ballot_w64(most >= (127 + ex - 5) << 23)) {
            const int row = row_max(most);
            const int top = max(max(__builtin_amdgcn_readlane(row, 15), __builtin_amdgcn_readlane(row, 31)),
                                max(__builtin_amdgcn_readlane(row, 47), __builtin_amdgcn_readlane(row, 63)));
            if (top > 0) ex = min(max((top >> 23) - 126, -24), 16);
        }
        const float unit = __int_as_float((127 + 15 - ex) << 23);
        const float base = vt ? unit * T.base : 0.0f, dm = vt ? unit * T.dm : 0.0f;
        const float gp = vt ? 0.125f * unit * T.gp : 0.0f;
        if (type == 0) {
            S.kc[lane] = make_float4(base, dm, gp, 0.0f);
        } else {
            S.vc[pgl][0][slot] = base;
            S.vc[pgl][1][slot] = dm;
            S.vc[pgl][2][slot] = gp;
        }
        if (lane == 0) S.ex[st & 3][type] = ex;
    };

    // ---- dense readings into the tiles, nibbles and COO bytes into the staging area ----------
    auto dense_phase = [&](PfTiles<D>& L) {
        if (wave < 4) *reinterpret_cast<uint4*>(&S.coo[type][(wave & 2) + hf][q32 * 16]) = coo;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int u = tid + NT * it;
            *reinterpret_cast<uint32_t*>(&S.dense[0][4 * u]) = kd[it];
            *reinterpret_cast<uint32_t*>(&S.dense[1][4 * u]) = vd[it];
            // eight readings x = base + u Delta + h Gp of a dword's nibbles
            auto readings = [&](uint32_t d, auto base, auto dm, auto gp, u4& hi, u4& lo) {
                const uint32_t d4 = d >> 4;
                const uint32_t e = d & 0x0f0f0f0fu, o = d4 & 0x0f0f0f0fu, eh = d & 0x08080808u, oh = d4 & 0x08080808u;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const float x0 = fmaf((float)byte_at(e, b), dm(2 * b), fmaf((float)byte_at(eh, b), gp(2 * b), base(2 * b)));
                    const float x1 = fmaf((float)byte_at(o, b), dm(2 * b + 1),
                                          fmaf((float)byte_at(oh, b), gp(2 * b + 1), base(2 * b + 1)));
                    uint32_t x, y;
                    split2(x0, x1, x, y);
                    hi[b] = x;
                    lo[b] = y;
                }
            };
            u4 hi, lo;
            {
                const int cb = u % (D / 8), t = u / (D / 8);
                const float4 c = S.kc[t];
                readings(kd[it], [&](int) { return c.x; }, [&](int) { return c.y; }, [&](int) { return c.z; }, hi, lo);
                const int at = cb * PfTiles<D>::KB + t * 16;
                *reinterpret_cast<u4*>(&L.k[0][at]) = hi;
                *reinterpret_cast<u4*>(&L.k[1][at]) = lo;
            }
            {
                const int pg = u / UP, ch = (u >> 1) % D, half = u & 1;
                float cb[8], cd[8], cg[8];
#pragma unroll
                for (int k = 0; k < 8; k += 4) {
                    const float4 x = *reinterpret_cast<const float4*>(&S.vc[pg][0][8 * half + k]);
                    const float4 y = *reinterpret_cast<const float4*>(&S.vc[pg][1][8 * half + k]);
                    const float4 z = *reinterpret_cast<const float4*>(&S.vc[pg][2][8 * half + k]);
                    cb[k] = x.x; cb[k + 1] = x.y; cb[k + 2] = x.z; cb[k + 3] = x.w;
                    cd[k] = y.x; cd[k + 1] = y.y; cd[k + 2] = y.z; cd[k + 3] = y.w;
                    cg[k] = z.x; cg[k + 1] = z.y; cg[k + 2] = z.z; cg[k + 3] = z.w;
                }
                readings(vd[it], [&](int k) { return cb[k]; }, [&](int k) { return cd[k]; }, [&](int k) { return cg[k]; }, hi, lo);
                // tokens 8 half + 0..3 belong to f = 0, + 4..7 to f = 1
                const int at = (((ch >> 5) * SP + pg) * 2) * 512 + (ch & 31) * 16 + half * 8;
                *reinterpret_cast<uint2*>(&L.v[0][at]) = make_uint2(hi[0], hi[1]);
                *reinterpret_cast<uint2*>(&L.v[0][at + 512]) = make_uint2(hi[2], hi[3]);
                *reinterpret_cast<uint2*>(&L.v[1][at]) = make_uint2(lo[0], lo[1]);
                *reinterpret_cast<uint2*>(&L.v[1][at + 512]) = make_uint2(lo[2], lo[3]);
            }
        }
    };

    // ---- COO entries: their true values over the middle readings ------------------------------
    // Lane = token; the four waves of a type share its entries.
    auto entry_phase = [&](PfTiles<D>& L, int st) {
        const float unit = __int_as_float((127 + 15 - __builtin_amdgcn_readfirstlane(S.ex[st & 3][type])) << 23);
        const float t_lo = unit * th[0], t_hi = unit * th[3];
        i_m *= unit; i_d *= unit; o_m *= unit; o_d *= unit;
        const Run r = unpack_run(run_c);
        const int per = (r.cnt + 3) >> 2, first = per * (wave >> 1);
        const int n = min(per, r.cnt - first);
        auto far_coo = [&](int e) -> uint32_t {       // (streams past the staging area)
            const int at = r.st + e;
            if constexpr (PG) {
                return sparse_page(reinterpret_cast<const int32_t*>(mine_c + LY.sparse)[at / kSparsePage])[at % kSparsePage];
            } else {
                return mine_c[LY.sparse + at];
            }
        };
        const uint8_t* near = &S.coo[type][pgl][r.st];
        // th +- (Min + c Delta), c counted from the threshold: nothing to cancel in tokens with an
        // extreme outlier, whose scores dominate long contexts (as B + n K, 32K keys were 3.2e-6
        // off the 64-bit result instead of 7.7e-7)
        auto value = [&](uint32_t en, uint32_t nib, _Float16& hi, _Float16& lo) {
            const bool outer = (en & 0x40u) != 0;
            const uint32_t low = ~(uint32_t)((int)(en << 24) >> 31);   // all ones on the lower side
            const float mag = fmaf((float)(nib ^ (low & 15u)), outer ? o_d : i_d, outer ? o_m : i_m);
            const float edge = outer ? (low ? t_lo : t_hi) : 0.0f;
            const float x = edge + __uint_as_float(__float_as_uint(mag) ^ (low & 0x80000000u));
            hi = (_Float16)x;
            lo = (_Float16)(x - (float)hi);
        };
        // NE entries of the lane's run from its kk-th; past its end the last one again
        auto some = [&](auto NE_, int kk, auto byte) {
            constexpr int NE = decltype(NE_)::value;
            uint32_t en[NE], ch[NE], nib[NE];
            int at[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e) en[e] = byte(first + min(kk + e, n - 1));
#pragma unroll
            for (int e = 0; e < NE; ++e) ch[e] = (en[e] & 63u) | (NC == 2 && first + min(kk + e, n - 1) >= r.c0 ? 64u : 0u);
            if (type == 0) {
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    nib[e] = ((uint32_t)S.dense[0][lane * (D / 2) + (ch[e] >> 1)] >> (4 * (ch[e] & 1u))) & 15u;
                    at[e] = (int)((ch[e] >> 3) * PfTiles<D>::KB + lane * 16 + (ch[e] & 7u) * 2);
                }
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    _Float16 hi, lo;
                    value(en[e], nib[e], hi, lo);
                    *reinterpret_cast<_Float16*>(&L.k[0][at[e]]) = hi;
                    *reinterpret_cast<_Float16*>(&L.k[1][at[e]]) = lo;
                }
            } else {
                const int vat = pgl * 1024 + ((slot >> 2) & 1) * 512 + (slot >> 3) * 8 + (slot & 3) * 2;
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    nib[e] = ((uint32_t)S.dense[1][pgl * (P * D / 2) + ch[e] * 8 + (slot >> 1)] >> (4 * (slot & 1))) & 15u;
                    at[e] = (int)((ch[e] >> 5) * (SP * 1024) + (ch[e] & 31u) * 16) + vat;
                }
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    _Float16 hi, lo;
                    value(en[e], nib[e], hi, lo);
                    *reinterpret_cast<_Float16*>(&L.v[0][at[e]]) = hi;
                    *reinterpret_cast<_Float16*>(&L.v[1][at[e]]) = lo;
                }
            }
        };
        // (four, then two at a time: at the usual outlier share of 10 % a token's quarter holds
        // three entries, five in the fullest token of a step)
        if (fit_c) {
            auto near_coo = [&](int e) -> uint32_t { return near[e]; };
            if (n > 0) some(std::integral_constant<int, 4>{}, 0, near_coo);
            for (int kk = 4; kk < n; kk += 2) some(std::integral_constant<int, 2>{}, kk, near_coo);
        } else {
            for (int kk = 0; kk < n; ++kk) some(std::integral_constant<int, 1>{}, kk, far_coo);
        }
    };

    // (the first step's bytes are requested before the queries: small calls wait for both at once)
    Step sn = open_step(0), snn = open_step(1);
    if (n_steps > 0) ld_step(sn);

    // ---- rows -----------------------------------------------------------------------------------
    // scores in base-2 units; a negative scale goes into the query's signs
    const float sl2 = fabsf(a.scale) * 1.44269504088896341f;
    const uint32_t flip = a.scale < 0.0f ? 0x80008000u : 0u;
    const int wrow = 32 * (KH == 2 ? wave & 3 : wave);  // the wave's first row
    const int row0 = wrow + q32;                        // this lane's row of the block
    const bool rok = row0 < n_rows, work = wrow < n_rows;   // (work: uniform per wave)
    const int tk = rok ? row0 / G : 0, hd = rok ? row0 % G : 0;
    const int rpos = pos + tk, rlo = a.window > 0 ? max(0, rpos + 1 - a.window) : 0;
    const int64_t row = (int64_t)(tok + tk) * a.Hq + h * G + hd;
    u4 bq[KST];
    {
        const uint16_t* qp = a.q + row * D + 8 * hf;
        const bool al = (reinterpret_cast<uintptr_t>(a.q) & 15) == 0;   // (uniform)
#pragma unroll
        for (int k = 0; k < KST; ++k) {
            u4 x = u4{0, 0, 0, 0};
            if (rok) {
                if (al) {
                    x = *reinterpret_cast<const u4*>(qp + 16 * k);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = (uint32_t)qp[16 * k + 2 * e] | ((uint32_t)qp[16 * k + 2 * e + 1] << 16);
                }
            }
            bq[k] = x ^ flip;
        }
    }
    const int vis_hi = pos;           // keys up to here are seen by every row
    const int vis_lo = a.window > 0 ? max(0, end - a.window) : 0;
    float m = -INFINITY, l = 0.0f;    // reference of the exponentials (lane's row), sum (lane's keys)
    int eo = 15;                      // the outputs' units: 2^(eo - 15)
    f16v o[VT];
#pragma unroll
    for (int n = 0; n < VT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[n][r] = 0.0f;

    // ---- one half (32 keys) of a step ----------------------------------------------------------------
    // Scores: lane (q, f) gets keys 8 b + 4 f + r of its row (the small low parts first).  Online
    // softmax: the reference moves only when a maximum passed it by 2^8 (the probabilities, 64
    // times theirs, stay below 2^14).
    u4 ph[2], pl[2];
    auto scores = [&](const PfTiles<D>& L, int hb, int st, int nv4) {
        const int2 e2 = *reinterpret_cast<const int2*>(&S.ex[st & 3][0]);
        f16v sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
#pragma unroll
        for (int part = 1; part >= 0; --part)
#pragma unroll
            for (int k = 0; k < KST; ++k)
                sc = mfma(*reinterpret_cast<const u4*>(&L.k[part][(2 * k + hf) * PfTiles<D>::KB + (32 * hb + q32) * 16]), bq[k], sc);
        const int k0 = (pg0 + SP * st + 2 * hb) * P;
        const int na = (nv4 >> (16 * hb)) & 0xff, nb = (nv4 >> (16 * hb + 8)) & 0xff;
        const bool full = min(na, nb) == P && k0 + 31 <= vis_hi && k0 >= vis_lo;
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (!full) {
                const int kp = k0 + 8 * (r >> 2) + 4 * hf + (r & 3);
                const bool in = (kp & (P - 1)) < (r < 8 ? na : nb);
                if (!(rok && in && kp <= rpos && kp >= rlo)) sc[r] = -INFINITY;
            }
            mx = fmaxf(mx, sc[r]);
        }
        mx = fmaxf(mx, other_half(mx));
        // (the step's unit is a power of two: as good as unscaled keys)
        const int ek = __builtin_amdgcn_readfirstlane(e2.x), ev = __builtin_amdgcn_readfirstlane(e2.y);
        const float sls = sl2 * __int_as_float((127 - 15 + ek) << 23);
        mx = mx == -INFINITY ? mx : sls * mx;
        const bool up = mx > m + 8.0f;
        if (__builtin_amdgcn_ballot_w64(up || ev != eo)) {
            float alpha = up ? __builtin_amdgcn_exp2f(m - mx) : 1.0f;
            m = up ? mx : m;
            l *= alpha;
            alpha *= __int_as_float((127 + eo - ev) << 23);   // (into this step's units)
            eo = ev;
#pragma unroll
            for (int n = 0; n < VT; ++n) o[n] *= alpha;
        }
        const float ms = (m == -INFINITY) ? 0.0f : m - 6.0f;   // (no visible key yet: l and o stay 0)
        float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            float e0 = fmaf(sls, sc[r], -ms), e1 = fmaf(sls, sc[r + 1], -ms);
            if (!full) {   // (a zero scale times a hidden key's -inf)
                e0 = sc[r] == -INFINITY ? -INFINITY : e0;
                e1 = sc[r + 1] == -INFINITY ? -INFINITY : e1;
            }
            const float p0 = __builtin_amdgcn_exp2f(e0), p1 = __builtin_amdgcn_exp2f(e1);
            sum[(r >> 1) & 3] += p0 + p1;
            uint32_t x, y;
            split2(p0, p1, x, y);
            ph[r >> 3][(r & 7) >> 1] = x;
            pl[r >> 3][(r & 7) >> 1] = y;
        }
        l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    };
    // Outputs: k-slots (page, f, e) as the lane holds them.
    auto outputs = [&](const PfTiles<D>& L, int hb) {
#pragma unroll
        for (int n = 0; n < VT; ++n)
#pragma unroll
            for (int pg = 0; pg < 2; ++pg) {
                const int at = ((n * SP + 2 * hb + pg) * 2 + hf) * 512 + q32 * 16;
                const u4 vh = *reinterpret_cast<const u4*>(&L.v[0][at]), vl = *reinterpret_cast<const u4*>(&L.v[1][at]);
                o[n] = mfma(vl, ph[pg], o[n]);
                o[n] = mfma(vh, pl[pg], o[n]);
                o[n] = mfma(vh, ph[pg], o[n]);
            }
    };

    // ---- pipeline ----------------------------------------------------------------------------------
    int nv4 = sn.nv4;                 // valid slots of the pages in the current tiles
    if (n_steps > 0) {
        token_phase(sn, 0);
        lds_barrier();
        dense_phase(S.tl[0]);
        ld_step(snn);
        lds_barrier();
        entry_phase(S.tl[0], 0);
        sn = snn;
        snn = open_step(2);
        token_phase(sn, 1);
        lds_barrier();
    }
    for (int st = 0; st < n_steps; ++st) {
        // (here: sn = step st + 1, its bytes in flight; snn = step st + 2, its counts in flight)
        if ((st & 15) == 0 && st > 0) {   // (the block table just done takes the pages after next)
            if ((st >> 4) & 1) ids0 = ld_blocks((st >> 4) + 1);
            else ids1 = ld_blocks((st >> 4) + 1);
        }
        const PfTiles<D>& Tc = S.tl[st & 1];
        PfTiles<D>& Tn = S.tl[(st & 1) ^ 1];
        const bool next = st + 1 < n_steps;
        const int hb = wave >> 2;         // (KH = 2: the wave's half)
        // (a wave that contracts goes before its SIMD's other wave: its matrix instructions are
        // few and long, and the other's vector work fills the gaps)
        auto contract_a = [&]() {
            if (!work) return;
            __builtin_amdgcn_s_setprio(1);
            scores(Tc, KH == 2 ? hb : 0, st, nv4);
            if constexpr (KH == 1) outputs(Tc, 0);
            __builtin_amdgcn_s_setprio(0);
        };
        auto contract_b = [&]() {
            if (!work) return;
            __builtin_amdgcn_s_setprio(1);
            if constexpr (KH == 1) scores(Tc, 1, st, nv4);
            outputs(Tc, KH == 2 ? hb : 1);
            __builtin_amdgcn_s_setprio(0);
        };
        if (!late) contract_a();
        if (next) {
            dense_phase(Tn);
            ld_step(snn);
        }
        if (late) contract_a();
        lds_barrier();
        if (!late) contract_b();
        const int nv4_n = sn.nv4;
        if (next) {
            entry_phase(Tn, st + 1);
            sn = snn;
            snn = open_step(st + 3);
            token_phase(sn, st + 2);
        }
        if (late) contract_b();
        nv4 = nv4_n;
        lds_barrier();
    }

    // ---- outputs, or this range's partials ------------------------------------------------------------
    l += other_half(l);
    const float back = __int_as_float((127 - 15 + eo) << 23);   // (waves that share rows end on the same step)
    if constexpr (KH == 2) {
        // waves 4-7 hand their rows' sums to waves 0-3 (the tiles' LDS; all waves are past the
        // last barrier)
        float* X = reinterpret_cast<float*>(&S) + (wave & 3) * (16 * VT + 2) * 64 + lane;
        if (late && work) {
            X[0] = m;
            X[64] = l;
#pragma unroll
            for (int n = 0; n < VT; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) X[(2 + 16 * n + r) * 64] = o[n][r];
        }
        lds_barrier();
        if (late) return;
        if (work) {
            const float m2 = X[0], l2 = X[64], M = fmaxf(m, m2);
            const float f1 = l > 0.0f ? __builtin_amdgcn_exp2f(m - M) : 0.0f, f2_ = l2 > 0.0f ? __builtin_amdgcn_exp2f(m2 - M) : 0.0f;
            l = l * f1 + l2 * f2_;
            m = M;
#pragma unroll
            for (int n = 0; n < VT; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[n][r] = o[n][r] * f1 + X[(2 + 16 * n + r) * 64] * f2_;
        }
    }
    if (!rok) return;
    if (a.n_splits == 1) {
        const float inv = l > 0.0f ? back / l : 0.0f;
        float* dst = a.out + row * D;
#pragma unroll
        for (int n = 0; n < VT; ++n)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *reinterpret_cast<float4*>(&dst[32 * n + 8 * b + 4 * hf]) =
                    make_float4(o[n][4 * b] * inv, o[n][4 * b + 1] * inv, o[n][4 * b + 2] * inv, o[n][4 * b + 3] * inv);
    } else {
        float* pp = a.partial + (row * a.n_splits + split) * (D + 2);   // (8-byte aligned rows)
#pragma unroll
        for (int n = 0; n < VT; ++n)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                *reinterpret_cast<float2*>(&pp[32 * n + 8 * b + 4 * hf]) = make_float2(back * o[n][4 * b], back * o[n][4 * b + 1]);
                *reinterpret_cast<float2*>(&pp[32 * n + 8 * b + 4 * hf + 2]) = make_float2(back * o[n][4 * b + 2], back * o[n][4 * b + 3]);
            }
        if (hf == 0) {
            pp[D] = (m - 6.0f) * 0.693147180559945309f;
            pp[D + 1] = l;
        }
    }
}

// Row blocks: sequence s's chunk of C_s tokens is cut into ceil(C_s / T) blocks of T tokens.  They
// are listed backwards: a chunk's last block sees the most keys, goes out first, and the
// short ones fill the tail.  An entry holds all that a block's workgroup needs before its
// block table, so that nothing is looked up by sequence there.  One workgroup, sequences in
// rounds of 1024 with a prefix sum of the block counts (within waves, then over them).
__global__ __launch_bounds__(1024) void prefill_blocks_kernel(const int32_t* cu_tokens, const int32_t* start_pos,
                                                             int n_seqs, int T, int max_row_blocks, int4* row_blocks,
                                                             int32_t* n_row_blocks) {
    __shared__ int wave_sum[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int s0 = 0; s0 < n_seqs; s0 += 1024) {
        const int s = n_seqs - 1 - s0 - (int)threadIdx.x;
        const int tok0 = s >= 0 ? cu_tokens[s] : 0, C = s >= 0 ? max(0, cu_tokens[s + 1] - tok0) : 0;
        const int start = s >= 0 ? start_pos[s] : 0;
        const int nb = (C + T - 1) / T;
        int incl = nb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d, 64);
            incl += lane >= d ? v : 0;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            before += w < wave ? wave_sum[w] : 0;
            all += wave_sum[w];
        }
        const int first = base + before + incl - nb;
        for (int j = 0; j < nb; ++j) {
            const int i0 = (nb - 1 - j) * T;
            if (first + j < max_row_blocks) row_blocks[first + j] = make_int4(s, tok0 + i0, min(T, C - i0), start + i0);
        }
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) *n_row_blocks = min(base, max_row_blocks);
}

}  // namespace

PrefillPlan plan_prefill(int32_t n_tokens, int32_t n_seqs, int32_t n_q_heads, int32_t n_kv_heads, int32_t max_seq_len,
                         int32_t window, int32_t row_tiles) {
    PrefillPlan p{};
    const int G = n_q_heads / n_kv_heads;
    p.row_tiles = row_tiles;
    p.tokens_per_block = std::max(1, 16 * row_tiles / G);
    // pages a block can see: those of its own tokens and everything before them, or of a window
    // of W before its first token, which may start inside a page
    int64_t pages = ((int64_t)max_seq_len + kPage - 1) / kPage;
    if (window > 0) pages = std::min<int64_t>(pages, ((int64_t)window + p.tokens_per_block + kPage - 1) / kPage + 1);
    // row blocks of all KV heads; every sequence with tokens starts one of its own
    const int64_t units = std::max<int64_t>((n_tokens + p.tokens_per_block - 1) / p.tokens_per_block,
                                            std::min(n_seqs, n_tokens)) * n_kv_heads;
    auto parts = [](int64_t all, int64_t n) { return (all + n - 1) / n; };
    if (row_tiles <= 2) {
        // Single waves.  A range's partials (520 bytes a row, written and read) cost about as much
        // as two pages of work.  Where there are waves enough, ranges of ten pages or more
        // even them out; where they leave slots of the chip empty, ranges of two pages or more
        // fill it and cut the chain of pages, the longer the more waves there are.  Measured at 40
        // heads: 16 chunks of 16 tokens at 256 keys, 640 waves, 54 us in ranges of two pages, 45 in
        // four, 64 in one range; 64 chunks, 2560 waves, 187, 130, 104 us.
        const int64_t even = std::min(parts(row_tiles == 1 ? 6144 : 4096, units), pages / 10);
        const int64_t fill = std::min((row_tiles == 1 ? 3072 : 2048) / units, pages / std::max<int64_t>(2, units / 256));
        p.pages_per_split = (int32_t)parts(pages, std::max<int64_t>({1, even, fill}));
    } else {
        // Workgroups that fill a CU each; the partials stay small beside the work of 32 pages, and
        // of 8 where the chip is not full.  Whole ranges of that (a ninth page alone would cost 496
        // blocks 126 MB of partials), or a shorter last one where few blocks leave most CUs idle.
        const int64_t least = std::min<int64_t>(32, std::max<int64_t>(8, units * pages / 512));
        const int64_t most = units < 64 ? parts(pages, least) : std::max<int64_t>(1, pages / least);
        p.pages_per_split = (int32_t)(parts(parts(pages, std::min(parts(512, units), most)), SP) * SP);   // (whole steps)
    }
    p.n_splits = (int32_t)parts(pages, p.pages_per_split);
    return p;
}

hipError_t launch_prefill(const PrefillArgs& a, int d, int4* row_blocks, int32_t* n_row_blocks, hipStream_t st) {
    hipLaunchKernelGGL(prefill_blocks_kernel, dim3(1), dim3(1024), 0, st, a.cu_tokens, a.start_pos, a.n_seqs, a.tokens_per_block,
                       a.max_row_blocks, row_blocks, n_row_blocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.row_tiles <= 2) return launch_rows(a, d, st);
    const int64_t n = (int64_t)a.max_row_blocks * a.H * a.n_splits;
    if (n <= 0 || n > 0x7fffffff || (a.row_tiles != 8 && a.row_tiles != 16)) return hipErrorInvalidValue;
    const bool pg = a.spool != nullptr;
    auto go = [&](auto half, auto whole) {
        hipLaunchKernelGGL(a.row_tiles == 8 ? half : whole, dim3((uint32_t)n), dim3(NT), 0, st, a);
    };
    if (d == 128)
        pg ? go(prefill_kernel<128, true, 2>, prefill_kernel<128, true, 1>)
           : go(prefill_kernel<128, false, 2>, prefill_kernel<128, false, 1>);
    else if (d == 64)
        pg ? go(prefill_kernel<64, true, 2>, prefill_kernel<64, true, 1>)
           : go(prefill_kernel<64, false, 2>, prefill_kernel<64, false, 1>);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace oaken
