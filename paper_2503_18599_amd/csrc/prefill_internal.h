// Private declarations of the chunked-prefill attention (attention_prefill.hip, api.hip),
// kept apart from the decode-attention declarations.
#pragma once

#include "oaken_internal.h"

namespace oaken {

// Chunked prefill (attention_prefill.hip): row blocks of (query token, query head) rows of
// one sequence's chunk and one KV head, each reading its pages once.
struct PrefillArgs {
    const uint8_t* pool;
    const float* thr;             // [H][2][4]
    const uint16_t* q;            // fp16 bits [n_tokens][Hq][d]
    const int32_t* block_table;   // [n_seqs][max_blocks]
    const int32_t* start_pos;     // [n_seqs]
    const int32_t* cu_tokens;     // [n_seqs + 1]
    const int4* row_blocks;       // per row block: sequence, first token, tokens, the first's position
    const int32_t* n_row_blocks;  // number of row blocks (device)
    float* out;                   // fp32 [n_tokens][Hq][d]
    float* partial;               // [n_tokens][Hq][n_splits][d + 2] when n_splits > 1
    int64_t stride;
    int32_t num_blocks, H, Hq, max_blocks, n_seqs, n_tokens, max_seq_len;
    int32_t tokens_per_block, max_row_blocks, pages_per_split, n_splits, window;
    float scale;
    const uint8_t* spool;         // on-demand sparse pages (nullptr: fixed records)
    int32_t spages;
    int32_t row_tiles;            // 16-row tiles per block (1, 2, 8 or 16)
    const int32_t* seq_lens;      // decode: one row block per sequence, at its last position (row_blocks unused)
};
struct PrefillPlan {
    int32_t tokens_per_block, pages_per_split, n_splits, row_tiles;
};
// More sequences never plan more ranges: the plan of one sequence bounds the workspace.
PrefillPlan plan_prefill(int32_t n_tokens, int32_t n_seqs, int32_t n_q_heads, int32_t n_kv_heads, int32_t max_seq_len,
                         int32_t window, int32_t row_tiles);
constexpr int32_t kRowTiles[] = {1, 2, 8, 16};
// The 16-row tiles a block takes for chunks of about n_tokens / n_seqs tokens over contexts of
// up to max_seq_len (blocks then hold that many rows at most: longer chunks get more blocks).
// Up to 64 rows, one wave per 16 or 32 (16 chunks of 40 and 64 tokens x 40 heads at 2048 keys: 470
// and 468 us in waves, 499 and 501 in workgroups; 30 single tokens beside two prompts of 512:
// 312 us, 474).  With more, waves of 32 rows at 0.74 us of a CU per page each against workgroups
// that dequantize a page once for 128 rows (1.3 us a page) or 256 (1.7 us) but take some 10 us to
// fill their pipeline, one per CU (head_dim 128; at 64 all of them cost about two thirds).  A
// chunk's blocks see its keys up to their own tokens; where the waves fill the chip several times
// over (four rounds of 2048) only their average counts, else the longest (256 prompts of 30-100
// tokens, 32 / 8 heads: 205 us in waves, 249 in workgroups; 60 prompts: 70 and 65).
inline int32_t prefill_row_tiles(int32_t n_tokens, int32_t n_seqs, int32_t n_q_heads, int32_t n_kv_heads,
                                 int32_t max_seq_len, int32_t window) {
    const int64_t chunk = ((int64_t)n_tokens + n_seqs - 1) / std::max<int32_t>(1, n_seqs);
    const int64_t G = n_q_heads / n_kv_heads, rows = chunk * G, waves = (rows + 31) / 32;
    if (rows <= 64) return rows <= 16 ? 1 : 2;
    const int64_t keys = window > 0 ? std::min<int64_t>(max_seq_len, window + chunk) : max_seq_len;
    const bool full = waves * n_seqs * n_kv_heads >= 4 * 2048;
    auto pages = [&](int64_t block_rows) {
        const int64_t hidden = full ? std::max<int64_t>(0, chunk - block_rows / G) / 2 : 0;
        return (keys - hidden + kPage - 1) / kPage;
    };
    const int64_t big = rows <= 128 ? 1000 + 130 * pages(128) : (rows + 255) / 256 * (1000 + 170 * pages(256));
    return 74 * waves * pages(32) < big ? 2 : rows <= 128 ? 8 : 16;
}
hipError_t launch_prefill(const PrefillArgs& a, int d, int4* row_blocks, int32_t* n_row_blocks, hipStream_t st);
// One wave per block of up to 16 or 32 rows (row_tiles 1, 2; attention_rows.hip).
hipError_t launch_rows(const PrefillArgs& a, int d, hipStream_t st);

}  // namespace oaken
