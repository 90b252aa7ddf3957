// Pieces shared by the kernels that read and write the packed records: a token's
// dequantization constants, its run of COO entries, the wave-local hand-over through LDS
// and the sub-dword operand selects of the entry walks.
#pragma once

#include "oaken_internal.h"

#include <hip/hip_fp16.h>

namespace oaken {
namespace {

__device__ __forceinline__ float h2f(uint32_t b) { return __half2float(__ushort_as_half((uint16_t)b)); }
__device__ __forceinline__ float fin(float x) { return __builtin_isfinite(x) ? x : 0.0f; }

// Inclusive prefix sum within each row of 16 lanes (DPP row shifts).
__device__ __forceinline__ int row_scan16(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    return x;
}

// Running maximum of non-negative integers (or the bits of non-negative floats) along each row
// of 16 lanes (its last lane: the row's).
__device__ __forceinline__ int row_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));
    return v;
}

// Per-token constants of the dequantization (thresholds th = lo_o, lo_i, hi_i, hi_o).
struct Tok {
    float base, dm, gp;   // middle reading: base + u*dm + h*gp
    float b_il, b_ol, b_ih, b_oh, kd_i, kd_o;
};

// The token's 12 metadata bytes (three fp16 pairs Min, Delta: inner, middle, outer).
struct Meta {
    uint32_t w0, w1, w2;
};

__device__ __forceinline__ Tok token_consts(const Meta& mt, const float* th) {
    const uint32_t w0 = mt.w0, w1 = mt.w1, w2 = mt.w2;
    const float mi = h2f(w0 & 0xffff), di = h2f(w0 >> 16);
    const float mm = h2f(w1 & 0xffff), dm = h2f(w1 >> 16);
    const float mo = h2f(w2 & 0xffff), dd = h2f(w2 >> 16);
    Tok T;
    T.base = th[1] - mm - 7.0f * dm;
    T.dm = dm;
    T.gp = th[2] - th[1] + 2.0f * mm - dm;
    T.b_il = -mi - 15.0f * di;
    T.b_ih = mi;
    T.b_ol = th[0] - mo - 15.0f * dd;
    T.b_oh = th[3] + mo;
    T.kd_i = di - dm;
    T.kd_o = dd - dm;
    return T;
}

// Between lanes of one wave (LDS areas that no other wave touches).  The LDS operations of a
// wave execute in issue order, so handing data between its lanes through LDS needs no wait
// at all: only wavefront-scope fences, which keep the compiler from moving memory operations
// across the hand-over and emit no instructions.  (A workgroup barrier would wait for every
// global load in flight and stall the prefetch pipeline; draining the LDS counter would
// stall on every outstanding LDS operation.)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint4 ld16(const uint8_t* p) {
    return *reinterpret_cast<const uint4*>(p);
}

// The COO entries of the lane's token, in stream order: cnt entries from byte st of its
// page's stream, the first c0 of them in chunk 0.  Carried packed in one register: st (bits
// 0-11), c0 (12-19), cnt (20-31).
struct Run {
    int st, c0, cnt;
};
__device__ __forceinline__ uint32_t pack_run(const Run& r) {
    return (uint32_t)r.st | ((uint32_t)r.c0 << 12) | ((uint32_t)r.cnt << 20);
}
__device__ __forceinline__ Run unpack_run(uint32_t x) {
    return Run{(int)(x & 0xfffu), (int)((x >> 12) & 0xffu), (int)(x >> 20)};
}

__device__ __forceinline__ uint32_t byte_at(uint32_t x, int i) { return (x >> (8 * i)) & 0xffu; }

// base | byte i of x, and byte i of x << s, each one VALU operation with a sub-dword
// operand select (i is a constant after unrolling).
#define OAKEN_SDWA_OR(I)                                                                              \
    asm("v_or_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #I " src1_sel:DWORD" \
        : "=v"(r) : "v"(x), "v"(base))
__device__ __forceinline__ uint32_t or_byte(uint32_t x, uint32_t base, int i) {
    uint32_t r;
    switch (i) {
        case 0: OAKEN_SDWA_OR(0); break;
        case 1: OAKEN_SDWA_OR(1); break;
        case 2: OAKEN_SDWA_OR(2); break;
        default: OAKEN_SDWA_OR(3); break;
    }
    return r;
}
#undef OAKEN_SDWA_OR
#define OAKEN_SDWA_SHL(I)                                                                                  \
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_" #I \
        : "=v"(r) : "v"(sh), "v"(x))
__device__ __forceinline__ uint32_t shl_byte(uint32_t x, uint32_t sh, int i) {
    uint32_t r;
    switch (i) {
        case 0: OAKEN_SDWA_SHL(0); break;
        case 1: OAKEN_SDWA_SHL(1); break;
        case 2: OAKEN_SDWA_SHL(2); break;
        default: OAKEN_SDWA_SHL(3); break;
    }
    return r;
}
#undef OAKEN_SDWA_SHL

}  // namespace
}  // namespace oaken
