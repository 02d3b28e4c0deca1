// Products with few activation rows, bfloat16: one wavefront multiplies 16 columns of a K-contiguous weight matrix
// with a few fragments of 16 rows, both operands straight from memory to registers.
#pragma once
#include "kernels.h"

namespace unipool {

namespace {

// The two MFMA operands of 16 columns x 64 indices from two loads that cover whole 128-byte lines: lane l of lo
// (hi) holds 16-byte chunk l / 8 of row l % 8 (8 + l % 8).  even: chunks 0 2 4 6, odd: chunks 1 3 5 7, lane l with
// row l % 16; half of the lanes keep what they loaded, the others take it from the lane eight further on.
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void few_fragments(const u32x4v& lo, const u32x4v& hi, bf16x8& even, bf16x8& odd) {
    constexpr int kRowRor8 = 0x128;
    union { u32x4v u; bf16x8 v; } e, o;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        e.u[i] = __builtin_amdgcn_update_dpp(lo[i], hi[i], kRowRor8, 0xf, 0xc, false);
        o.u[i] = __builtin_amdgcn_update_dpp(hi[i], lo[i], kRowRor8, 0xf, 0x3, false);
    }
    even = e.v;
    odd = o.v;
}

// Sum over steps [s0, s1) of 64 indices for R row fragments, NF weight fragments.  D steps are in flight.
// wp: this lane's chunk of columns 0..7 (hi: 8 columns further on), xp: this lane's two chunks of a row.
// STREAM: nobody else reads these weights.
template <int NF, int R, int D, bool STREAM>
__device__ __forceinline__ void few_reduce(const bf16* const (&wp)[NF], size_t hi, const bf16* const (&xp)[R], int s0,
                                           int s1, f32x4 (&acc)[NF][R]) {
    u32x4v wq[D][NF][2];
    bf16x8 xq[D][R][2];
#pragma unroll
    for (int f = 0; f < NF; f++)
#pragma unroll
        for (int r = 0; r < R; r++) acc[f][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (s0 >= s1) return;
    auto fetch = [&](int u, int s) {
        const size_t o = (size_t)min(s, s1 - 1) * 64;          // past the end: the last step again, never used
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const u32x4v* src = reinterpret_cast<const u32x4v*>(wp[f] + o + h * hi);
                if constexpr (STREAM) wq[u][f][h] = __builtin_nontemporal_load(src);
                else wq[u][f][h] = *src;
            }
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int h = 0; h < 2; h++) xq[u][r][h] = *reinterpret_cast<const bf16x8*>(xp[r] + o + 8 * h);
    };
    auto multiply = [&](int u) {
#pragma unroll
        for (int f = 0; f < NF; f++) {
            bf16x8 even, odd;
            few_fragments(wq[u][f][0], wq[u][f][1], even, odd);
#pragma unroll
            for (int r = 0; r < R; r++) {
                acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(even, xq[u][r][0], acc[f][r], 0, 0, 0);
                acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(odd, xq[u][r][1], acc[f][r], 0, 0, 0);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < D; u++) fetch(u, s0 + u);
    int s = s0;
    for (; s + D <= s1; s += D) {
#pragma unroll
        for (int u = 0; u < D; u++) {
            multiply(u);
            fetch(u, s + D + u);
        }
    }
#pragma unroll
    for (int u = 0; u < D; u++)
        if (s + u < s1) multiply(u);
}

}  // namespace

}  // namespace unipool
