// Products with few activation rows, bfloat16: one wavefront multiplies 16 columns of a K-contiguous weight matrix
// with a few fragments of 16 rows, both operands straight from memory to registers.  A sum runs over K in slices of 32
// indices in ascending order, lane group g with indices 8 g .. 8 g + 7 of a slice: the order of the tile kernels, so a
// row's result has the same bits whichever of them computed it.
#pragma once
#include "kernels.h"

namespace unipool {

namespace {

// The two MFMA operands of 16 columns x 64 indices from two loads that cover whole 128-byte lines: lane l of lo (hi)
// holds a 16-byte chunk of row l % 8 (8 + l % 8): chunk j in the lanes with l / 8 = 2 j, chunk 4 + j in those with
// 2 j + 1.  first: chunks 0 to 3, second: chunks 4 to 7, lane l with row l % 16 and chunk l / 16; half of the lanes keep
// what they loaded, the others take it from the lane eight further on.
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int few_chunk(int lane) { return (lane >> 4) + ((lane >> 3) & 1) * 4; }
__device__ __forceinline__ void few_fragments(const u32x4v& lo, const u32x4v& hi, bf16x8& first, bf16x8& second) {
    constexpr int kRowRor8 = 0x128;
    union { u32x4v u; bf16x8 v; } e, o;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        e.u[i] = __builtin_amdgcn_update_dpp(lo[i], hi[i], kRowRor8, 0xf, 0xc, false);
        o.u[i] = __builtin_amdgcn_update_dpp(hi[i], lo[i], kRowRor8, 0xf, 0x3, false);
    }
    first = e.v;
    second = o.v;
}

// Sum over ns >= 1 steps of 64 indices for R row fragments, NF weight fragments.  D steps are in flight.
// wp: this lane's chunk of columns 0..7 (hi: 8 columns further on), xp: this lane's chunk of a row's first slice.
// STREAM: these weights will not be read again soon.
template <int NF, int R, int D, bool STREAM>
__device__ __forceinline__ void few_reduce(const bf16* const (&wp)[NF], size_t hi, const bf16* const (&xp)[R], int ns,
                                           f32x4 (&acc)[NF][R]) {
    u32x4v wq[D][NF][2];
    bf16x8 xq[D][R][2];
#pragma unroll
    for (int f = 0; f < NF; f++)
#pragma unroll
        for (int r = 0; r < R; r++) acc[f][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int u, int s) {
        const size_t o = (size_t)min(s, ns - 1) * 64;          // past the end: the last step again, never used
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
            for (int h = 0; h < 2; h++) xq[u][r][h] = *reinterpret_cast<const bf16x8*>(xp[r] + o + 32 * h);
    };
    auto multiply = [&](int u) {
#pragma unroll
        for (int f = 0; f < NF; f++) {
            bf16x8 first, second;
            few_fragments(wq[u][f][0], wq[u][f][1], first, second);
#pragma unroll
            for (int r = 0; r < R; r++) {
                acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(first, xq[u][r][0], acc[f][r], 0, 0, 0);
                acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(second, xq[u][r][1], acc[f][r], 0, 0, 0);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < D; u++) fetch(u, u);
    int s = 0;
    for (; s + D < ns; s += D) {
#pragma unroll
        for (int u = 0; u < D; u++) {
            multiply(u);
            fetch(u, s + D + u);
        }
    }
#pragma unroll
    for (int u = 0; u < D; u++)
        if (s + u < ns) multiply(u);
}

}  // namespace

}  // namespace unipool
