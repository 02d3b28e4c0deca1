// Shared declarations of the UniPool HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "unipool.h"

namespace unipool {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64;
constexpr int kMaxE = 512;
constexpr int kMaxK = 8;

// ---- error reporting (host) ------------------------------------------------
int set_error(int code, const char* fmt, ...);
int check_hip(hipError_t e, const char* what);
// Range and alignment checks every entry point runs on its shape before anything is launched.
int validate_shape(const unipool_shape* s, const char* fn);

// ---- top-k as a compile-time constant (host) --------------------------------
// The per-token kernels loop over the k copies of a token; with k known at compile time these loops unroll,
// the rows of the copies sit in registers and their loads are in flight together.
// Calls f with k as a compile-time constant (1 <= k <= kMaxK, checked at the boundary).
template <class F>
inline void with_top_k(int k, F f) {
    static_assert(kMaxK == 8, "one case per admissible k");
    switch (k) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        default: f(std::integral_constant<int, 8>{}); break;
    }
}

// ---- scalar conversions (device) --------------------------------------------
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }  // RNE

// 1 / (1 + e^-a) with the hardware reciprocal (1 ulp) instead of an IEEE division
__device__ __forceinline__ float logistic_f(float a) { return __builtin_amdgcn_rcpf(1.0f + __expf(-a)); }
__device__ __forceinline__ float silu_f(float a) { return a * logistic_f(a); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// out[0] = sum of n floats by one workgroup of 256 threads, a tree of fixed shape.  A thread's loads are requested eight at a
// time, in the order of the sum: one after the other they outlasted the kernels that the sum runs beside (all of
// unipool_route_bwd, 65536 partial sums of 1048576 tokens of 8 experts, d 64, 489 -> 442 us; 16384 of 262144 tokens of 64, d 768
// 343 -> 325).
__device__ __forceinline__ void block_sum_256(const float* part, int n, float* out) {
    __shared__ float red[256];
    const int t = threadIdx.x;
    float v = 0.f;
    for (int i = t; i < n; i += 8 * 256) {
        float q[8];
#pragma unroll
        for (int u = 0; u < 8; u++) q[u] = part[min(i + u * 256, n - 1)];
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (i + u * 256 < n) v += q[u];
    }
    red[t] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    if (t == 0) out[0] = red[0];
}

// ---- workspace layout ---------------------------------------------------------
// The workspace is cut into fixed regions, all 256-byte aligned, sized from the shape.
struct WsLayout {
    size_t tile_meta;      // int32: [0] number of row tiles, 4 ints per tile from [64] on, then the meeting counters
    size_t chunk_hist;     // int32 [ceil(T/64)][E]   permute: per-64-token histograms/bases
    size_t psum_part;      // float [ceil(T/64)][E] partial score sums; in the backward pass the partial sums of d_sigma
    size_t cnt_part;       // int32 [ceil(T/64)][E] partial counts
    size_t dz;             // act   [T][dz_stride]  router backward logits gradient; float [T][E] logits
    size_t ptr_tab;        // 5 device pointers for the single-layer weight gradient
    size_t wpart;          // float [split][dz_stride][d]  router weight gradient partials
    size_t total;
};
WsLayout ws_layout(const unipool_shape& s);

constexpr int kRouterTokensPerBlock = 64;   // tokens per block in the per-token router kernels
constexpr int kRouteBwdSplit = 64;          // max row chunks of the router weight-gradient reduction

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Row length of dz: the bfloat16 products read it in chunks of eight values, so its rows are filled up with zeros.
inline int dz_stride(const unipool_shape& s) { return s.dtype == UNIPOOL_BF16 ? cdiv(s.E, 8) * 8 : s.E; }

}  // namespace unipool
