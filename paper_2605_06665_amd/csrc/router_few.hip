// Router of a few tokens (decoding, short prompts), bfloat16: the kernel that owns 64 tokens against all experts
// would run on T / 64 compute units, each walking the whole router matrix.  Here a wavefront owns 16 experts and 16
// tokens, so the matrix is read by E / 16 compute units at once, eight steps of 64 features ahead; the selection follows
// in a kernel of its own.
#include "few_rows.h"

namespace unipool {

namespace {

// z[t][e] = sum_i x[t][i] w[e][i].  E is a multiple of 8, d of 64.
template <int D>
__global__ __launch_bounds__(64) void router_few_kernel(const bf16* __restrict__ x, const bf16* __restrict__ w, int T, int d,
                                                        int E, float* __restrict__ z) {
    const int lane = threadIdx.x, l16 = lane & 15, lg = lane >> 4;
    const int e0 = blockIdx.x * 16, t = blockIdx.y * 16 + l16;
    const bf16* const xp[1] = {x + (size_t)min(t, T - 1) * d + 8 * lg};
    const bf16* const wp[1] = {w + (size_t)(e0 + (lane & 7)) * d + 8 * few_chunk(lane)};
    f32x4 acc[1][1];
    few_reduce<1, 1, D, false>(wp, e0 + 8 < E ? (size_t)8 * d : 0, xp, d / 64, acc);
    const int e = e0 + 4 * lg;
    if (t < T && e < E) *reinterpret_cast<f32x4*>(z + (size_t)t * E + e) = acc[0][0];
}

}  // namespace

bool router_few_supported(const unipool_shape& s) {
    // Up to 16 tokens a wavefront reads little of x beside its rows of the matrix; with 64 tokens it pays only where the
    // matrix is what takes the time.  All of the entry point (launches back to back in a graph), this path / the
    // one-kernel router, us: 192 experts, d_model 1536, 4 tokens 10 / 19; 512 experts, d_model 1024, k = 8, 48 tokens
    // 14 / 49.
    return mfma_router_supported(s) && (s.T <= 16 || (s.T <= 64 && s.E > 256));
}

hipError_t router_few_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st) {
    const bf16 *xb = (const bf16*)x, *wb = (const bf16*)w;
    const dim3 grid(cdiv(s.E, 16), cdiv(s.T, 16));
    if (s.d_model >= 512) router_few_kernel<8><<<grid, 64, 0, st>>>(xb, wb, s.T, s.d_model, s.E, z);
    else router_few_kernel<4><<<grid, 64, 0, st>>>(xb, wb, s.T, s.d_model, s.E, z);
    return hipGetLastError();
}

}  // namespace unipool
