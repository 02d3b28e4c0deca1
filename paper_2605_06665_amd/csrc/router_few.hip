// Router of a few tokens (decoding, short prompts), bfloat16: the kernel that owns 64 tokens against all experts
// would run on T / 64 compute units, each walking the whole router matrix (22 us at 4 tokens, 192 experts,
// d_model 1536; 63 us at 48 tokens, 512 experts, d_model 1024).  Here a workgroup owns 16 experts and 64 tokens and
// its wavefronts split the reduction, so the matrix is read by E / 16 compute units at once (5.7 and 7.4 us); the
// selection follows in a kernel of its own.
#include "few_rows.h"

namespace unipool {

namespace {

constexpr int kRlWaves = 8;

// z[t][e] = sum_i x[t][i] w[e][i]; R: fragments of 16 tokens per workgroup.  E is a multiple of 8, d of 64.
template <int R>
__global__ __launch_bounds__(64 * kRlWaves) void router_few_kernel(const bf16* __restrict__ x, const bf16* __restrict__ w,
                                                                   int T, int d, int E, float* __restrict__ z) {
    __shared__ f32x4 red[kRlWaves][R][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int e0 = blockIdx.x * 16, t0 = blockIdx.y * 16 * R;
    const bf16* xp[R];
#pragma unroll
    for (int r = 0; r < R; r++) xp[r] = x + (size_t)min(t0 + 16 * r + l16, T - 1) * d + 16 * lg;
    const bf16* wp[1] = {w + (size_t)(e0 + (lane & 7)) * d + 8 * (lane >> 3)};
    const int ns = d / 64;
    f32x4 acc[1][R];
    few_reduce<1, R, 3, false>(wp, e0 + 8 < E ? (size_t)8 * d : 0, xp, wave * ns / kRlWaves, (wave + 1) * ns / kRlWaves, acc);
#pragma unroll
    for (int r = 0; r < R; r++) red[wave][r][lane] = acc[0][r];
    __syncthreads();
    // wavefront r adds up the parts of fragment r in wavefront order
    if (wave < R) {
        f32x4 v = red[0][wave][lane];
#pragma unroll
        for (int q = 1; q < kRlWaves; q++) v += red[q][wave][lane];
        const int t = t0 + 16 * wave + l16, e = e0 + 4 * lg;
        if (t < T && e < E) *reinterpret_cast<f32x4*>(z + (size_t)t * E + e) = v;
    }
}

}  // namespace

bool router_few_supported(const unipool_shape& s) {
    // Up to 16 tokens a workgroup reads little of x beside its rows of the matrix (with the selection, us, against
    // the one-kernel router: 192 experts, d_model 1536, 4 tokens 11 / 19); with 64 tokens it pays only where the
    // matrix is what takes the time (512 experts, d_model 1024, k = 8, 48 tokens 19 / 50; 192 experts 20 / 20).
    return mfma_router_supported(s) && (s.T <= 16 || (s.T <= 64 && s.E > 256));
}

hipError_t router_few_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st) {
    const bf16 *xb = (const bf16*)x, *wb = (const bf16*)w;
    const int ne = cdiv(s.E, 16);
    if (s.T <= 16) router_few_kernel<1><<<dim3(ne, 1), 64 * kRlWaves, 0, st>>>(xb, wb, s.T, s.d_model, s.E, z);
    else if (s.T <= 32) router_few_kernel<2><<<dim3(ne, 1), 64 * kRlWaves, 0, st>>>(xb, wb, s.T, s.d_model, s.E, z);
    else router_few_kernel<4><<<dim3(ne, cdiv(s.T, 64)), 64 * kRlWaves, 0, st>>>(xb, wb, s.T, s.d_model, s.E, z);
    return hipGetLastError();
}

}  // namespace unipool
