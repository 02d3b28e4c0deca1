// Router backward of bfloat16 pools whose size is not a multiple of 8, one thread per output element.
// Sums run in float in index order.
#include "kernels.h"

namespace unipool {

namespace {

template <typename TA>
__global__ void route_dw_kernel(const TA* __restrict__ dz, const TA* __restrict__ x, int T, int d,
                                int E, float* __restrict__ dw) {
    const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (size_t)E * d) return;
    const int e = (int)(id / d), c = (int)(id % d);
    float acc = 0.f;
    for (int t = 0; t < T; t++) acc += to_f32(dz[(size_t)t * E + e]) * to_f32(x[(size_t)t * d + c]);
    dw[id] = acc;
}

template <typename TA>
__global__ void route_dx_kernel(const TA* __restrict__ dz, const TA* __restrict__ w, int T, int d,
                                int E, int accumulate, TA* __restrict__ dx) {
    const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (size_t)T * d) return;
    const int t = (int)(id / d), c = (int)(id % d);
    float acc = accumulate ? to_f32(dx[id]) : 0.f;
    for (int e = 0; e < E; e++) acc += to_f32(dz[(size_t)t * E + e]) * to_f32(w[(size_t)e * d + c]);
    dx[id] = from_f32<TA>(acc);
}

inline unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t naive_route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz,
                              float* dw, void* dx, int dx_accumulate, hipStream_t st) {
    route_dw_kernel<bf16><<<blocks_for((size_t)s.E * s.d_model), 256, 0, st>>>((const bf16*)dz, (const bf16*)x, s.T,
                                                                            s.d_model, s.E, dw);
    route_dx_kernel<bf16><<<blocks_for((size_t)s.T * s.d_model), 256, 0, st>>>(
        (const bf16*)dz, (const bf16*)w, s.T, s.d_model, s.E, dx_accumulate, (bf16*)dx);
    return hipGetLastError();
}

}  // namespace unipool
