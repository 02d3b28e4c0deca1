// Expert FFN forward for calls with few rows per expert (decoding, short prompts), bfloat16.
//
// With a handful of rows per expert the two products are a single pass over the weights of the experts that
// have rows (2 FLOP per weight byte and row), so HBM is the bound and what counts is how many weight bytes
// are in flight.  Nothing is shared between wavefronts, hence no LDS tiles, no tile table and no barriers in
// the reduction:
//   * a task is one expert and 16 output columns (gate-up: 16 gate columns and the 16 up columns they meet),
//     and a wavefront owns it for all rows of the expert, so each weight is read by one wavefront only;
//   * a sum is never cut: a row comes out with the bits of the tile kernels.  Where there are few tasks a wavefront
//     has a SIMD's registers to itself and fills them with loads instead (up to 12 or 16 steps of 64 reduction indices
//     ahead, three to six with many wavefronts per SIMD);
//   * weights go straight from memory to registers.  A load covers 8 columns x 128 bytes, whole cache lines (16 columns
//     x 64 bytes, the layout the MFMA A operand wants, reached 5.2 TB/s where this reached 5.8), and a rotation of half
//     of the lanes by eight turns two of them into two A operands.  Each weight is used once, so the loads are streaming
//     loads (5.8 -> 6.3 TB/s; they serve pools that fit the caches too: 16 experts of 768 x 2048, k = 1, 16 tokens 22.9 ->
//     21.6 us);
//   * activation fragments (the B operand) come the same way, up to 32 rows per pass over the weights; rows past
//     the expert's last repeat it, so they add no cache lines.
// Every workgroup finds the experts with rows by itself (one pass over the offsets), which costs less than
// the launch that a table would need.
// Measured, both products (launches back to back in a graph), against the tiles of gemm_xw: 192 experts of 1536 x 4096,
// k = 2: 1 token 54 -> 20 us, 4 tokens 93 -> 52 (5.7 TB/s), 64 tokens 662 -> 575; 512 experts of 1024 x 704, k = 8, 48
// tokens 250 -> 188 us (6.2 TB/s); pools that fit the caches: 32 experts of 512 x 512, k = 2, 64 tokens 23 -> 15 us, 16
// experts of 1536 x 1536, k = 1, 32 tokens 42 -> 40.
#include "few_rows.h"

namespace unipool {

namespace {

constexpr int kFewMaxE = 512;

struct FewArgs {
    const bf16* X;                      // [rows][K], or the tokens when gather is given
    const int32_t* gather;              // row r is row gather[r] / gather_div of X
    int gather_div;
    const bf16* W;                      // [E][columns][K]
    long long w_stride;
    int up_rows;                        // gate-up: first up column (= d_ff)
    const int32_t* offsets;
    int E, K, N;
    bf16* out0;                         // y, or A
    bf16* out1;                         // B
    bf16* out2;                         // H
};

__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    union { bf16 h[4]; uint2 u; } p;
    p.h[0] = (bf16)a; p.h[1] = (bf16)b; p.h[2] = (bf16)c; p.h[3] = (bf16)d;
    return p.u;
}

// One task: rows row0 .. row0 + rows - 1 (at most 16 R) of an expert against columns c0 .. c0 + 15.
template <bool GATE_UP, int R, int D>
__device__ __forceinline__ void few_task(const FewArgs& a, const bf16* We, int c0, int row0, int rows, int lane) {
    constexpr int NF = GATE_UP ? 2 : 1;
    const int l16 = lane & 15, lg = lane >> 4;
    const bf16* xp[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        int row = row0 + min(16 * r + l16, rows - 1);
        if (a.gather != nullptr) row = a.gather[row] / a.gather_div;
        xp[r] = a.X + (size_t)row * a.K + 8 * lg;
    }
    const bf16* wp[NF];
#pragma unroll
    for (int f = 0; f < NF; f++) wp[f] = We + (size_t)(f * a.up_rows + c0 + (lane & 7)) * a.K + 8 * few_chunk(lane);
    f32x4 acc[NF][R];
    few_reduce<NF, R, D, true>(wp, (size_t)8 * a.K, xp, a.K / 64, acc);
    // acc[f][r][i] = C[row 16 r + l16][column c0 + 4 lg + i]
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (16 * r + l16 < rows) {
            const size_t o = (size_t)(row0 + 16 * r + l16) * a.N + c0 + 4 * lg;
            const f32x4 v = acc[0][r];
            *reinterpret_cast<uint2*>(a.out0 + o) = pack_bf16x4(v[0], v[1], v[2], v[3]);
            if constexpr (GATE_UP) {
                const f32x4 up = acc[1][r];
                float h[4];
#pragma unroll
                for (int i = 0; i < 4; i++) h[i] = silu_f(v[i]) * up[i];
                *reinterpret_cast<uint2*>(a.out1 + o) = pack_bf16x4(up[0], up[1], up[2], up[3]);
                *reinterpret_cast<uint2*>(a.out2 + o) = pack_bf16x4(h[0], h[1], h[2], h[3]);
            }
        }
    }
}

// RM: most row fragments per pass over an expert's weights, D1 / DM: steps in flight with one / RM fragments
template <bool GATE_UP, int WAVES, int RM, int D1, int DM>
__global__ __launch_bounds__(64 * WAVES) void ffn_few_kernel(const FewArgs a) {
    constexpr int kThreads = 64 * WAVES;
    __shared__ int list_e[kFewMaxE], list_r0[kFewMaxE], list_n[kFewMaxE];
    __shared__ int wcnt[kFewMaxE / kThreads][WAVES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // experts with rows, in ascending order
    int n_list = 0;
#pragma unroll
    for (int p = 0; p < kFewMaxE / kThreads; p++) {
        const int e = p * kThreads + tid;
        int r0 = 0, n = 0;
        if (e < a.E) {
            r0 = a.offsets[e];
            n = a.offsets[e + 1] - r0;
        }
        const unsigned long long has = __ballot(n > 0);
        if (lane == 0) wcnt[p][wave] = __popcll(has);
        __syncthreads();
        int at = n_list;
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            if (w < wave) at += wcnt[p][w];
            n_list += wcnt[p][w];
        }
        if (n > 0) {
            at += __popcll(has & ((1ull << lane) - 1ull));
            list_e[at] = e;
            list_r0[at] = r0;
            list_n[at] = n;
        }
    }
    __syncthreads();
    const int per_e = a.N / 16;
    const int tasks = n_list * per_e;
    for (int t = blockIdx.x * WAVES + wave; t < tasks; t += gridDim.x * WAVES) {
        const int i = t / per_e, c0 = (t % per_e) * 16;
        const int e = __builtin_amdgcn_readfirstlane(list_e[i]);
        const int r0 = __builtin_amdgcn_readfirstlane(list_r0[i]);
        const int n = __builtin_amdgcn_readfirstlane(list_n[i]);
        const bf16* We = a.W + (long long)e * a.w_stride;
        for (int c = 0; c < n; c += 16 * RM) {
            const int rows = min(n - c, 16 * RM);
            if (RM == 1 || rows <= 16) few_task<GATE_UP, 1, D1>(a, We, c0, r0 + c, rows, lane);
            else few_task<GATE_UP, RM, DM>(a, We, c0, r0 + c, rows, lane);
        }
    }
}

// One wavefront per workgroup and task, D1 (D2) steps in flight with one (two) row fragments.
template <bool GATE_UP, int D1, int D2>
hipError_t run_one(const FewArgs& a, bool one, int tasks, hipStream_t st) {
    if (one) ffn_few_kernel<GATE_UP, 1, 1, D1, D1><<<tasks, 64, 0, st>>>(a);
    else ffn_few_kernel<GATE_UP, 1, 2, D1, D2><<<tasks, 64, 0, st>>>(a);
    return hipGetLastError();
}

template <bool GATE_UP>
hipError_t run_few(const FewArgs& a, int tokens, int total_rows, hipStream_t st) {
    // tasks if every row had an expert of its own
    const int most = (total_rows < a.E ? total_rows : a.E) * (a.N / 16);
    const int cus = num_cus();
    const bool one = tokens <= 16;                // an expert gets a token at most once
    const int ns = a.K / 64;
    // At most one task per SIMD: all registers are its own and as many steps are in flight as they hold, fewer where
    // they would mostly repeat the last step.
    if (most <= 4 * cus) {
        if (ns < 8) return run_one<GATE_UP, 4, 4>(a, one, most, st);
        if constexpr (GATE_UP) {
            if (ns >= 24 || ns % 12 == 0) return run_one<true, 12, 8>(a, one, most, st);
        } else {
            if (ns >= 32 || ns % 16 == 0) return run_one<false, 16, 8>(a, one, most, st);
        }
        return run_one<GATE_UP, 8, 6>(a, one, most, st);
    }
    // At most two: half of the registers each.
    if (most <= 8 * cus) {
        if (ns < 6) return run_one<GATE_UP, 4, 4>(a, one, most, st);
        if (GATE_UP || ns < 8) return run_one<GATE_UP, 6, 4>(a, one, most, st);
        return run_one<false, 8, 6>(a, one, most, st);
    }
    const int blocks = cdiv(most, 4) < 4 * cus ? cdiv(most, 4) : 4 * cus;
    constexpr int D1 = GATE_UP ? 4 : 6;
    if (one) ffn_few_kernel<GATE_UP, 4, 1, D1, D1><<<blocks, 256, 0, st>>>(a);
    else ffn_few_kernel<GATE_UP, 4, 2, D1, 3><<<blocks, 256, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace

bool few_rows_supported(const unipool_shape& s) {
    // Up to 16 tokens an expert has at most one row fragment; up to 64 it pays while the experts have eight rows on
    // average.  Both products, this path / the tiles (us): 192 experts of 1536 x 4096, k = 2, 4 tokens 52 / 93, 64 tokens
    // 575 / 662; 512 experts of 1024 x 704, k = 8, 64 tokens 225 / 288; 16 experts of 1024 x 1024, k = 4, 32 tokens (8
    // rows) 24 / 30, 64 tokens (16 rows) 27 / 30, under skewed use 32 / 31; 8 experts, k = 8, 64 tokens (64 rows) 35 / 30.
    return mfma_ffn_supported(s) && (s.T <= 16 || (s.T <= 64 && s.T * s.k <= 8 * s.E));
}

hipError_t few_ffn_gate_up(const unipool_shape& s, const void* x, const int32_t* offsets, const void* wgu, void* a_out,
                           void* b_out, void* h_out, hipStream_t st, const int32_t* slot_of_row) {
    FewArgs a = {};
    a.X = (const bf16*)x; a.gather = slot_of_row; a.gather_div = s.k;
    a.W = (const bf16*)wgu; a.w_stride = 2LL * s.d_ff * s.d_model; a.up_rows = s.d_ff;
    a.offsets = offsets; a.E = s.E; a.K = s.d_model; a.N = s.d_ff;
    a.out0 = (bf16*)a_out; a.out1 = (bf16*)b_out; a.out2 = (bf16*)h_out;
    return run_few<true>(a, s.T, s.T * s.k, st);
}

hipError_t few_ffn_fwd(const unipool_shape& s, const void* x, const int32_t* offsets, const void* wgu, const void* wd,
                       void* a_out, void* b_out, void* h_out, void* y, hipStream_t st, const int32_t* slot_of_row) {
    hipError_t e = few_ffn_gate_up(s, x, offsets, wgu, a_out, b_out, h_out, st, slot_of_row);
    if (e != hipSuccess) return e;
    FewArgs a = {};
    a.X = (const bf16*)h_out;
    a.W = (const bf16*)wd; a.w_stride = (long long)s.d_model * s.d_ff;
    a.offsets = offsets; a.E = s.E; a.K = s.d_ff; a.N = s.d_model;
    a.out0 = (bf16*)y;
    return run_few<false>(a, s.T, s.T * s.k, st);
}

}  // namespace unipool
