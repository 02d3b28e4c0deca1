// Host-side launchers of the HIP kernels.  Each returns a hipError_t from the launch.
#pragma once

#include "common.h"

namespace unipool {

// ---- router.hip -------------------------------------------------------------------
// Per-token NormRouter score, top-k, gates and block-partial statistics from logits.
hipError_t launch_route_score_topk(const unipool_shape& s, const float* logits, int32_t* topk_idx,
                                   float* topk_gate, int32_t* counts, float* psum,
                                   int32_t* cnt_part, float* psum_part, float* wpart, hipStream_t st);
// Sums of the block partials.
hipError_t launch_route_finalize(const unipool_shape& s, const int32_t* cnt_part, const float* psum_part,
                                 int32_t* counts, float* psum, hipStream_t st);
// Per-token backward of the score: writes dz (act dtype) and partial sums of d_sigma, which the kernels of the contractions add
// up.  dsigma_part: one float per block of dz_tokens_per_block tokens, so 1, 4 or 8 floats per 64 tokens, never more than the E
// that the area of the partial score sums, where they lie, has for 64 tokens.
inline int dz_tokens_per_block(const unipool_shape& s) { return s.E < 4 ? kRouterTokensPerBlock : s.E <= 256 ? 16 : 8; }
hipError_t launch_route_bwd_dz(const unipool_shape& s, const float* logits, const int32_t* topk_idx,
                               const float* dgate, const float* aux_coef, void* dz,
                               float* dsigma_part, hipStream_t st);

// ---- permute.hip ------------------------------------------------------------------
hipError_t launch_permute(const unipool_shape& s, const void* x, const int32_t* topk_idx,
                          const int32_t* counts, void* x_perm, int32_t* expert_offsets,
                          int32_t* row_of_slot, int32_t* slot_of_row, int32_t* chunk_hist,
                          hipStream_t st);

// ---- combine.hip ------------------------------------------------------------------
hipError_t launch_combine(const unipool_shape& s, const void* y_perm, const int32_t* row_of_slot,
                          const float* gate, void* out, hipStream_t st);
hipError_t launch_combine_bwd(const unipool_shape& s, const void* dout, const void* y_perm,
                              const int32_t* row_of_slot, const float* gate, void* dy_perm,
                              float* dgate, hipStream_t st);

// ---- aux_loss.hip -----------------------------------------------------------------
hipError_t launch_pool_aux_loss(const unipool_shape& s, const int32_t* counts, const float* psum,
                                const float* fbar_in, int32_t* pool_counts, float* fbar_out,
                                float* loss, float* aux_coef, hipStream_t st);

// ---- analysis.hip -----------------------------------------------------------------
int c_blocks(int n);     // partial sums the c estimate needs for n draws
hipError_t launch_estimate_c(int E, int k, const float* samples, int n, float* part_sum,
                             int32_t* part_used, float* c_out, int32_t* used_out, hipStream_t st);
hipError_t launch_distinct_experts(const int32_t* const* idx_layers, int L, int T, int k,
                                   int32_t* distinct, int32_t* part_sum, float* mean_out, hipStream_t st);

// ---- router_fused.hip: logits on the matrix cores, scores, top-k and block statistics in one kernel -----
bool router_fused_supported(const unipool_shape& s);
hipError_t router_fused(const unipool_shape& s, const void* x, const void* w, float* z, int32_t* topk_idx,
                        float* topk_gate, int32_t* cnt_part, float* psum_part, hipStream_t st);

// ---- router_few.hip: logits of a few bfloat16 tokens ------------------------------------------
bool router_few_supported(const unipool_shape& s);
hipError_t router_few_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st);

// ---- gemm_f32.hip: float contractions on the matrix cores, any sizes; the router's also of bfloat16 operands -----
hipError_t f32_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st);
// slot_of_row != nullptr: x_perm is the un-permuted x and row r reads token slot_of_row[r] / k of it
hipError_t f32_ffn_fwd(const unipool_shape& s, const void* x_perm, const int32_t* offsets, const void* wgu,
                       const void* wd, void* a, void* b, void* h, void* y, hipStream_t st,
                       const int32_t* slot_of_row = nullptr);
hipError_t f32_ffn_gate_up(const unipool_shape& s, const void* x_perm, const int32_t* offsets, const void* wgu,
                           void* a, void* b, void* h, hipStream_t st, const int32_t* slot_of_row = nullptr);
hipError_t f32_ffn_dgrad(const unipool_shape& s, const void* dy, const void* a, const void* b,
                         const int32_t* offsets, const void* wgu, const void* wd, void* dx, void* d_act,
                         hipStream_t st);
hipError_t f32_ffn_wgrad(const unipool_shape& s, int n_layers, const void* const* x_perm_l,
                         const void* const* d_act_l, const void* const* h_l, const void* const* dy_l,
                         const int32_t* const* offsets_l, float* dwgu, float* dwd, int accumulate, hipStream_t st);
hipError_t f32_route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz, float* dw,
                            void* dx, int dx_accumulate, const float* dsigma_part, float* d_sigma, float* wpart,
                            hipStream_t st);

int num_cus();

// ---- gemm_mfma.hip: bf16 MFMA grouped GEMMs -----------------------------------------
bool mfma_ffn_supported(const unipool_shape& s);
bool mfma_router_supported(const unipool_shape& s);
hipError_t mfma_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st);
hipError_t mfma_ffn_fwd(const unipool_shape& s, const void* x_perm, const int32_t* offsets,
                        const void* wgu, const void* wd, void* a, void* b, void* h, void* y,
                        int32_t* tile_meta, int32_t* extra_meta, hipStream_t st, const int32_t* slot_of_row = nullptr);
hipError_t mfma_ffn_gate_up(const unipool_shape& s, const void* x_perm, const int32_t* offsets,
                            const void* wgu, void* a, void* b, void* h, int32_t* tile_meta,
                            int32_t* extra_meta, hipStream_t st);
hipError_t mfma_ffn_dgrad(const unipool_shape& s, const void* dy, const void* a, const void* b,
                          const int32_t* offsets, const void* wgu, const void* wd, void* dx,
                          void* d_act, int32_t* tile_meta, int32_t* extra_meta, hipStream_t st);
hipError_t mfma_ffn_wgrad(const unipool_shape& s, int n_layers, const void* const* x_perm_l,
                          const void* const* d_act_l, const void* const* h_l,
                          const void* const* dy_l, const int32_t* const* offsets_l,
                          float* dwgu, float* dwd, int accumulate, hipStream_t st);
hipError_t mfma_ffn_wgrad_layer(const unipool_shape& s, const void* x_perm, const void* d_act, const void* h, const void* dy,
                                const int32_t* offsets, float* dwgu, float* dwd, hipStream_t st);     // added to dwgu, dwd
int mfma_tile_forms(const unipool_shape& s, bool extra, int n_layers, int accumulate);
bool mfma_route_bwd_supported(const unipool_shape& s, const void* x, const void* w, const void* dx);
hipError_t mfma_route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz,
                             float* dw, void* dx, int dx_accumulate, const float* dsigma_part, float* d_sigma,
                             float* wpart, hipStream_t st);

// ---- ffn_few.hip: bf16 expert FFN forward where an expert has few rows -----------------------
bool few_rows_supported(const unipool_shape& s);
hipError_t few_ffn_gate_up(const unipool_shape& s, const void* x, const int32_t* offsets, const void* wgu, void* a_out,
                           void* b_out, void* h_out, hipStream_t st, const int32_t* slot_of_row = nullptr);
hipError_t few_ffn_fwd(const unipool_shape& s, const void* x, const int32_t* offsets, const void* wgu, const void* wd,
                       void* a_out, void* b_out, void* h_out, void* y, hipStream_t st,
                       const int32_t* slot_of_row = nullptr);

// ---- small utilities (api.hip) ---------------------------------------------------------
hipError_t launch_set_ptrs(void** table, const void* p0, const void* p1, const void* p2,
                           const void* p3, const void* p4, hipStream_t st);

}  // namespace unipool
