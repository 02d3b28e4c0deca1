// Contractions on v_mfma_f32_16x16x4_f32: float mode (which is checked to 1e-5), and the router products of the
// bfloat16 shapes and operands that the bfloat16 router kernels do not take.  Any sizes, any alignment.
//
// The instruction adds its four products in index order, each with one rounding (test_gpu_f32_chain.py compares logits
// with a chain of fused multiply-adds, bit for bit), so a sum here is the plain index-order chain and does not depend on
// tile sizes; no kernel in this file cuts a reduction except the router's weight gradient over the tokens.
//
// A workgroup is four wavefronts (2 x 2) of WT x WT outputs, WT = 32 or 16.  A 16x16x4 step keeps the matrix
// core busy for 32 cycles (157 TFLOP/s for the card, a sixteenth of what bfloat16 steps reach), so what is hidden is latency:
// tiles pass through registers (the next two stages are requested, without a branch, while one is multiplied) into two LDS
// buffers as 16-byte pieces, one barrier per stage, whichever index is the contiguous one in memory; neighbouring tiles run
// on one XCD and meet in its L2.
// 3003 rows, d = 252, f = 500, 12 experts, us, launches back to back in a graph: both forward products 45 -> 42, both
// backward products 52 -> 47, weight gradients of two layers 108 -> 70 (with one stage requested ahead, a branch around
// every load, strided operands transposed on their way into LDS, single tiles dealt to the XCDs in turn -> now); 32 experts of
// 320 x 640, 4500 rows: 89 -> 85, 106 -> 90, 213 -> 139.  The matrix cores are busy half of the time there (74.5 of 148
// million cycles of the gate and up projections), the rest is the start of the workgroups and the last round.
#include "kernels.h"

namespace unipool {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxLayers = 256;    // of one weight gradient: what unipool_expert_wgrad takes

enum Epilogue {
    kStore,        // output in the activation type, optionally added to the destination
    kFloat,        // float output (logits, weight gradients), optionally added
    kSwigluFwd,    // columns come in pairs of 16 gate and 16 up: writes A, B, H
    kSwigluBwd,    // the product is dH: reads A, B, writes dA | dB
};

// C[m][n] = sum_k A(m, k) B(n, k); layouts by template, leading dimensions here.
struct Args {
    const void* A;
    const void* B;
    int lda, ldb;
    long long b_stride;            // elements of B between experts
    int M, N, K;                   // M: rows of all groups (or of the matrix); N per half for kSwigluFwd
    int n_tiles;                   // column tiles
    const int32_t* offsets;        // row groups [E + 1]; null: one matrix
    int E;                         // row groups, or weight gradients
    const int32_t* gather;         // row r of A is row gather[r] / gather_div (null: r)
    int gather_div;
    void* out0;
    void* out1;
    void* out2;
    int ldo, add;
    const void* aux_a;
    const void* aux_b;
    int vec_a, vec_b, vec_o;       // four elements at a time: leading dimension and pointers allow it
    // kFloat over row groups of several layers (K runs over the rows of expert e in every layer)
    int n_layers;
    const void* const* a_l;
    const void* const* b_l;
    const int32_t* const* off_l;
    int m_tiles;
    long long out_stride;
    int chunk;                     // rows per partial sum (flat K ranges); 0: none
    // a sum of floats that the first workgroup of the launch does on the way (null: none)
    const float* sum_part;
    int sum_n;
    float* sum_out;
};

template <typename TA> __device__ __forceinline__ f32x4 fetch_vec(const TA* p);
template <> __device__ __forceinline__ f32x4 fetch_vec<float>(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
template <> __device__ __forceinline__ f32x4 fetch_vec<bf16>(const bf16* p) {
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
// four elements from p on, of which the first n exist (n <= 0: none; with vec: all or none)
template <typename TA>
__device__ __forceinline__ f32x4 fetch4(const TA* p, int n, bool vec) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        if (n > 0) v = fetch_vec(p);
    } else {
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (i < n) v[i] = to_f32(p[i]);
    }
    return v;
}
template <typename T>
__device__ __forceinline__ void store4(T* p, f32x4 v, int n, bool vec, bool add) {
    if (vec && n >= 4) {
        if (add) {
            const f32x4 o = fetch_vec(p);
            v = o + v;
        }
        if constexpr (std::is_same<T, float>::value) {
            *reinterpret_cast<f32x4*>(p) = v;
        } else {
            const bf16x4 h = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
            *reinterpret_cast<bf16x4*>(p) = h;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (i < n) p[i] = from_f32<T>((add ? to_f32(p[i]) : 0.f) + v[i]);
    }
}

// Place of this workgroup in a list of `total` tiles that is cut into eight parts, one per XCD (workgroups are dealt to the
// XCDs in turn): neighbouring tiles, which share operands, meet in one L2.  total or more: nothing to do.
__device__ __forceinline__ int tile_of_block(int total) {
    const int per_xcd = (total + 7) / 8, slot = blockIdx.x / 8;
    return slot < per_xcd ? (blockIdx.x % 8) * per_xcd + slot : total;
}

// The same where tiles differ in length: the list is dealt to the XCDs in turn, up to a row of n_tiles tiles at a time (which
// share an operand), fewer where that gave an XCD less than four turns.  Workgroups past the list get tiles past it.
// Weight gradients, whose tiles are as long as their expert has rows: the experts with many rows, wherever they are in the pool,
// are spread over all XCDs (in eight parts / dealt, us: 32 experts of 320 x 640, 4500 rows of two layers, about half of them on
// the first six 332 / 151, on six others 239 / 170, on all alike 155 / 154; whole experts in turn 162, 221, 159; all of these
// before LDS rows lost their padding, which made 151 and 154 into 137 and 139).  Chunks of one
// matrix, which are equally long, keep the eight parts (router backward of 90 experts, d 832, 4000 tokens 45 us, dealt 52).
// Row tiles of pools beyond 64 experts, most of which have few rows: half of the rows with a fifth of the experts, both forward
// products in eight parts / dealt 158 experts of 40 x 114 17.8 / 15.0, 458 of 44 x 77 34.4 / 29.3; even rows 90 of 128 x 256
// 19.0 / 18.7, 400 of 64 x 128 16.6 / 17.3.  Up to 64 experts the eight parts share more in L2 (12 of 252 x 500 42.3 / 44.7; 24
// of 256 x 512, rows by Zipf's law 66.9 / 69.7).
__device__ __forceinline__ int dealt_tile_of_block(int total, int n_tiles) {
    const int run = max(1, min(n_tiles, total / 32)), slot = blockIdx.x / 8;
    return (slot / run * 8 + blockIdx.x % 8) * run + slot % run;
}

// Row tile of the row groups, BM rows a tile, that this workgroup works on with which of n_tiles column tiles.  Up to 64
// experts every wavefront finds it by itself; of larger pools a thread counts the tiles of two experts, so that the offsets
// are waited for once.  (Batches of 64 experts one after the other, which every wavefront went through twice, once for the
// number of tiles and once for its own: 400 experts of 64 x 128, 600 rows, us, both forward products 30.5 -> 16.9, both
// backward products 29.8 -> 16.2; 90 experts of 128 x 256, 600 rows 20.3 -> 19.0 and 19.7 -> 18.5.)
struct RowTile {
    int expert, row0, rows, nt;    // rows = 0: past the last tile
};
template <int BM>
__device__ __forceinline__ RowTile find_row_tile(const int32_t* offsets, int E, int n_tiles, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    auto scan = [&](int v) {                       // inclusive, over the wavefront
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(v, d, 64);
            if (lane >= d) v += o;
        }
        return v;
    };
    if (E <= 64) {
        const int r0 = offsets[min(lane, E)], r1 = offsets[min(lane + 1, E)];
        const int mine = (r1 - r0 + BM - 1) / BM, upto = scan(mine), first = upto - mine;
        const int total = __shfl(upto, 63, 64);
        const int tile = tile_of_block(total * n_tiles), want = tile / n_tiles;
        if (want >= total) return RowTile{0, 0, 0, 0};
        const unsigned long long hit = __ballot(want >= first && want < upto);
        const int src = __ffsll((long long)hit) - 1;
        const int row0 = __shfl(r0, src, 64) + (want - __shfl(first, src, 64)) * BM;
        return RowTile{src, row0, min(BM, __shfl(r1, src, 64) - row0), tile % n_tiles};
    }
    static_assert(kMaxE <= 2 * kThreads, "two experts per thread");
    __shared__ int wsum[kThreads / 64];
    __shared__ int found[3];
    const int e = 2 * tid;
    const int r0 = offsets[min(e, E)], r1 = offsets[min(e + 1, E)], r2 = offsets[min(e + 2, E)];
    const int t0 = (r1 - r0 + BM - 1) / BM, t1 = (r2 - r1 + BM - 1) / BM;
    int upto = scan(t0 + t1);
    if (lane == 63) wsum[wave] = upto;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; w++) {
        if (w < wave) upto += wsum[w];
        total += wsum[w];
    }
    const int tile = dealt_tile_of_block(total * n_tiles, n_tiles), want = tile / n_tiles;
    if (want >= total) return RowTile{0, 0, 0, 0};
    const int nth = want - (upto - t0 - t1);       // of this thread's tiles
    if (nth >= 0 && want < upto) {
        const bool second = nth >= t0;
        found[0] = e + second;
        found[1] = (second ? r1 : r0) + (second ? nth - t0 : nth) * BM;
        found[2] = second ? r2 : r1;
    }
    __syncthreads();
    return RowTile{found[0], found[1], min(BM, found[2] - found[1]), tile % n_tiles};
}

// ATR / BTR: the operand's reduction index is the strided one in memory ([k][m], [k][n]).
// LAYERS: K runs over the rows of one expert in all layers (weight gradients; both operands strided).
template <typename TA, int WT, bool ATR, bool BTR, Epilogue EPI, bool LAYERS>
__global__ __launch_bounds__(kThreads) void gemm_f32_kernel(const Args g) {
    constexpr int BM = 2 * WT;                 // tile of the workgroup, both ways
    constexpr int BK = WT == 32 ? 32 : 64;     // reduction indices per stage: 2048 values of each operand
    constexpr int CH = BK / 16;                // 16-index chunks per stage
    // LDS rows in floats, so that the 16 x 4 values of a fragment read lie in 64 banks: K-contiguous operands keep their
    // rows of BK indices and four values of padding, strided ones their rows of BM columns, in groups of 16 that trade places
    // from row to row.  (With 16 columns of padding instead a CU ran two or three workgroups where it now runs four: weight
    // gradients, us: 508 experts of 528 x 576, 76 rows of two layers, added 310 -> 263, written 474 -> 408; 315 of 295 x 636, 112
    // rows of eight 194 -> 162, 400 -> 341; 32 of 320 x 640, 4500 rows 153 -> 139; 12 of 252 x 500, 3003 rows, both backward
    // products 51.9 -> 48.2.)
    constexpr int LD = BK + 4, LDT = BM;
    auto swz = [](int k) { return (BM == 64 ? k & 3 : k >> 1 & 1) * 16; };       // of a strided operand's row k
    constexpr int ABUF = ATR ? BK * LDT : BM * LD, BBUF = BTR ? BK * LDT : BM * LD;
    constexpr int NF = WT / 16;                // 16-wide fragments per wavefront and side
    static_assert(BM * BK == 8 * kThreads, "two groups of four values per thread and operand");
    __shared__ __attribute__((aligned(16))) float lds[2][ABUF + BBUF];
    // row ranges and operands of the expert in every layer
    struct Layer {
        const TA* a;
        const TA* b;
        int r0, r1;
    };
    __shared__ Layer layers[LAYERS ? kMaxLayers : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lg = lane >> 4;

    // ---- which tile
    int expert = 0, row0 = 0, rows = 0, n0, k_begin = 0, k_end = g.K;
    if constexpr (LAYERS) {
        if (blockIdx.x == 0 && g.sum_part != nullptr) block_sum_256(g.sum_part, g.sum_n, g.sum_out);
        const int per = g.m_tiles * g.n_tiles;
        const int tile = g.n_layers > 0 ? dealt_tile_of_block(g.E * per, g.n_tiles) : tile_of_block(g.E * per);
        expert = tile / per;
        if (expert >= g.E) return;
        const int r = tile % per;
        row0 = (r / g.n_tiles) * BM;
        rows = min(BM, g.M - row0);
        n0 = (r % g.n_tiles) * BM;
        if (g.n_layers == 0) {                 // one matrix cut into chunks of rows: "expert" is the chunk
            k_begin = expert * g.chunk;
            k_end = min(g.K, k_begin + g.chunk);
        }
    } else if (g.offsets != nullptr) {
        const RowTile t = find_row_tile<BM>(g.offsets, g.E, g.n_tiles, tid);
        if (t.rows <= 0) return;
        expert = t.expert;
        row0 = t.row0;
        rows = t.rows;
        n0 = t.nt * BM;
    } else {
        const int m_tiles = (g.M + BM - 1) / BM, tile = tile_of_block(m_tiles * g.n_tiles), mt = tile / g.n_tiles;
        if (mt >= m_tiles) return;
        row0 = mt * BM;
        rows = min(BM, g.M - row0);
        n0 = (tile % g.n_tiles) * BM;
    }
    const TA* A = reinterpret_cast<const TA*>(g.A);
    const TA* B = reinterpret_cast<const TA*>(g.B);
    if constexpr (!LAYERS) B += (long long)expert * g.b_stride;

    // ---- this thread's two groups of four values of either operand: fixed tile rows (K-contiguous operands)
    // or fixed tile columns and K rows that advance by BK per stage (strided operands)
    constexpr int KG = BK / 4, MG = BM / 4;    // groups per row
    int kq[2], mq[2];                          // K-contiguous: first index, tile row
    int kr[2], nq[2];                          // strided: K row, first tile column
    const TA* arow[2];
    const TA* brow[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int id = i * kThreads + tid;
        kq[i] = (id % KG) * 4;
        mq[i] = id / KG;
        nq[i] = (id % MG) * 4;
        kr[i] = id / MG;
        arow[i] = brow[i] = nullptr;
        if constexpr (!ATR) {
            if (mq[i] < rows) {
                size_t r = (size_t)(row0 + mq[i]);
                if (g.gather != nullptr) r = (size_t)(g.gather[r] / g.gather_div);
                arow[i] = A + r * g.lda;
            }
        }
        if constexpr (!BTR) {
            int n;
            bool ok;
            if constexpr (EPI == kSwigluFwd) {
                // tile rows in groups of 32: 16 gate rows, the 16 up rows of the same columns
                const int c = n0 / 2 + (mq[i] >> 5) * 16 + (mq[i] & 15);
                ok = c < g.N;
                n = (mq[i] & 16) ? g.N + c : c;
            } else {
                n = n0 + mq[i];
                ok = n < g.N;
            }
            if (ok) brow[i] = B + (size_t)n * g.ldb;
        }
    }
    // cursors over the rows of the expert, layer after layer: the K rows of this thread's two groups
    int cl[2] = {-1, -1}, cr[2] = {kr[0], kr[1]}, ce[2] = {0, 0};
    const TA* ca[2] = {nullptr, nullptr};      // the layer's operands
    const TA* cb[2] = {nullptr, nullptr};
    int total_k = k_end - k_begin;
    bool vec_a = g.vec_a != 0, vec_b = g.vec_b != 0;     // (the layers' operands are only known by address here)
    auto settle = [&](int i) {                 // move past ended layers
        while (cr[i] >= ce[i] && cl[i] < g.n_layers) {
            const int over = cr[i] - ce[i];
            if (++cl[i] >= g.n_layers) break;
            const Layer l = layers[cl[i]];
            ce[i] = l.r1;
            cr[i] = l.r0 + over;
            ca[i] = l.a;
            cb[i] = l.b;
        }
    };
    if constexpr (LAYERS) {
        if (g.n_layers > 0) {
            for (int l = tid; l < g.n_layers; l += kThreads)
                layers[l] = Layer{reinterpret_cast<const TA*>(g.a_l[l]), reinterpret_cast<const TA*>(g.b_l[l]),
                                  g.off_l[l][expert], g.off_l[l][expert + 1]};
            __syncthreads();
            total_k = 0;
            for (int l = 0; l < g.n_layers; l++) {
                total_k += layers[l].r1 - layers[l].r0;
                vec_a = vec_a && ((size_t)layers[l].a & (4 * sizeof(TA) - 1)) == 0;
                vec_b = vec_b && ((size_t)layers[l].b & (4 * sizeof(TA) - 1)) == 0;
            }
            A = layers[0].a;
            B = layers[0].b;
            if (g.add && total_k == 0) return;
            settle(0);
            settle(1);
        }
    }
    const int stages = (total_k + BK - 1) / BK;

    f32x4 acc[NF][NF];
#pragma unroll
    for (int a = 0; a < NF; a++)
#pragma unroll
        for (int b = 0; b < NF; b++) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Operands of the next two stages on their way, as they are in memory (a conversion here would wait for the load).
    // FA / FB: four values of the operand at a time without a branch, so that the loads of two stages stay in flight; a group
    // past an end is loaded from the operand's start and put down as zeros.  An operand whose rows are not aligned to four
    // values goes value by value, and the other one keeps its wide loads (12 experts, 3003 rows, us, one form for both / a form
    // each: d 252, f 501 both backward products 83 / 67, weight gradients of two layers 103 / 86; d 250, f 500 77 / 61, 103 / 86;
    // router backward, 4000 tokens of 90 experts, d 832 52 / 44).
    using Raw = typename std::conditional<std::is_same<TA, float>::value, f32x4, bf16x4>::type;
    auto main_loop = [&](auto fa_c, auto fb_c) __attribute__((always_inline)) {
        constexpr bool FA = decltype(fa_c)::value, FB = decltype(fb_c)::value;
        Raw ra[2][2], rb[2][2];
        int oka[2] = {0, 0}, okb[2] = {0, 0};      // bit set: the set's group exists
        auto fetch = [&](int s, auto set_c) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            const int k0 = k_begin + s * BK;
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const TA* pa = nullptr;
                const TA* pb = nullptr;
                int na = 0, nb = 0;
                if constexpr (LAYERS) {
                    const int am = row0 + nq[i], bn = n0 + nq[i];
                    if (g.n_layers > 0) {
                        if (cl[i] < g.n_layers) {
                            pa = ca[i] + (size_t)cr[i] * g.lda + am;
                            pb = cb[i] + (size_t)cr[i] * g.ldb + bn;
                            na = g.M - am;
                            nb = g.N - bn;
                            cr[i] += BK;
                            settle(i);
                        }
                    } else if (k0 + kr[i] < k_end) {
                        pa = A + (size_t)(k0 + kr[i]) * g.lda + am;
                        pb = B + (size_t)(k0 + kr[i]) * g.ldb + bn;
                        na = g.M - am;
                        nb = g.N - bn;
                    }
                } else {
                    static_assert(LAYERS || !ATR, "a strided first operand belongs to the weight gradients");
                    pa = arow[i] + k0 + kq[i];
                    na = arow[i] != nullptr ? k_end - k0 - kq[i] : 0;
                    if constexpr (BTR) {
                        pb = B + (size_t)(k0 + kr[i]) * g.ldb + n0 + nq[i];
                        nb = k0 + kr[i] < k_end ? g.N - n0 - nq[i] : 0;
                    } else {
                        pb = brow[i] + k0 + kq[i];
                        nb = brow[i] != nullptr ? k_end - k0 - kq[i] : 0;
                    }
                }
                if constexpr (FA) {
                    ra[set][i] = *reinterpret_cast<const Raw*>(na > 0 ? pa : A);
                    oka[i] = (oka[i] & ~(1 << set)) | ((na > 0) << set);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; q++) ra[set][i][q] = q < na ? pa[q] : (TA)0.f;
                }
                if constexpr (FB) {
                    rb[set][i] = *reinterpret_cast<const Raw*>(nb > 0 ? pb : B);
                    okb[i] = (okb[i] & ~(1 << set)) | ((nb > 0) << set);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; q++) rb[set][i][q] = q < nb ? pb[q] : (TA)0.f;
                }
            }
        };
        auto put = [&](float* t, const Raw& v, bool ok, bool tr, int i) __attribute__((always_inline)) {
            const f32x4 f = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            *reinterpret_cast<f32x4*>(t + (tr ? kr[i] * LDT + (nq[i] ^ swz(kr[i])) : mq[i] * LD + kq[i])) =
                ok ? f : f32x4{0.f, 0.f, 0.f, 0.f};
        };
        // operands of the four instructions of chunk c: the lane's row (or column) at indices 4 q + lg
        auto frag = [&](const float* t, bool tr, int r, int c) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; q++) v[q] = t[tr ? (c * 16 + 4 * q + lg) * LDT + (r ^ swz(lg)) : r * LD + c * 16 + 4 * q + lg];
            return v;
        };

        auto stage = [&](int s, auto set_c) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            float* ta = lds[set];
            float* tb = ta + ABUF;
#pragma unroll
            for (int i = 0; i < 2; i++) {
                put(ta, ra[set][i], !FA || (oka[i] >> set & 1), ATR, i);
                put(tb, rb[set][i], !FB || (okb[i] >> set & 1), BTR, i);
            }
            __syncthreads();                       // the other buffer is free: its readers passed the barrier before
            if (s + 2 < stages) fetch(s + 2, set_c);
#pragma unroll
            for (int c = 0; c < CH; c++) {
                f32x4 fa[NF], fb[NF];
#pragma unroll
                for (int a = 0; a < NF; a++) fa[a] = frag(ta, ATR, wm * WT + a * 16 + l16, c);
#pragma unroll
                for (int b = 0; b < NF; b++) fb[b] = frag(tb, BTR, wn * WT + b * 16 + l16, c);
#pragma unroll
                for (int q = 0; q < 4; q++)
#pragma unroll
                    for (int a = 0; a < NF; a++)
#pragma unroll
                        for (int b = 0; b < NF; b++)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[b][q], fa[a][q], acc[a][b], 0, 0, 0);
            }
        };
        {
            using Even = std::integral_constant<int, 0>;
            using Odd = std::integral_constant<int, 1>;
            if (stages > 0) fetch(0, Even{});
            if (stages > 1) fetch(1, Odd{});
            for (int s = 0; s < stages; s += 2) {
                stage(s, Even{});
                if (s + 1 < stages) stage(s + 1, Odd{});
            }
        }
    };
    if (vec_a && vec_b) main_loop(std::true_type{}, std::true_type{});
    else if (vec_a) main_loop(std::true_type{}, std::false_type{});
    else if (vec_b) main_loop(std::false_type{}, std::true_type{});
    else main_loop(std::false_type{}, std::false_type{});

    // ---- epilogue: acc[a][b][r] = C[row wm WT + 16 a + l16][column wn WT + 16 b + 4 lg + r]
#pragma unroll
    for (int a = 0; a < NF; a++) {
        const int m = wm * WT + a * 16 + l16;
        if (m >= rows) continue;
        const size_t row = (size_t)(row0 + m);
        if constexpr (EPI == kSwigluFwd) {
            static_assert(EPI != kSwigluFwd || NF == 2, "a wavefront owns 16 gate columns and their 16 up columns");
            const int c = n0 / 2 + wn * 16 + 4 * lg, n = g.N - c;
            f32x4 h;
#pragma unroll
            for (int r = 0; r < 4; r++) h[r] = silu_f(acc[a][0][r]) * acc[a][NF - 1][r];
            const size_t o = row * g.ldo + c;
            store4((TA*)g.out0 + o, acc[a][0], n, g.vec_o != 0, false);
            store4((TA*)g.out1 + o, acc[a][NF - 1], n, g.vec_o != 0, false);
            store4((TA*)g.out2 + o, h, n, g.vec_o != 0, false);
        } else {
#pragma unroll
            for (int b = 0; b < NF; b++) {
                const int c = n0 + wn * WT + b * 16 + 4 * lg, n = g.N - c;
                if (n <= 0) continue;
                if constexpr (EPI == kStore) {
                    store4((TA*)g.out0 + row * g.ldo + c, acc[a][b], n, g.vec_o != 0, g.add != 0);
                } else if constexpr (EPI == kFloat) {
                    float* o = (float*)g.out0 + (long long)expert * g.out_stride + row * g.ldo + c;
                    store4(o, acc[a][b], n, g.vec_o != 0, g.add != 0);
                } else {
                    const f32x4 va = fetch4((const TA*)g.aux_a + row * g.N + c, n, g.vec_o != 0);
                    const f32x4 vb = fetch4((const TA*)g.aux_b + row * g.N + c, n, g.vec_o != 0);
                    f32x4 da, db;
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const float sg = logistic_f(va[r]), dh = acc[a][b][r];
                        da[r] = dh * vb[r] * sg * (1.0f + va[r] * (1.0f - sg));
                        db[r] = dh * va[r] * sg;
                    }
                    TA* o = (TA*)g.out0 + row * g.ldo + c;
                    store4(o, da, n, g.vec_o != 0, false);
                    store4(o + g.N, db, n, g.vec_o != 0, false);
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void sum_chunks_kernel(const float* __restrict__ part, int nparts, size_t n,
                                                         float* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float v = 0.f;
    for (int p = 0; p < nparts; p++) v += part[(size_t)p * n + i];
    out[i] = v;
}

// ---------------------------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------------------------
bool aligned(const void* p, int ld, size_t elem) { return ld % 4 == 0 && ((uintptr_t)p & (4 * elem - 1)) == 0; }

// Tiles of 64 x 64 where they give every compute unit a workgroup, 32 x 32 otherwise: at small sizes the time is
// the latency of the stages, and a quarter of the tile is four times the workgroups.
bool big_tiles(long long row_tiles_64, int n) { return row_tiles_64 * cdiv(n, 64) >= num_cus(); }

template <typename TA, int WT, bool BTR, Epilogue EPI>
hipError_t run_rows_wt(Args a, int n_cols, hipStream_t st) {
    constexpr int BM = 2 * WT;
    a.n_tiles = cdiv(n_cols, BM);
    const long long row_tiles = a.offsets ? (long long)a.M / BM + min(a.E, a.M) : cdiv(a.M, BM);
    // a multiple of eight, and for dealt_tile_of_block room for the last round of the XCDs
    const long long grid = ((row_tiles + (a.offsets && a.E > 64 ? 8 : 0)) * a.n_tiles + 7) / 8 * 8;
    if (grid >= (1LL << 31)) return hipErrorInvalidValue;
    gemm_f32_kernel<TA, WT, false, BTR, EPI, false><<<(unsigned)grid, kThreads, 0, st>>>(a);
    return hipGetLastError();
}
// n_cols: columns of the tile axis (both halves for kSwigluFwd)
template <typename TA, bool BTR, Epilogue EPI>
hipError_t run_rows(const Args& a, int n_cols, hipStream_t st) {
    if constexpr (EPI == kSwigluFwd) return run_rows_wt<TA, 32, BTR, EPI>(a, n_cols, st);
    else return big_tiles(cdiv(a.M, 64), n_cols) ? run_rows_wt<TA, 32, BTR, EPI>(a, n_cols, st)
                                                 : run_rows_wt<TA, 16, BTR, EPI>(a, n_cols, st);
}
template <typename TA, int WT>
hipError_t run_layers_wt(Args a, int groups, hipStream_t st) {
    a.m_tiles = cdiv(a.M, 2 * WT);
    a.n_tiles = cdiv(a.N, 2 * WT);
    a.E = groups;
    const long long grid = (((long long)groups * a.m_tiles + 8) * a.n_tiles + 7) / 8 * 8;      // as in run_rows_wt
    if (grid >= (1LL << 31)) return hipErrorInvalidValue;
    gemm_f32_kernel<TA, WT, true, true, kFloat, true><<<(unsigned)grid, kThreads, 0, st>>>(a);
    return hipGetLastError();
}
template <typename TA>
hipError_t run_layers(const Args& a, int groups, hipStream_t st) {
    return big_tiles((long long)groups * cdiv(a.M, 64), a.N) ? run_layers_wt<TA, 32>(a, groups, st)
                                                             : run_layers_wt<TA, 16>(a, groups, st);
}

}  // namespace

hipError_t f32_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st) {
    Args a = {};
    a.A = x; a.lda = s.d_model; a.B = w; a.ldb = s.d_model;
    a.M = s.T; a.N = s.E; a.K = s.d_model;
    a.out0 = z; a.ldo = s.E;
    const size_t el = s.dtype == UNIPOOL_BF16 ? 2 : 4;
    a.vec_a = aligned(x, s.d_model, el); a.vec_b = aligned(w, s.d_model, el); a.vec_o = aligned(z, s.E, 4);
    return s.dtype == UNIPOOL_BF16 ? run_rows<bf16, false, kFloat>(a, s.E, st) : run_rows<float, false, kFloat>(a, s.E, st);
}

hipError_t f32_ffn_gate_up(const unipool_shape& s, const void* x_perm, const int32_t* offsets, const void* wgu,
                           void* a_out, void* b_out, void* h_out, hipStream_t st, const int32_t* slot_of_row) {
    const int d = s.d_model, f = s.d_ff;
    Args a = {};
    a.A = x_perm; a.lda = d; a.B = wgu; a.ldb = d; a.b_stride = 2LL * f * d;
    a.M = s.T * s.k; a.N = f; a.K = d; a.offsets = offsets; a.E = s.E;
    a.gather = slot_of_row; a.gather_div = s.k;
    a.out0 = a_out; a.out1 = b_out; a.out2 = h_out; a.ldo = f;
    a.vec_a = aligned(x_perm, d, 4); a.vec_b = aligned(wgu, d, 4);
    a.vec_o = aligned(a_out, f, 4) && aligned(b_out, f, 4) && aligned(h_out, f, 4);
    return run_rows<float, false, kSwigluFwd>(a, 2 * f, st);
}

hipError_t f32_ffn_fwd(const unipool_shape& s, const void* x_perm, const int32_t* offsets, const void* wgu,
                       const void* wd, void* a_out, void* b_out, void* h_out, void* y, hipStream_t st,
                       const int32_t* slot_of_row) {
    const int d = s.d_model, f = s.d_ff;
    hipError_t e = f32_ffn_gate_up(s, x_perm, offsets, wgu, a_out, b_out, h_out, st, slot_of_row);
    if (e != hipSuccess) return e;
    Args a = {};
    a.A = h_out; a.lda = f; a.B = wd; a.ldb = f; a.b_stride = (long long)d * f;
    a.M = s.T * s.k; a.N = d; a.K = f; a.offsets = offsets; a.E = s.E;
    a.out0 = y; a.ldo = d;
    a.vec_a = aligned(h_out, f, 4); a.vec_b = aligned(wd, f, 4); a.vec_o = aligned(y, d, 4);
    return run_rows<float, false, kStore>(a, d, st);
}

hipError_t f32_ffn_dgrad(const unipool_shape& s, const void* dy, const void* a_in, const void* b_in,
                         const int32_t* offsets, const void* wgu, const void* wd, void* dx, void* d_act,
                         hipStream_t st) {
    const int d = s.d_model, f = s.d_ff;
    Args a = {};                                       // dH = dY W_down, then SwiGLU backward
    a.A = dy; a.lda = d; a.B = wd; a.ldb = f; a.b_stride = (long long)d * f;
    a.M = s.T * s.k; a.N = f; a.K = d; a.offsets = offsets; a.E = s.E;
    a.out0 = d_act; a.ldo = 2 * f; a.aux_a = a_in; a.aux_b = b_in;
    a.vec_a = aligned(dy, d, 4); a.vec_b = aligned(wd, f, 4);
    a.vec_o = aligned(d_act, f, 4) && aligned(a_in, f, 4) && aligned(b_in, f, 4);
    hipError_t e = run_rows<float, true, kSwigluBwd>(a, f, st);
    if (e != hipSuccess) return e;
    Args b = {};                                       // dX = [dA | dB] W_gate_up
    b.A = d_act; b.lda = 2 * f; b.B = wgu; b.ldb = d; b.b_stride = 2LL * f * d;
    b.M = s.T * s.k; b.N = d; b.K = 2 * f; b.offsets = offsets; b.E = s.E;
    b.out0 = dx; b.ldo = d;
    b.vec_a = aligned(d_act, 2 * f, 4); b.vec_b = aligned(wgu, d, 4); b.vec_o = aligned(dx, d, 4);
    return run_rows<float, true, kStore>(b, d, st);
}

hipError_t f32_ffn_wgrad(const unipool_shape& s, int n_layers, const void* const* x_perm_l,
                         const void* const* d_act_l, const void* const* h_l, const void* const* dy_l,
                         const int32_t* const* offsets_l, float* dwgu, float* dwd, int accumulate, hipStream_t st) {
    const int d = s.d_model, f = s.d_ff;
    Args a = {};                                       // d_w_gate_up[e][n][c] = sum d_act[row][n] x_perm[row][c]
    a.n_layers = n_layers; a.a_l = d_act_l; a.b_l = x_perm_l; a.off_l = offsets_l;
    a.lda = 2 * f; a.ldb = d; a.M = 2 * f; a.N = d; a.ldo = d; a.out_stride = 2LL * f * d;
    a.out0 = dwgu; a.add = accumulate;
    a.vec_a = (2 * f) % 4 == 0; a.vec_b = d % 4 == 0; a.vec_o = aligned(dwgu, d, 4);
    hipError_t e = run_layers<float>(a, s.E, st);
    if (e != hipSuccess) return e;
    Args b = {};                                       // d_w_down[e][c][n] = sum dy[row][c] h[row][n]
    b.n_layers = n_layers; b.a_l = dy_l; b.b_l = h_l; b.off_l = offsets_l;
    b.lda = d; b.ldb = f; b.M = d; b.N = f; b.ldo = f; b.out_stride = (long long)d * f;
    b.out0 = dwd; b.add = accumulate;
    b.vec_a = d % 4 == 0; b.vec_b = f % 4 == 0; b.vec_o = aligned(dwd, f, 4);
    return run_layers<float>(b, s.E, st);
}

namespace {

template <typename TA>
hipError_t route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz, float* dw, void* dx,
                        int dx_accumulate, const float* dsigma_part, float* d_sigma, float* wpart, hipStream_t st) {
    const int d = s.d_model, E = s.E, T = s.T, ez = dz_stride(s);
    const size_t el = sizeof(TA);
    // d_w_router = dz^T x.  The tokens are cut into chunks of at least 128 (two stages of a 32 x 32 tile) so that
    // the chunks' tiles fill the chip; the partial products are added in order.
    const int tiles = cdiv(E, 32) * cdiv(d, 32);
    const int nchunks = max(1, min(min(kRouteBwdSplit, T / 128), num_cus() / tiles));
    const int chunk = cdiv(cdiv(T, nchunks), 64) * 64;
    const int used = cdiv(T, chunk);
    Args a = {};
    a.A = dz; a.lda = ez; a.B = x; a.ldb = d; a.M = E; a.N = d; a.K = T; a.chunk = chunk;
    a.sum_part = dsigma_part; a.sum_n = cdiv(T, dz_tokens_per_block(s)); a.sum_out = d_sigma;
    a.out0 = used > 1 ? wpart : dw; a.ldo = d; a.out_stride = (long long)E * d;
    a.vec_a = aligned(dz, ez, el); a.vec_b = aligned(x, d, el); a.vec_o = aligned(a.out0, d, 4);
    hipError_t e = run_layers<TA>(a, used, st);
    if (e != hipSuccess) return e;
    if (used > 1) {
        const size_t n = (size_t)E * d;
        sum_chunks_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(wpart, used, n, dw);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    Args b = {};                                       // dx (+)= dz W
    b.A = dz; b.lda = ez; b.B = w; b.ldb = d; b.M = T; b.N = d; b.K = E;
    b.out0 = dx; b.ldo = d; b.add = dx_accumulate;
    b.vec_a = aligned(dz, ez, el); b.vec_b = aligned(w, d, el); b.vec_o = aligned(dx, d, el);
    return run_rows<TA, true, kStore>(b, d, st);
}

}  // namespace

hipError_t f32_route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz, float* dw,
                            void* dx, int dx_accumulate, const float* dsigma_part, float* d_sigma, float* wpart,
                            hipStream_t st) {
    return s.dtype == UNIPOOL_BF16
               ? route_bwd_mm<bf16>(s, x, w, dz, dw, dx, dx_accumulate, dsigma_part, d_sigma, wpart, st)
               : route_bwd_mm<float>(s, x, w, dz, dw, dx, dx_accumulate, dsigma_part, d_sigma, wpart, st);
}

}  // namespace unipool
