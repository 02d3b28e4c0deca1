// bfloat16 grouped GEMMs on the CDNA4 matrix cores (v_mfma_f32_16x16x32_bf16), float accumulate.
//
// Two kernels cover every dense contraction of the layer:
//
//   gemm_xw  : C[rows of e, N] = X[rows of e, K] * W_e          (row-grouped; forward, dgrad, router)
//              X is K-contiguous.  W_e is either [N][K] (K-contiguous) or [K][N] (N-contiguous).
//   gemm_ptq : out[e][i][j] (+)= sum_rows P[row][i] * Q[row][j]  (reduction over the rows of e,
//              possibly chained over several layers; weight gradients)
//
// Common structure
//   * One workgroup of 8 wavefronts per CU, a 256 x 256 output tile, 128 accumulator registers per
//     lane (gemm_xw also: two workgroups of 4 wavefronts, 128 x 128 each, see tile_form); fragments have one register set each and are refilled in place as their last use passes.
//   * Operand tiles go global -> LDS directly (global_load_lds_dwordx4), several stages deep, one
//     barrier per stage.  The loads are issued through inline assembly so that the wait counts
//     are ours: the compiler would otherwise wait for every outstanding load before any LDS read.
//   * LDS tiles hold 16-byte chunks in XOR-swizzled positions; a direct-to-LDS load writes 64
//     consecutive chunks, so the swizzle is applied on the global address of each lane.
//   * Operands whose reduction index is the strided one in memory are read from LDS with pairs of
//     ds_read_b64_tr_b16, each of which hands a lane four consecutive reduction indices of one column.
//   * The weight fragment is the MFMA A operand and the activation fragment the B operand, so a
//     lane ends up with four consecutive output columns of one row: results are staged through
//     LDS and leave the CU as 16-byte row segments.
//   * Row groups come from a device-side tile table; nothing is read back to the host.  Tiles are
//     walked in a fixed order that keeps the tiles of one expert on one XCD (workgroup ids are dealt
//     round-robin to the 8 XCDs, each of which has its own L2), runs the two row tiles of an expert
//     side by side so that they share its weight tiles in L2, and lets a workgroup request the first
//     stages of its next tile before the epilogue of the current one.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "gemm_common.h"

namespace unipool {

namespace {

// Profiling builds (-DUNIPOOL_PHASE_TIMES) add up, per workgroup, the time the first wavefront
// spends in the three phases of a gemm_xw tile (100 MHz ticks): pipeline fill, K loop, epilogue; one row per
// workgroup and launch slot.
#ifdef UNIPOOL_PHASE_TIMES
__device__ unsigned long long g_phase_times[1024][8];
#define PHASE_STAMP(var) const long long var = wall_clock64()
#define PHASE_COMMIT(t0, t1, t2, t3)                                                         \
    if (threadIdx.x == 0 && blockIdx.x < 256) {                                              \
        unsigned long long* pt_ = g_phase_times[blockIdx.x + 256 * (g.launch_slot & 3)];     \
        pt_[0] += (unsigned long long)((t1) - (t0));                                         \
        pt_[1] += (unsigned long long)((t2) - (t1));                                         \
        pt_[2] += (unsigned long long)((t3) - (t2));                                         \
        pt_[3] += 1ull;                                                                      \
        pt_[4] += (unsigned long long)acc_wait_;                                             \
        pt_[5] += (unsigned long long)acc_bar_;                                              \
        pt_[6] += (unsigned long long)acc_cyc_;                                              \
    }
#define PHASE_CLOCK(var) const long long var = clock64()
#else
#define PHASE_STAMP(var)
#define PHASE_COMMIT(t0, t1, t2, t3)
#endif

// Inclusive prefix sum over the 512 threads of a workgroup; wsum: eight words of LDS that nobody else uses.
__device__ __forceinline__ int scan512(int v, int* wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    if (lane == 63) wsum[wave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 7; w++)
        if (w < wave) v += wsum[w];
    return v;
}

// What reductions read past their end.  Never written.
__device__ __align__(256) uint32_t g_zero_page[64];
// Its address, once and for all: named in a loop it would be fetched from memory there each time.
__device__ __forceinline__ const void* zero_page() {
    const void* p = g_zero_page;
    asm volatile("" : "+s"(p));
    return p;
}

// Size class of a row count, larger counts in later classes: steps of 16 rows below 2048, a sixteenth of a
// power of two above.
constexpr int kSizeClasses = 512;
__device__ __forceinline__ int size_class(int rows) {
    if (rows < 2048) return rows >> 4;
    const int e = 31 - __clz(rows);
    return 128 + (e - 11) * 16 + ((rows >> (e - 4)) & 15);
}

// Tile table of one launch sequence, by one workgroup: its time is a chain of LDS latencies, so there is
// nothing in it that grows with E.  Experts are ordered by size class with a counting sort (two 512-wide
// scans); comparing every pair of row counts instead, as an exact sort by rank, cost 2 x 512 LDS reads per
// wavefront and took 24 us at E = 512 and 16 us at E = 192 (now 5.2 and 5.4, of which 4 are the launch).  The order of experts of one class
// follows the arrival of LDS atomics: it decides where a tile runs, never what it computes.
// Workgroup b builds the table of the tiles of tabs.bm[b] rows.
struct TileTables {
    int32_t* meta[2];
    int bm[2];
    int32_t* pair_cnt;        // meeting counters to clear
};
__global__ __launch_bounds__(512) void build_tiles_kernel(const int32_t* __restrict__ offsets, int E, const TileTables tabs) {
    int32_t* meta = tabs.meta[blockIdx.x];
    const int BM = tabs.bm[blockIdx.x];
    const bool pad_even = BM > 128;
    __shared__ int hist[kSizeClasses];    // experts per class, then the next free rank of the class
    __shared__ int ltiles[512];           // tiles of the expert at a given place
    __shared__ int wsum[2][8];
    const int t = threadIdx.x;
    int r0 = 0, r1 = 0;
    if (t < E) {
        r0 = offsets[t];
        r1 = offsets[t + 1];
    }
    hist[t] = 0;
    ltiles[t] = 0;
    if (blockIdx.x == 0)
        for (int i = t; i < kPairCap / 4; i += 512) reinterpret_cast<int4*>(tabs.pair_cnt)[i] = make_int4(0, 0, 0, 0);
    const int rt = r1 - r0;
    const int nt = (rt + BM - 1) / BM;
    // Every expert takes an even number of places in the list (the odd one out is an entry without
    // rows, which the workgroups skip): the kernels hand out the list in pairs of row tiles that run
    // side by side and share the weight tile through L2, and a pair must not straddle two experts.
    const int ns = pad_even ? (nt + 1) & ~1 : nt;
    __syncthreads();
    const int cls = kSizeClasses - 1 - size_class(rt);          // descending sizes
    if (t < E) atomicAdd(&hist[cls], 1);
    __syncthreads();
    const int h = hist[t];
    const int upto = scan512(h, wsum[0]);
    hist[t] = upto - h;                   // a class's first rank
    __syncthreads();
    // Order of the experts in the tile list.  The persistent workgroups walk the list in a fixed
    // pattern (one eighth of it per XCD, dealt in rounds to the workgroups of the XCD), so the list
    // is laid out for them: experts sorted by size, descending, are dealt to the eight parts in
    // serpentine order (0..7, 7..0, ...), which gives every XCD the same amount of work to within
    // one small expert and makes the tiles that run at the same time equally long.
    int dense = 0;                        // place of the expert: experts of the parts before its own, then its lap
    if (t < E) {
        const int rank = atomicAdd(&hist[cls], 1);
        const int lap = rank / kNumXcd, posn = rank % kNumXcd;
        const int part = (lap & 1) ? kNumXcd - 1 - posn : posn;
        // the last lap is short: its experts sit in the first parts, or in the last ones if it runs backwards
        const int laps = E / kNumXcd, left = E % kNumXcd;
        dense = part * laps + ((laps & 1) ? max(0, part - (kNumXcd - left)) : min(part, left)) + lap;
        ltiles[dense] = ns;
    }
    __syncthreads();
    const int mine = ltiles[t];
    const int end = scan512(mine, wsum[1]);
    ltiles[t] = end - mine;               // first tile of the expert at place t
    if (t == 511) meta[0] = end;
    __syncthreads();
    // The rows of an expert are cut into equal tiles (multiples of 16 rows, the MFMA's row count)
    // rather than into full tiles plus a remainder: tiles that share an expert's weights then take
    // equally long and stay in step, so the second reader of a weight tile still finds it in L2.
    if (t < E) {
        const int per = nt > 0 ? (((rt + nt - 1) / nt + 15) / 16) * 16 : 0;
        int4* m = reinterpret_cast<int4*>(meta + kTileBase) + ltiles[dense];
        for (int i = 0; i < ns; i++)
            m[i] = make_int4(t, r0 + i * per, max(0, min(per, r1 - (r0 + i * per))), 0);
    }
}

// ---------------------------------------------------------------------------------------------
// gemm_xw
// ---------------------------------------------------------------------------------------------
// One 256 x 256 output tile, eight wavefronts (two per SIMD), or one of 128 x 128, four wavefronts and half the LDS, so
// that a CU runs two of them.  Wavefront (wm, wn) owns the 64
// columns of group wn and every second 32-row strip starting at wm; in the large tile both wavefronts of a column
// group sit on the same SIMD, so a SIMD always carries the same share of the tile, however many
// strips hold rows.  MTV = strips of THIS wavefront that hold rows (0..4, small tile 0..2), LH = only the upper 16
// rows of its last strip do; the body is instantiated per (MTV, LH) so that the K loop is
// straight-line code and absent rows have no MFMAs.
// The products are v_mfma_f32_16x16x32_bf16 (at the card's power limit this form sustains about a
// sixth more than 32x32x16): a strip is two 16-row halves, the 64 columns four 16-column blocks.


// pre: what the previous tile has already requested for this one (bit 0: X(0) and W(0), bit 1: W(1));
// g0: number of K stages this workgroup has run before this tile (the LDS buffers rotate on).
template <int BM, int BN, int BK, int NS, bool WK, int EPI, bool KTAIL, bool ADD, int MTV, bool LH>
__device__ __forceinline__ void xw_tile(const GemmArgs& g, char* smem, TileRef cur, TileRef nxt, int pre,
                                        int g0) {
    constexpr int NW = BN / 32;                   // wavefronts: two along the rows, one per 64 columns
    constexpr int NWN = NW / 2;
    constexpr int TN = 2;
    constexpr int XBYTES = BM * BK * 2;
    constexpr int WBYTES = BN * BK * 2;
    constexpr int XI = BM * BK / 8 / (NW * 64);   // direct-to-LDS loads per wavefront, X tile
    constexpr int WI = BN * BK / 8 / (NW * 64);
    constexpr int KS = BK / 32;                   // slices of 32 reduction indices per stage
    static_assert(KS == 2, "the stage body below is written for two slices");
    static_assert((BM == 256 && NW == 8) || (BM == 128 && NW == 4), "strips of 32 rows interleaved by 2");
    using XT = KTile<BK>;
    using WTK = KTile<BK>;
    using WTN = NTile16<BN>;

    // The per-MTV bodies are alternatives of one switch.  Their set-up code is identical, and if
    // the compiler merges it in front of the switch the merged values stay live across all the
    // bodies and spill; spill code is scratch traffic, whose wait counts would then serialise the
    // direct-to-LDS pipeline.  Making the inputs opaque here keeps every body self-contained.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    int expert = __builtin_amdgcn_readfirstlane(cur.expert);
    int row0 = __builtin_amdgcn_readfirstlane(cur.row0);
    int rows = __builtin_amdgcn_readfirstlane(cur.rows);
    int nt = __builtin_amdgcn_readfirstlane(cur.nt);
    pre = __builtin_amdgcn_readfirstlane(pre);
    g0 = __builtin_amdgcn_readfirstlane(g0);
    asm volatile("" : "+s"(expert), "+s"(row0), "+s"(rows), "+s"(nt), "+s"(pre), "+s"(g0));
    PHASE_STAMP(t_begin);
#ifdef UNIPOOL_PHASE_TIMES
    long long acc_wait_ = 0, acc_bar_ = 0, acc_cyc_ = 0;
#endif
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % NWN, wm = wave / NWN;
    const unsigned lds0 = lds_addr_of(smem);
    const int n0 = nt * BN;                 // first column of the tile (plain epilogues)
    const int f0 = nt * (BN / 2);           // first column per half (SWIGLU_FWD)

    // ---- per-lane source pointers of the direct-to-LDS loads ----------------------------------
    // Load i of a wavefront fills LDS chunks (i*NW + wave)*64 .. +63: 8 rows of 128 bytes.  Loads
    // past the tile's last row are left out (xload[i] false, wave-uniform): what the MFMAs then read
    // for those rows is stale, and it only reaches output rows that are never stored.
    const char* xsrc[XI];
    bool xload[XI];
    const char* wsrc[WI];
    const size_t wstep = WK ? (size_t)BK * 2 : (size_t)BK * g.ldw * 2;      // bytes per K step
    auto set_sources = [&](int t_expert, int t_row0, int t_rows, int t_nt) {
        const bf16* We = g.W + (long long)t_expert * g.w_stride;
        const int t_n0 = t_nt * BN, t_f0 = t_nt * (BN / 2);
#pragma unroll
        for (int i = 0; i < XI; i++) {
            const int q = (i * NW + wave) * 64 + lane;
            const int row = q / XT::CPR;
            const int cc = (q % XT::CPR) ^ XT::swz(row);
            int grow = t_row0 + min(row, t_rows - 1);
            if (g.gather != nullptr) grow = g.gather[grow] / g.gather_div;
            xsrc[i] = reinterpret_cast<const char*>(g.X + (size_t)grow * g.ldx + cc * 8);
            xload[i] = ((i * NW + wave) * 64 / XT::CPR) < ((t_rows + 7) & ~7);
        }
        if constexpr (WK) {
#pragma unroll
            for (int i = 0; i < WI; i++) {
                const int q = (i * NW + wave) * 64 + lane;
                const int row = q / WTK::CPR;
                const int cc = (q % WTK::CPR) ^ WTK::swz(row);
                int wrow;
                if constexpr (EPI == EPI_SWIGLU_FWD) {
                    const int half = row / (BN / 2);
                    wrow = half * g.up_rows + min(t_f0 + row % (BN / 2), g.N - 1);
                } else {
                    wrow = min(t_n0 + row, g.N - 1);
                }
                wsrc[i] = reinterpret_cast<const char*>(We + (size_t)wrow * g.ldw + cc * 8);
            }
        } else {
#pragma unroll
            for (int i = 0; i < WI; i++) {
                const int q = (i * NW + wave) * 64 + lane;
                const int krow = q / WTN::CPR;
                const int cc = (q % WTN::CPR) ^ WTN::swz(krow);
                const int col = min(t_n0 + cc * 8, g.N - 8);
                wsrc[i] = reinterpret_cast<const char*>(We + (size_t)krow * g.ldw + col);
            }
        }
    };
    set_sources(expert, row0, rows, nt);

    // acc[tm][mh][nb]: strip tm of this wavefront, 16-row half mh, 16-column block nb
    f32x4 acc[MTV > 0 ? MTV : 1][2][4];
#pragma unroll
    for (int tm = 0; tm < MTV; tm++)
#pragma unroll
        for (int mh = 0; mh < 2; mh++)
#pragma unroll
            for (int nb = 0; nb < 4; nb++) acc[tm][mh][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS rows (K-contiguous W) or columns (N-contiguous W) of this wavefront's two fragments
    int wpos[TN];
    if constexpr (EPI == EPI_SWIGLU_FWD) {
        wpos[0] = wn * 32;
        wpos[1] = BN / 2 + wn * 32;
    } else {
        wpos[0] = wn * 64;
        wpos[1] = wn * 64 + 32;
    }

    const int nk = KTAIL ? (g.K + BK - 1) / BK : g.K / BK;
    // ---- software pipeline ----------------------------------------------------------------------
    // LDS holds NSX stages of the X tile and NSW stages of the W tile (BK reduction indices each).
    // While stage kt is multiplied, X(kt+1), W(kt+1) and W(kt+2) are landing, and from its meeting
    // point on X(kt+2) as well.  A stage is KS slices of 32 indices; every fragment has one register
    // set, and the LDS reads that refill it are interleaved one by one with the MFMAs (issue is in
    // order: a burst of LDS reads would hold back the MFMAs behind it).
    constexpr int NSX = NS, NSW = NS + 1;
    constexpr int WBASE = NSX * XBYTES;
    static_assert(NSX == 2 && NSW == 3, "buffer rotation and wait counts below");
    // Stage kt of this tile lives in X buffer (g0 + kt) mod 2 and W buffer (g0 + kt) mod 3: the
    // buffers rotate on from tile to tile, so the first stages of the next tile can be requested
    // while this tile's last stage and epilogue still hold theirs.
    // The loop carries their LDS offsets, of stage kt: xo (the other one: xo ^ XBYTES), and of W(kt), W(kt+1), W(kt+2).
    static_assert((XBYTES & (XBYTES - 1)) == 0, "the other X buffer by an exclusive or");
    unsigned xo = (g0 & 1) * XBYTES;
    unsigned wo0 = WBASE + g0 % 3 * WBYTES, wo1 = WBASE + (g0 + 1) % 3 * WBYTES, wo2 = WBASE + (g0 + 2) % 3 * WBYTES;
    // Fragments of one slice: W block nb (16 columns x 32 indices, the MFMA A operand) and X fragment
    // a (16 rows x 32 indices, the B operand: a < MTV the upper rows of strip a, a >= MTV the lower rows
    // of strip a - MTV), one register set each.  A slice is two halves; slot nb * MTV + tm of the first
    // takes the upper rows of the strips, slot nb * M2 + tm of the second the lower rows, so X[0 .. MTV)
    // and W[0..2] are free for the next slice's data during the second half, W[3] and the other X
    // fragments at its end.
    static_assert(!LH || MTV >= 2, "a lone strip is always computed whole");
    constexpr int M2 = MTV - (LH ? 1 : 0);          // strips whose lower 16 rows are computed
    constexpr int NXF = MTV + M2;
    constexpr int HM1 = 4 * MTV, HM2 = 4 * M2;      // MFMA slots of the two halves of a slice
    bf16x8 wfr[4], xfr[NXF > 0 ? NXF : 1];
    // per-lane part of the fragment addresses (rows that are multiples of 16 further down add whole rows)
    const int l16 = lane & 15, lg = lane >> 4;
    const int koff0 = XT::off(l16, lg), koff1 = XT::off(l16, 4 + lg);       // K-contiguous tiles, slice 0 / 1
    static_assert(XT::CPR == 8, "a slice is four 16-byte chunks of a 128-byte row");
    [[maybe_unused]] int noff[4];                                         // N-contiguous W
    if constexpr (!WK) {
#pragma unroll
        for (int nb = 0; nb < 4; nb++) noff[nb] = WTN::frag_off(wpos[nb >> 1] + 16 * (nb & 1), lane);
    }
    constexpr int ROWB = BK * 2;                                           // bytes per K-contiguous row
    auto load_w = [&](unsigned buf, int ks, int nb) {
        const char* wb = smem + buf;
        if constexpr (WK) {
            wfr[nb] = lds_read16(wb + (wpos[nb >> 1] + 16 * (nb & 1)) * ROWB + (ks ? koff1 : koff0));
        } else {
            const char* p = wb + ks * (32 * WTN::CPR * 16) + noff[nb];
            wfr[nb] = lds_read_tr8(p, p + 4 * WTN::CPR * 16);
        }
    };
    auto load_x = [&](unsigned buf, int ks, int a) {
        const int tm = a < MTV ? a : a - MTV, mh = a < MTV ? 0 : 1;
        const char* xb = smem + buf;
        xfr[a] = lds_read16(xb + ((wm + 2 * tm) * 32 + 16 * mh) * ROWB + (ks ? koff1 : koff0));
    };
    auto mfma_one = [&](int a, int nb) {
        const int tm = a < MTV ? a : a - MTV, mh = a < MTV ? 0 : 1;
        acc[tm][mh][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfr[nb], xfr[a], acc[tm][mh][nb], 0, 0, 0);
    };
    // KTAIL: K is not a multiple of BK; chunks past K come from a page of zeros in both operands
    static_assert(!KTAIL || !WK, "the reduction tail is implemented for N-contiguous W only");
    [[maybe_unused]] const void* const zeros = KTAIL ? zero_page() : nullptr;
    int xk[KTAIL ? XI : 1], wk[KTAIL ? WI : 1];   // first reduction index of the lane's chunk / row
    if constexpr (KTAIL) {
#pragma unroll
        for (int i = 0; i < XI; i++) {
            const int q = (i * NW + wave) * 64 + lane;
            xk[i] = ((q % XT::CPR) ^ XT::swz(q / XT::CPR)) * 8;
        }
#pragma unroll
        for (int i = 0; i < WI; i++) wk[i] = ((i * NW + wave) * 64 + lane) / WTN::CPR;
    }
    // load i of stage kt of the tile the sources point at, into the given buffer
    auto issue_x = [&](int kt, int i, unsigned buf) {
        if (!xload[i]) return;
        const char* src = xsrc[i] + (size_t)kt * BK * 2;
        if constexpr (KTAIL)
            if (kt * BK + xk[i] >= g.K) src = reinterpret_cast<const char*>(zeros);
        glds16(src, lds0 + buf + ((i * NW + wave) * 64) * 16);
    };
    auto issue_w = [&](int kt, int i, unsigned buf) {
        const char* src = wsrc[i] + (size_t)kt * wstep;
        if constexpr (KTAIL)
            if (kt * BK + wk[i] >= g.K) src = reinterpret_cast<const char*>(zeros);
        glds16(src, lds0 + buf + ((i * NW + wave) * 64) * 16);
    };
    // One stage.  The wavefronts meet between the halves of the second slice: stage kt+1 has landed,
    // nobody reads stage kt any more, and the second half, whose operands are in registers, covers the
    // first fragment loads of stage kt+1.  Loads go out two stages ahead, into the buffers that the
    // meeting points release: W(kt+2), whose buffer stage kt-1 held, during the MFMAs ahead of the
    // meeting (IW), X(kt+2), whose buffer is the one stage kt is reading, right behind it.  They are
    // spread between the MFMAs: a wavefront whose load finds the address unit's queue full stands
    // still, MFMAs included, so a burst of loads from all wavefronts at once would cost the matrix
    // cores the whole time the queue takes to drain.
    auto stage_body = [&](auto iw_c, int kt) {
        constexpr bool IW = decltype(iw_c)::value;
        constexpr int SL = 2 * HM1 + HM2;             // slots before the meeting point
        const bool ix = kt + 2 < nk;                  // X(kt+2) exists
        auto w_loads = [&](int slot) {
            if constexpr (IW) {
#pragma unroll
                for (int u = 0; u < WI; u++)
                    if (u * SL / WI == slot) issue_w(kt + 2, u, wo2);
            }
        };
        auto x_loads = [&](int slot) {
#pragma unroll
            for (int u = 0; u < XI; u++)
                if (u * HM2 / XI == slot && ix) issue_x(kt + 2, u, xo);
        };
        if constexpr (SL == 0 && IW) {
#pragma unroll
            for (int u = 0; u < WI; u++) issue_w(kt + 2, u, wo2);
        }
        auto first_half = [&](int ks, int slot0) {         // of stage kt
#pragma unroll
            for (int sl = 0; sl < HM1; sl++) {
                mfma_one(sl % MTV, sl / MTV);
                if (sl == 0) load_w(wo0, ks, 3);                       // what the previous slice still held
                if (sl >= 1 && sl <= M2) load_x(xo, ks, MTV + sl - 1);
                w_loads(slot0 + sl);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto second_half = [&](unsigned nxo, unsigned nwo, int nks, int slot0) {       // where the slice that follows is
#pragma unroll
            for (int sl = 0; sl < HM2; sl++) {
                mfma_one(MTV + sl % M2, sl / M2);
                if (sl < MTV) load_x(nxo, nks, sl);
                if (sl >= M2 && sl % M2 == 0) load_w(nwo, nks, sl / M2 - 1);
                if (slot0 >= 0) w_loads(slot0 + sl);
                else x_loads(sl);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        first_half(0, 0);
        second_half(xo, wo0, 1, HM1);
        first_half(1, HM1 + HM2);
        // X(kt+1) and W(kt+1) must have landed.  Loads complete in issue order, and the only ones
        // issued after those two batches are the W loads of stage kt+2.
#ifdef UNIPOOL_PHASE_TIMES
        PHASE_CLOCK(c0_);
#endif
        if (nk - 2 - kt >= 1) wait_vmcnt<WI>();
        else wait_vmcnt<0>();
#ifdef UNIPOOL_PHASE_TIMES
        PHASE_CLOCK(c1_);
#endif
        lds_barrier();
#ifdef UNIPOOL_PHASE_TIMES
        PHASE_CLOCK(c2_);
        acc_wait_ += c1_ - c0_;
        acc_bar_ += c2_ - c1_;
#endif
        if constexpr (HM2 == 0) {
            if (ix) {
#pragma unroll
                for (int u = 0; u < XI; u++) issue_x(kt + 2, u, xo);
            }
        }
        second_half(xo ^ XBYTES, wo1, 0, -1);         // after the last stage: unused, in bounds
        const unsigned w = wo0;
        wo0 = wo1; wo1 = wo2; wo2 = w;
        xo ^= XBYTES;
    };
    // prologue: X(0) W(0) X(1) W(1) W(2), less what the previous tile has requested already
    if (!(pre & 1)) {
#pragma unroll
        for (int i = 0; i < XI; i++) issue_x(0, i, xo);
#pragma unroll
        for (int i = 0; i < WI; i++) issue_w(0, i, wo0);
    }
    if (nk > 1) {
#pragma unroll
        for (int i = 0; i < XI; i++) issue_x(1, i, xo ^ XBYTES);
        if (!(pre & 2)) {
#pragma unroll
            for (int i = 0; i < WI; i++) issue_w(1, i, wo1);
        }
    }
    if (nk > 2) {
#pragma unroll
        for (int i = 0; i < WI; i++) issue_w(2, i, wo2);
    }
    // stage 0 has landed when at most the two W batches of stages 1 and 2 are outstanding (the X
    // batch of stage 1, which may be shorter than XI loads, then has landed too: stricter than needed)
    if (nk >= NSW) wait_vmcnt<(NSW - 1) * WI>();
    else wait_vmcnt<0>();
    lds_barrier();
    PHASE_STAMP(t_filled);
#ifdef UNIPOOL_PHASE_TIMES
    PHASE_CLOCK(cl0_);
#endif
#pragma unroll
    for (int a = 0; a < MTV; a++) load_x(xo, 0, a);
    if constexpr (MTV > 0) {
#pragma unroll
        for (int nb = 0; nb < 3; nb++) load_w(wo0, 0, nb);
    }
    {
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        // stage 0: the prologue has issued X(1) and W(2) already
        stage_body(F{}, 0);
        int kt = 1;
        for (; kt + 2 < nk; kt++) stage_body(T{}, kt);
        for (; kt < nk; kt++) stage_body(F{}, kt);
    }
    lds_barrier();   // every wavefront is done with the operand tiles
    PHASE_STAMP(t_looped);
    // The buffers of the last stage become the staging space of the epilogue; the others take the
    // first stages of the next tile now, so that its pipeline is full when the epilogue ends.
    constexpr bool PREW1 = Staging<EPI, NW>::PREW1;
    if constexpr (!KTAIL) {
        if (nxt.valid) {
            set_sources(nxt.expert, nxt.row0, nxt.rows, nxt.nt);
#pragma unroll
            for (int i = 0; i < XI; i++) issue_x(0, i, xo);
#pragma unroll
            for (int i = 0; i < WI; i++) issue_w(0, i, wo0);
            if (PREW1 && nk > 1) {
#pragma unroll
                for (int i = 0; i < WI; i++) issue_w(1, i, wo1);
            }
        }
    }
#ifdef UNIPOOL_PHASE_TIMES
    PHASE_CLOCK(cl1_);
    acc_cyc_ = cl1_ - cl0_;
#endif

    // ---- epilogue ---------------------------------------------------------------------------------
    // acc[tm][mh][nb][r] = C[row (wm + 2 tm)*32 + 16 mh + lane%16][column 16 nb + 4*(lane/16) + r of the wavefront's 64]

    if constexpr (EPI == EPI_F32) {
        float* out = reinterpret_cast<float*>(g.out0);
#pragma unroll
        for (int tm = 0; tm < MTV; tm++)
#pragma unroll
            for (int mh = 0; mh < 2; mh++) {
                if (LH && tm == MTV - 1 && mh == 1) continue;
                const int r_in = (wm + 2 * tm) * 32 + 16 * mh + l16;
                if (r_in < rows) {
                    float* orow = out + (size_t)(row0 + r_in) * g.ldo;
#pragma unroll
                    for (int nb = 0; nb < 4; nb++)
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            const int col = n0 + wpos[nb >> 1] + 16 * (nb & 1) + 4 * lg + r;
                            if (col < g.N) orow[col] = acc[tm][mh][nb][r];
                        }
                }
            }
    } else {
        using SG = Staging<EPI, NW>;
        // Staging area of this wavefront: region 0 is the X buffer of the last stage, region 1 its W
        // buffer, region 2 (SwiGLU backward only) the W buffer that would otherwise hold W(1) of the
        // next tile.
        const int region = wave / SG::RW;
        // (by now the offsets are those of stage nk: the last stage's are xo ^ XBYTES and wo2)
        const unsigned rbase = region == 0 ? xo ^ XBYTES : region == 1 ? wo2 : wo1;
        char* stg = smem + rbase + (wave % SG::RW) * SG::WSTG;
        char* stg2 = nullptr;
        if constexpr (SG::SPLIT)       // second areas: buffer 2, the rest behind the first areas in buffer 1
            stg2 = smem + (wave < SG::RW ? wo1 + wave * SG::AREA : wo2 + (NW - SG::RW + wave - SG::RW) * SG::AREA);
        xw_staged_epilogue<EPI, NW, MTV, LH, ADD>(epi_args(g), AccArray<MTV>{acc}, stg, stg2, rows, row0, n0, f0, wm, 2, wn,
                                                  lane);
    }
    PHASE_STAMP(t_end);
    PHASE_COMMIT(t_begin, t_filled, t_looped, t_end);
}

template <int BM, int BN, int BK, int NS, bool WK, int EPI, bool KTAIL, bool ADD>
__global__ __launch_bounds__(2 * BN, 2) void gemm_xw_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    TileWalk walk(g);
    const int wm = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BN);        // upper half of the wavefronts: odd strips
    const int nk = KTAIL ? (g.K + BK - 1) / BK : g.K / BK;
    TileRef cur = walk.next(g);
    int pre = 0, g0 = 0;
#ifdef UNIPOOL_PHASE_TIMES
    int tile_i_ = 0;
#endif
    while (cur.valid) {
        const TileRef nxt = walk.next(g);
#ifdef UNIPOOL_PHASE_TIMES
        if (threadIdx.x == 0 && (g.launch_slot & 3) == 1 && tile_i_ < 8)
            g_phase_times[768 + (blockIdx.x & 255)][tile_i_] = (unsigned long long)wall_clock64();
        tile_i_++;
#endif
        meet_partner(g, cur);
        // strips wm, wm+2, ... of this wavefront that hold rows, and whether the last of them is the
        // tile's last strip with rows in its upper half only; every body runs the same barriers
        const int strips = (cur.rows + 31) >> 5;
        const int mtv = max(0, (strips - wm + 1) >> 1);
        const bool lh = mtv >= 2 && wm + 2 * (mtv - 1) == strips - 1 && (((cur.rows + 15) >> 4) & 1) != 0;
        const int form = 2 * mtv + (lh ? 1 : 0);
        if constexpr (BM == 256) {
            switch (form) {
                case 0: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 0, false>(g, smem, cur, nxt, pre, g0); break;
                case 2: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 1, false>(g, smem, cur, nxt, pre, g0); break;
                case 4: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 2, false>(g, smem, cur, nxt, pre, g0); break;
                case 5: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 2, true>(g, smem, cur, nxt, pre, g0); break;
                case 6: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 3, false>(g, smem, cur, nxt, pre, g0); break;
                case 7: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 3, true>(g, smem, cur, nxt, pre, g0); break;
                case 9: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 4, true>(g, smem, cur, nxt, pre, g0); break;
                default: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 4, false>(g, smem, cur, nxt, pre, g0); break;
            }
        } else {
            switch (form) {
                case 0: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 0, false>(g, smem, cur, nxt, pre, g0); break;
                case 2: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 1, false>(g, smem, cur, nxt, pre, g0); break;
                case 5: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 2, true>(g, smem, cur, nxt, pre, g0); break;
                default: xw_tile<BM, BN, BK, NS, WK, EPI, KTAIL, ADD, 2, false>(g, smem, cur, nxt, pre, g0); break;
            }
        }
        lds_barrier();                // the staging space is free: the next tile may load into it
        pre = (!KTAIL && nxt.valid) ? ((Staging<EPI, BN / 32>::PREW1 && nk > 1) ? 3 : 1) : 0;
        g0 = (g0 + nk) % 6;           // the buffers repeat with period 2 and 3
        cur = nxt;
    }
}

// ---------------------------------------------------------------------------------------------
// gemm_ptq: out[e][i][j] (+)= sum_l sum_{row in group e of layer l} P_l[row][i] * Q_l[row][j]
// ---------------------------------------------------------------------------------------------
// One weight gradient of all experts (or one matrix cut into chunks of rows, whose partial products are the "experts").
struct PtqArgs {
    const void* const* P;        // device arrays of device pointers, one entry per layer
    const void* const* Q;
    const void* P1;              // the operands of a single layer or matrix (P, Q and off are null then)
    const void* Q1;
    int chunk_rows, total_rows;
    int mdim, ndim;
    int m_tiles, n_tiles;
    float* out;
    long long out_stride;        // elements between experts
};
// What a launch computes: the tiles of `first`, then those of `second` (none where it is not used).
struct PtqLaunch {
    PtqArgs first, second;
    const int32_t* const* off;   // row offsets of the experts, one entry per layer; or
    const int32_t* off1;         // those of a single layer; or none: chunks
    int n_layers, E, accumulate;
};

// BOTH: the tiles of launch.second follow those of launch.first (if it has any), and the operands of a single layer or matrix may
// come by pointer; without it launch.first alone, by table.  STREAM: see the epilogue.
template <int BK, int NS, int NW, bool STREAM, bool BOTH>
__global__ __launch_bounds__(64 * NW) void gemm_ptq_kernel(const PtqLaunch launch) {
    // 256 x 256 float tile, 2 x 4 wavefronts of 128 x 64, v_mfma_f32_16x16x32_bf16 (at the card's power
    // limit it sustains about a sixth more than the 32x32x16 form): 8 x 4 accumulator blocks of 16 x 16.
    // NW = 4: 128 x 128, 2 x 2 wavefronts of 64 x 64, several workgroups to a CU (see ptq_form).
    constexpr int BM = NW == 8 ? 256 : 128, BN = BM;
    constexpr int NT = 64 * NW;               // threads
    constexpr int WNC = NW / 2;               // wavefronts along n (two along m)
    constexpr int CW = BN / WNC;              // columns of a wavefront's block
    constexpr int RW = BM / 2;                // rows of a wavefront's block
    constexpr int NA = RW / 16, NB = CW / 16; // 16-wide fragments of P and of Q per wavefront
    static_assert((NW == 8 || NW == 4) && BK == 32 && NB == 4, "one 32-deep slice per stage, NA x 4 blocks per wavefront");
    constexpr int PBYTES = BK * BM * 2;
    constexpr int STAGE = 2 * PBYTES;
    constexpr int PI = BK * BM / 8 / NT;      // loads per wavefront per operand per stage
    constexpr int LPS = 2 * PI;
    using PT = NTile16<BM>;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int total1 = launch.E * launch.first.m_tiles * launch.first.n_tiles;
    const int total = total1 + (BOTH ? launch.E * launch.second.m_tiles * launch.second.n_tiles : 0);
    const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
    const int slot = blockIdx.x / kNumXcd;
    if (slot >= per_xcd) return;
    int lt = (blockIdx.x % kNumXcd) * per_xcd + slot;
    if (lt >= total) return;
    const PtqArgs g = BOTH && lt >= total1 ? launch.second : launch.first;
    if (BOTH && lt >= total1) lt -= total1;
    const int n_layers = launch.n_layers, accumulate = launch.accumulate;
    const void* const zeros = zero_page();
    const int per_e = g.m_tiles * g.n_tiles;
    const int e = lt / per_e;
    // The 32 workgroups of an XCD run 32 consecutive tiles side by side and share their operand blocks
    // through L2: with the shorter tile axis running fastest the 32 tiles form the squarest block
    // (about 6 x 5 instead of 2 x 16), which needs the fewest distinct operand blocks.
    const int idx = lt % per_e;
    const int m0 = (g.m_tiles <= g.n_tiles ? idx % g.m_tiles : idx / g.n_tiles) * BM;
    const int n0 = (g.m_tiles <= g.n_tiles ? idx / g.m_tiles : idx % g.n_tiles) * BN;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WNC, wn = wave % WNC;
#ifdef UNIPOOL_PHASE_TIMES
    const long long pt_begin = wall_clock64();
#endif
    const unsigned lds0 = lds_addr_of(smem);

    // Per-layer row range and operand pointers of expert e, fetched once into LDS: the K loop then
    // advances from layer to layer without global loads of its own (whose wait counts would also
    // wait for the operand loads in flight) and with wave-uniform control flow.
    __shared__ int lds_r0[kMaxPtqLayers], lds_r1[kMaxPtqLayers];
    __shared__ const bf16* lds_p[kMaxPtqLayers];
    __shared__ const bf16* lds_q[kMaxPtqLayers];
    if (BOTH && g.P == nullptr) {
        lds_r0[0] = launch.off1 ? launch.off1[e] : min(g.total_rows, e * g.chunk_rows);
        lds_r1[0] = launch.off1 ? launch.off1[e + 1] : min(g.total_rows, (e + 1) * g.chunk_rows);
        lds_p[0] = reinterpret_cast<const bf16*>(g.P1);
        lds_q[0] = reinterpret_cast<const bf16*>(g.Q1);
    } else {
        for (int l = threadIdx.x; l < n_layers; l += NT) {
            lds_r0[l] = launch.off[l][e];
            lds_r1[l] = launch.off[l][e + 1];
            lds_p[l] = reinterpret_cast<const bf16*>(g.P[l]);
            lds_q[l] = reinterpret_cast<const bf16*>(g.Q[l]);
        }
    }
    __syncthreads();
    // The rows of expert e in all the layers form one reduction, cut into K blocks of BK rows without
    // regard to the layers: a block may end one layer's range and begin the next one's, and only the
    // very last block is filled up with zero rows.
    int k_total = 0;
    for (int l = 0; l < n_layers; l++) k_total += max(0, __builtin_amdgcn_readfirstlane(lds_r1[l] - lds_r0[l]));
    const int nb = (k_total + BK - 1) / BK;
    float* otile = g.out + (long long)e * g.out_stride;
    if (nb == 0) {
        if (!accumulate) {
            for (int i = threadIdx.x; i < BM * BN; i += NT) {
                const int r = m0 + i / BN, c = n0 + i % BN;
                if (r < g.mdim && c < g.ndim) otile[(size_t)r * g.ndim + c] = 0.f;
            }
        }
        return;
    }

    // lane geometry of the direct-to-LDS loads: load i of a wavefront fills LDS slots
    // (i*NW + wave)*64 + lane, i.e. K row 16 i + RPL wave + lane / CPR, chunk position lane % CPR.  The
    // swizzle depends on bits 0, 1 and 3 of the K row, which are the same for all i.
    constexpr int RPL = 64 / PT::CPR;         // K rows of one load
    static_assert(RPL * NW == 16, "the K rows of a lane's loads differ by multiples of 16");
    static_assert(2 * PI == 4, "four loads per K block");
    const int krow0 = RPL * wave + lane / PT::CPR;
    const int cc = (lane % PT::CPR) ^ PT::swz(krow0);
    const int pcol = min(m0 + cc * 8, g.mdim - 8);
    const int qcol = min(n0 + cc * 8, g.ndim - 8);

    // A K block that lies inside one layer's row range is loaded from a wave-uniform row address plus
    // these per-lane byte offsets (no vector arithmetic per load); a block that runs over the end of a
    // range finds, lane by lane, the layer and row of its K index, or the page of zeros past the end.
    const unsigned voff_p = ((unsigned)krow0 * (unsigned)g.mdim + (unsigned)pcol) * 2u;
    const unsigned voff_q = ((unsigned)krow0 * (unsigned)g.ndim + (unsigned)qcol) * 2u;

    // load cursor over the rows of expert e, layer after layer
    int ld_r = 0, ld_end = 0;
    const bf16* ld_p = nullptr;
    const bf16* ld_q = nullptr;
    auto uniform_ptr = [](const bf16* p) {
        const unsigned long long v = (unsigned long long)p;
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
        return reinterpret_cast<const bf16*>(((unsigned long long)hi << 32) | lo);
    };
    // The cursor also holds the next layer in which the expert has rows, fetched from LDS when the
    // cursor moves (once per layer): a block that straddles two layers then needs no LDS access.
    int nx_layer = -1, nx_r = 0, nx_end = 0;
    const bf16* nx_p = nullptr;
    const bf16* nx_q = nullptr;
    auto fetch_next = [&]() {
        nx_r = nx_end = 0;
        while (++nx_layer < n_layers) {
            nx_r = __builtin_amdgcn_readfirstlane(lds_r0[nx_layer]);
            nx_end = __builtin_amdgcn_readfirstlane(lds_r1[nx_layer]);
            if (nx_end > nx_r) {
                nx_p = uniform_ptr(lds_p[nx_layer]);
                nx_q = uniform_ptr(lds_q[nx_layer]);
                return;
            }
        }
        nx_layer = n_layers;
        nx_r = nx_end = 0;
    };
    fetch_next();
    auto next_layer = [&]() {     // the cursor moves to the next layer with rows (wave-uniform); false past the last
        if (nx_layer >= n_layers) return false;
        ld_r = nx_r;
        ld_end = nx_end;
        ld_p = nx_p;
        ld_q = nx_q;
        fetch_next();
        return true;
    };
    // The cursor is always on a row, as long as there is one: it moves to the next layer as soon as one ends.
    auto advance_block = [&]() {  // move the cursor BK rows on, from layer to layer
        ld_r += BK;
        if (__builtin_expect(ld_r < ld_end, 1)) return;
        int over = ld_r - ld_end;
        for (;;) {
            if (!next_layer()) {
                ld_r = ld_end;
                return;
            }
            if (over < ld_end - ld_r) break;
            over -= ld_end - ld_r;
        }
        ld_r += over;
    };
    next_layer();
    // Per-lane source addresses of the LPS loads of the K block at the cursor (P rows for i < PI, Q
    // rows after), worked out in one place per block so that the load slots between the MFMAs hold
    // nothing but the load.
    const void* blk_src[2 * PI];
    auto block_sources = [&]() {
        if (__builtin_expect(ld_r + BK <= ld_end, 1)) {
#pragma unroll
            for (int i = 0; i < 2 * PI; i++) {
                const int rb = ld_r + 16 * (i < PI ? i : i - PI);         // wave-uniform
                blk_src[i] = i < PI ? reinterpret_cast<const char*>(ld_p + (size_t)rb * g.mdim) + voff_p
                                    : reinterpret_cast<const char*>(ld_q + (size_t)rb * g.ndim) + voff_q;
            }
        } else {
            // K index j of this lane inside the block: in the rest of the cursor's layer, in the next
            // layer, or (the next layer being shorter than the block) further on
            const int rem = ld_end - ld_r, nrows = nx_end - nx_r;
#pragma unroll
            for (int i = 0; i < 2 * PI; i++) {
                const int j = 16 * (i < PI ? i : i - PI) + krow0;
                const int dim = i < PI ? g.mdim : g.ndim, col = i < PI ? pcol : qcol;
                const void* src = zeros;
                if (j < rem) src = (i < PI ? ld_p : ld_q) + (size_t)(ld_r + j) * dim + col;
                else if (j - rem < nrows) src = (i < PI ? nx_p : nx_q) + (size_t)(nx_r + j - rem) * dim + col;
                int j0 = rem + nrows;
                for (int lay = nx_layer + 1; j0 < BK && lay < n_layers; lay++) {
                    const int r = __builtin_amdgcn_readfirstlane(lds_r0[lay]);
                    const int n = min(__builtin_amdgcn_readfirstlane(lds_r1[lay]) - r, BK - j0);
                    if (n <= 0) continue;
                    const bf16* base = uniform_ptr(i < PI ? lds_p[lay] : lds_q[lay]);
                    if (j >= j0 && j < j0 + n) src = base + (size_t)(r + j - j0) * dim + col;
                    j0 += n;
                }
                blk_src[i] = src;
            }
        }
    };
    auto issue_one = [&](int stage, int i) {
        const int ii = i < PI ? i : i - PI;
        glds16(blk_src[i], lds0 + stage * STAGE + (i < PI ? 0 : PBYTES) + ((ii * NW + wave) * 64) * 16);
    };

    f32x4 acc[NA][NB];
#pragma unroll
    for (int a = 0; a < NA; a++)
#pragma unroll
        for (int b = 0; b < NB; b++) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Fragments: P block a (rows of the output) and Q block b (columns), one register set each.  A
    // stage is NA * NB MFMA slots, slot HA b + a in each half (a < HA in the first half, the others in the
    // second), so P[0 .. HA) and Q[0..2] become free for the next stage's data during the second half,
    // Q[3] and the other P at its end; the wavefronts meet in the middle, where the next stage's data has
    // landed.
    static_assert(NS >= 2 && (NS - 1) * LPS < 64, "outstanding loads must fit the wait counter");
    bf16x8 pfr[NA], qfr[NB];
    int foff_p[NA], foff_q[NB];
#pragma unroll
    for (int a = 0; a < NA; a++) foff_p[a] = PT::frag_off(wm * RW + a * 16, lane);
#pragma unroll
    for (int b = 0; b < NB; b++) foff_q[b] = PBYTES + PT::frag_off(wn * CW + b * 16, lane);
    constexpr int SECOND = 4 * PT::CPR * 16;          // bytes between the two reads of a fragment
    auto load_p = [&](int stage, int a) {
        const char* b_ = smem + stage * STAGE + foff_p[a];
        pfr[a] = lds_read_tr8(b_, b_ + SECOND);
    };
    auto load_q = [&](int stage, int b) {
        const char* b_ = smem + stage * STAGE + foff_q[b];
        qfr[b] = lds_read_tr8(b_, b_ + SECOND);
    };
    auto mfma_one = [&](int a, int b) {
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfr[a], qfr[b], acc[a][b], 0, 0, 0);
    };
#ifdef UNIPOOL_PHASE_TIMES
    long long pc_wait = 0, pc_bar = 0;
#endif
    // ISSUE: the loads of K block kb-1+NS go out during the first half of this stage, into the buffer
    // that stage kb-1 has released, spaced by three MFMAs (a burst of loads stalls the issuing
    // wavefronts, MFMAs included, until the address unit's queue has drained).
    auto stage_body = [&](auto issue_c, int kb) {
        constexpr bool ISSUE = decltype(issue_c)::value;
        const int stage = kb % NS, nstage = (kb + 1) % NS;
        static_assert(LPS == 4, "load slots below");
        constexpr int HA = NA / 2, HS = HA * NB;          // slots of a half
        constexpr int GAP = HS == 16 ? 3 : 1;
        if constexpr (ISSUE) {
            block_sources();
        }
#pragma unroll
        for (int s = 0; s < HS; s++) {
            mfma_one(s % HA, s / HA);
            if (s == 0) load_q(stage, 3);                       // what the previous stage still held
            if (s >= 1 && s <= HA) load_p(stage, HA - 1 + s);
            if constexpr (ISSUE) {
                constexpr int S0 = HS - 3 * GAP - (HS == 16 ? 2 : 1);
                if (s >= S0 && (s - S0) % GAP == 0 && (s - S0) / GAP < 4) issue_one((kb + NS - 1) % NS, (s - S0) / GAP);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (ISSUE) advance_block();
#ifdef UNIPOOL_PHASE_TIMES
        const long long pw0 = clock64();
#endif
        if (nb - 2 - kb >= NS - 2) wait_vmcnt<(NS - 2) * LPS>();
        else wait_vmcnt<0>();
#ifdef UNIPOOL_PHASE_TIMES
        const long long pw1 = clock64();
#endif
        __syncthreads();
#ifdef UNIPOOL_PHASE_TIMES
        pc_wait += pw1 - pw0;
        pc_bar += clock64() - pw1;
#endif
#pragma unroll
        for (int s = 0; s < HS; s++) {
            mfma_one(HA + s % HA, s / HA);
            if (s < HA) load_p(nstage, s);                      // after the last stage: unused, in bounds
            else if (s % HA == 0) load_q(nstage, s / HA - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int s = 0; s < NS; s++)
        if (s < nb) {
            block_sources();
#pragma unroll
            for (int i = 0; i < LPS; i++) issue_one(s, i);
            advance_block();
        }
    if (nb > NS - 1) wait_vmcnt<(NS - 1) * LPS>();
    else wait_vmcnt<0>();
    __syncthreads();
#ifdef UNIPOOL_PHASE_TIMES
    const long long pt_filled = wall_clock64(), pc_filled = clock64();
#endif
#pragma unroll
    for (int a = 0; a < NA / 2; a++) load_p(0, a);
#pragma unroll
    for (int b = 0; b < 3; b++) load_q(0, b);
    {
        stage_body(std::integral_constant<bool, false>{}, 0);       // nb >= 1 here
        int kb = 1;
        for (; kb - 1 + NS < nb; kb++) stage_body(std::integral_constant<bool, true>{}, kb);
        for (; kb < nb; kb++) stage_body(std::integral_constant<bool, false>{}, kb);
    }
#ifdef UNIPOOL_PHASE_TIMES
    const long long pt_looped = wall_clock64(), pc_looped = clock64();
#endif

    // acc[a][b][r] = out[i = m0 + wm*RW + a*16 + 4*(lane/16) + r][j = n0 + wn*CW + b*16 + lane%16]
    // The block of a wavefront leaves in passes of 32 rows through a wave-private LDS
    // area (rows of CW floats + 4 of padding), so that every lane stores 16 bytes and a wavefront
    // instruction covers whole row segments of 4*CW bytes; when accumulating, the old values are
    // fetched in the same layout.
    __syncthreads();                          // every wavefront is done with the operand stages
    {
        constexpr int SLD = CW + 4;           // staging row stride in floats
        constexpr int LPR = CW / 4;           // lanes per row
        constexpr int RPI = 64 / LPR;         // rows per wavefront instruction
        float* stg = reinterpret_cast<float*>(smem) + wave * (32 * SLD);
        const int jw = n0 + wn * CW;          // first column of the wavefront's block
        const bool vec_ok = (g.ndim & 3) == 0 && (reinterpret_cast<size_t>(g.out) & 15) == 0;
        // Accumulating, the old values are fetched a pass of 32 rows ahead (the fragments' registers are free by
        // now): 8 KiB per wavefront in flight at any time, where fetching four rows, adding and storing them
        // in turn left the reads waiting for each other (one layer's gradients of 90 experts of 832 x 1472, 200 rows
        // each: 945 -> 780 us, streamed 752).  STREAM: the output is larger than the caches, old and new values go past them, and the
        // operands that neighbouring tiles share stay there (the whole backward call of these 90 experts with 256 tokens
        // 852 -> 780 us).  A choice at run time would not do: the compiler merges the two forms of an access into the
        // plain one.
        constexpr int ITS = 32 / RPI;
        const bool add_vec = vec_ok && accumulate;
        const int c4 = (lane % LPR) * 4, j = jw + c4;
        f32x4 old[2][ITS];
        auto fetch_old = [&](int a2) {
#pragma unroll
            for (int it = 0; it < ITS; it++) {
                const int i = m0 + wm * RW + a2 * 32 + it * RPI + lane / LPR;
                if (i < g.mdim && j < g.ndim) {
                    const f32x4* src = reinterpret_cast<const f32x4*>(otile + (size_t)i * g.ndim + j);
                    if constexpr (STREAM) old[a2 & 1][it] = __builtin_nontemporal_load(src);
                    else old[a2 & 1][it] = *src;
                }
            }
        };
        if (add_vec) fetch_old(0);
#pragma unroll
        for (int a2 = 0; a2 < NA / 2; a2++) {
            if (add_vec && a2 + 1 < NA / 2) fetch_old(a2 + 1);
#pragma unroll
            for (int ah = 0; ah < 2; ah++)
#pragma unroll
                for (int b = 0; b < NB; b++)
#pragma unroll
                    for (int r = 0; r < 4; r++)
                        stg[(16 * ah + 4 * (lane >> 4) + r) * SLD + b * 16 + (lane & 15)] = acc[2 * a2 + ah][b][r];
            const int i_blk = m0 + wm * RW + a2 * 32;
#pragma unroll
            for (int it = 0; it < ITS; it++) {
                const int row = it * RPI + lane / LPR;
                const int i = i_blk + row;
                if (i >= g.mdim || j >= g.ndim) continue;
                f32x4 v = *reinterpret_cast<const f32x4*>(stg + row * SLD + c4);
                float* dst = otile + (size_t)i * g.ndim + j;
                if (vec_ok) {                 // then j + 3 < ndim as well
                    if (add_vec) v += old[a2 & 1][it];
                    if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
                    else *reinterpret_cast<f32x4*>(dst) = v;
                } else {
                    const float vv[4] = {v[0], v[1], v[2], v[3]};
                    for (int q = 0; q < 4; q++)
                        if (j + q < g.ndim) dst[q] = (accumulate ? dst[q] : 0.f) + vv[q];
                }
            }
        }
    }
#ifdef UNIPOOL_PHASE_TIMES
    if (threadIdx.x == 0) {
        unsigned long long* pt_ = g_phase_times[512 + (blockIdx.x & 255)];
        atomicAdd(&pt_[0], (unsigned long long)(pt_filled - pt_begin));
        atomicAdd(&pt_[1], (unsigned long long)(pt_looped - pt_filled));
        atomicAdd(&pt_[2], (unsigned long long)(wall_clock64() - pt_looped));
        atomicAdd(&pt_[3], 1ull);
        atomicAdd(&pt_[4], (unsigned long long)pc_wait);
        atomicAdd(&pt_[5], (unsigned long long)pc_bar);
        atomicAdd(&pt_[6], (unsigned long long)(pc_looped - pc_filled));
        atomicAdd(&pt_[7], (unsigned long long)nb);
    }
#endif
}

// out = sum of nparts partial products in index order; the last workgroup adds up the partial sums of d_sigma, which
// saves their launch.  Four values per thread where the addresses allow, and the loads of eight parts are requested
// together: the chain of single loads took 19 us for 64 parts of 96 x 1024, now 8.
template <typename V>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ part, int nparts, size_t stride, size_t n,
                                                              float* __restrict__ out, const float* __restrict__ dsigma_part,
                                                              int n_dsigma, float* __restrict__ d_sigma) {
    if (blockIdx.x == gridDim.x - 1) {
        block_sum_256(dsigma_part, n_dsigma, d_sigma);
        return;
    }
    constexpr size_t W = sizeof(V) / 4;
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * W;
    if (i >= n) return;
    V v = {};
    for (int p = 0; p < nparts; p += 8) {
        V q[8];
#pragma unroll
        for (int u = 0; u < 8; u++) q[u] = *reinterpret_cast<const V*>(part + (size_t)min(p + u, nparts - 1) * stride + i);
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (p + u < nparts) v += q[u];
    }
    *reinterpret_cast<V*>(out + i) = v;
}

// ---------------------------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------------------------
constexpr int kBM = 256, kBN = 256, kBK = 64, kNS = 2;   // gemm_xw: 128-byte row segments per load
constexpr int kPtqBK = 32, kPtqNS = 4;       // gemm_ptq
constexpr int kGemmLds = kNS * kBM * kBK * 2 + (kNS + 1) * kBN * kBK * 2;   // 2 X stages + 3 W stages = 160 KiB
constexpr int kPtqLds = kPtqNS * 2 * kPtqBK * 256 * 2;            // 128 KiB


// Small tiles: 80 KiB of LDS, two workgroups to a CU.  They are no faster with fragments fetched a whole slice ahead (two
// register sets), nor alone on a CU with five stages in flight: a CU keeps about 32 KB of loads in flight, whatever the depth.
constexpr int kSmallBM = 128, kSmallBN = 128;
constexpr int kSmallLds = kNS * kSmallBM * kBK * 2 + (kNS + 1) * kSmallBN * kBK * 2;

enum Tile { TILE_BIG, TILE_SMALL };

template <int TILE, bool WK, int EPI, bool KTAIL = false, bool ADD = false>
hipError_t run_xw(GemmArgs a, hipStream_t st) {
    constexpr bool SMALL = TILE != TILE_BIG;
    constexpr int BM = SMALL ? kSmallBM : kBM, BN = SMALL ? kSmallBN : kBN;
    constexpr int LDS = SMALL ? kSmallLds : kGemmLds;
    auto kern = gemm_xw_kernel<BM, BN, kBK, kNS, WK, EPI, KTAIL, ADD>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    a.group_m = SMALL ? 1 : 2;
    a.n_tiles_n = cdiv(a.N, EPI == EPI_SWIGLU_FWD ? BN / 2 : BN);
    const int grid = max(kNumXcd, num_cus() / kNumXcd * kNumXcd) * (SMALL ? 2 : 1);
    kern<<<grid, 2 * BN, LDS, st>>>(a);
    return hipGetLastError();
}

constexpr int kPtqSmallNS = 3, kPtqSmallLds = kPtqSmallNS * 2 * kPtqBK * 128 * 2;   // 48 KiB

template <int NW, bool STREAM, bool BOTH>
hipError_t run_ptq_form(PtqLaunch a, hipStream_t st) {
    constexpr int BM = NW == 8 ? 256 : 128, NS = NW == 8 ? kPtqNS : kPtqSmallNS, LDS = NW == 8 ? kPtqLds : kPtqSmallLds;
    auto kern = gemm_ptq_kernel<kPtqBK, NS, NW, STREAM, BOTH>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    for (PtqArgs* p : {&a.first, &a.second}) {
        p->m_tiles = cdiv(p->mdim, BM);
        p->n_tiles = cdiv(p->ndim, BM);
    }
    const int total = a.E * (a.first.m_tiles * a.first.n_tiles + a.second.m_tiles * a.second.n_tiles);
    const int grid = cdiv(total, kNumXcd) * kNumXcd;
    kern<<<grid, 64 * NW, LDS, st>>>(a);
    return hipGetLastError();
}

template <int NW, bool BOTH> hipError_t run_ptq_nw(const PtqLaunch& a, bool stream, hipStream_t st) {
    return stream ? run_ptq_form<NW, true, BOTH>(a, st) : run_ptq_form<NW, false, BOTH>(a, st);
}

// Weight gradients of the experts, `rows` rows each in all layers on average.  A 256 x 256 tile takes its CU 0.0235 us per
// row, and then 11 us for its floats, 24 when they are added to old ones; in four 128 x 128 tiles, which read twice as many
// operand bytes but of which a CU runs two at a time, so that one stores while the other multiplies, 0.034 us per row and
// 10.2 or 17.7 us (fitted to 64 experts of 768 x 2048 with 512 and 2048 rows; short of a whole tile the floats count).
// The 18 shapes this was checked on follow it to 10 %, hence the margins (us, big / small tiles, added: 90 experts of
// 832 x 1472 with 200 rows 711 / 522, with 400 825 / 663; 96 of 1024 x 2816 with 682 rows 1974 / 2072; written: 60 of
// 320 x 320 with 400 rows 60 / 42, 90 of 832 x 1472 483 / 513).
// Both gradients go out in one launch, the second's tiles in the wake of the first's (16 of 576 x 320, 1500 rows: two
// launches 93, one 52; 200 of 640 x 1024, 28 rows: 336 / 320), except where each is many rounds of long tiles: then tiles of
// both kinds side by side share less in L2 (written, ms, two / one, rounds of 256 tiles: 96 of 1024 x 2816, 50 rounds, 5460 rows
// 7.88 / 7.96, 8190 rows 11.60 / 11.75; 512 of 1024 x 704, 72 rounds, 4096 rows 8.90 / 8.96; 90 of 832 x 1472, 25 rounds, 4800
// rows 3.52 / 3.57).  With fewer rows or rounds one launch is the shorter or they are alike (96 of 1024 x 2816, 2730 rows
// 4.03 / 4.01, 682 rows 1.45 / 1.43, added 2.02 / 1.97; 64 of 768 x 2048, 18 rounds, 4096 rows 2.26 / 2.22, 1024 rows 0.69 / 0.67,
// added 0.89 / 0.86; 192 of 1536 x 4096, 216 rounds, 2728 rows 18.14 / 18.19).
struct PtqForm {
    bool small, two_launches, stream;
};
PtqForm ptq_form(const PtqLaunch& a, double rows, bool stream) {
    const double cus = num_cus();
    auto tiles = [&](int bm) {
        return (double)a.E * ((double)cdiv(a.first.mdim, bm) * cdiv(a.first.ndim, bm) +
                              (double)cdiv(a.second.mdim, bm) * cdiv(a.second.ndim, bm));
    };
    const double nb = tiles(256), ns = tiles(128);
    const double whole = (double)a.E * ((double)a.first.mdim * a.first.ndim + (double)a.second.mdim * a.second.ndim) / 65536;
    const double big = std::ceil(nb / cus) * (0.0235 * rows + (a.accumulate ? 24.0 : 11.0) * whole / nb);
    const double small = std::ceil(ns / (2 * cus)) * 0.5 * (0.034 * rows + (a.accumulate ? 17.7 : 10.2) * 4 * whole / ns);
    bool take_small = small < (a.accumulate ? 0.98 : 0.9) * big;
#ifdef UNIPOOL_DEBUG_SWITCHES
    if (const char* e = getenv("UNIPOOL_PTQ")) take_small = e[0] == '1';
#endif
    return PtqForm{take_small, !take_small && rows > 4000 && nb > 20 * cus, stream};
}
hipError_t run_ptq(const PtqLaunch& a, const PtqForm& form, hipStream_t st) {
    if (form.small) return run_ptq_nw<4, true>(a, form.stream, st);
    if (form.two_launches && a.off != nullptr) {          // (a single layer's operands only come in one launch)
        PtqLaunch one = a;
        one.second = PtqArgs{};
        hipError_t e = run_ptq_nw<8, false>(one, form.stream, st);
        if (e != hipSuccess) return e;
        one.first = a.second;
        return run_ptq_nw<8, false>(one, form.stream, st);
    }
    return run_ptq_nw<8, true>(a, form.stream, st);
}

// the meeting counters live behind the largest possible tile table (total_rows / 128 + 2 E entries)
int32_t* pair_counters(int32_t* meta, int E, int total_rows) {
    return meta + kTileBase + 4 * ((size_t)total_rows / kSmallBM + 2 * E);
}

// Timing aid of debugging builds: UNIPOOL_W0=1 makes every expert read the weights of expert 0, so that the
// weight stream comes from the caches instead of HBM (same instructions, results meaningless).
long long debug_w_stride(long long w_stride) {
#ifdef UNIPOOL_DEBUG_SWITCHES
    static int v = -1;
    if (v < 0) {
        const char* e = getenv("UNIPOOL_W0");
        v = (e && e[0] == '1') ? 1 : 0;
    }
    return v == 1 ? 0 : w_stride;
#else
    return w_stride;
#endif
}

constexpr int tile_rows(int tile) { return tile == TILE_SMALL ? kSmallBM : kBM; }

// Tables of one entry point's products: the first product's tile size in `main`, the second's, where it is another, in `extra`.
hipError_t build_tiles(const unipool_shape& s, const int32_t* offsets, int tile0, int tile1, int32_t* main, int32_t* extra,
                       hipStream_t st) {
    TileTables t = {};
    t.meta[0] = main; t.bm[0] = tile_rows(tile0);
    t.meta[1] = extra; t.bm[1] = tile_rows(tile1);
    t.pair_cnt = pair_counters(main, s.E, s.T * s.k);
    build_tiles_kernel<<<tile0 == tile1 ? 1 : 2, 512, 0, st>>>(offsets, s.E, t);
    return hipGetLastError();
}

// one row-grouped product of the FFN with tiles of the given size
template <bool WK, int EPI>
hipError_t run_grouped(const GemmArgs& a, int tile, hipStream_t st) {
    return tile == TILE_SMALL ? run_xw<TILE_SMALL, WK, EPI>(a, st) : run_xw<TILE_BIG, WK, EPI>(a, st);
}

// Row tiles that an expert with r rows on average takes: the sizes of one layer spread by about sqrt(r), so a mean just
// below a multiple of the tile already gives part of the experts one tile more.
double row_tiles(double r, int bm) {
    const double s = 0.5 * sqrt(r);
    double m = std::max(1.0, std::floor((r - s) / bm) + 1.0);          // tiles that every expert takes
    for (double j = m; bm * j < r + s; j++) m += std::min(1.0, (r + s - bm * j) / (2.0 * s));
    return m;
}

// Tile size of the FFN's product `which` (gate and up, down, dH, dX) with N output columns (2 d_ff for gate and up).  A tile's time goes
// with the columns of W it brings in and, at 0.4 of their weight, with its rows, which mostly come from L2 (the reduction
// length scales both forms alike), and the launch ends when the CU with the most tiles does:
//   big:   ceil(tiles / 256) rounds of 256 + 0.4 rows;
//   small: ceil(tiles / 512) rounds, two tiles to a CU, of 2 (128 + 0.4 rows), times 0.9 (gate and up 0.95, whose rows of 64
//          + 64 columns are stored in shorter pieces) since one workgroup's epilogue runs beside the other's loop; up to 256
//          tiles every workgroup has a CU to itself, which takes 0.6 of that.
// So small tiles are taken where big ones leave CUs without work or columns without use.  Where big tiles all run at once and
// small ones two to a CU, the longest CU gets 256 columns either way, and with few rows there is little epilogue to overlap: big
// ones then (dX of 31 experts, 1280 columns, 6 rows each, share of both backward products: 5.7 to 7.9 % longer in small
// tiles; 29 of 1600, 44 rows 3 to 4 %; 33 of 1088, 53 rows 3.6 %; 97 of 320, 56 rows 2 %; but 30 of 1152, 61 rows 4 to 5 %
// shorter, 23 of 1856, 64 rows 1 %).  Experts without rows have no tiles: with fewer picks than experts they are left out of the
// count (both backward products of 96 experts of 1024 x 2816, 64 picks 158 us as if all had rows, now 145; 64 of 768 x 2048, 60
// picks 89 and 78).  Over 218 shapes (4 to 512 experts, d_model 64 to 1664, d_ff 64 to 4096, 1 to 37000
// rows per expert, even and skewed routing) both FFN entry points together are 11 % shorter than with big tiles alone, the
// worst shape 2 % longer and the best 46 % shorter; the worst single entry point is 4 % longer.  One layer, us, big / small: down projection of 16 experts of 768 x 2048, 188 rows each (48 tiles / 192) 41 / 27,
// dX of these 67 / 39, dH 34 / 27; but gate and up of 192 experts of 1536 x 4096, 341 rows each 1880 / 2700.
int tile_form(const unipool_shape& s, int N, int which, bool extra) {
    if (!extra) return TILE_BIG;                       // there is no room for a second table
#ifdef UNIPOOL_DEBUG_SWITCHES
    if (const char* e = getenv("UNIPOOL_TILES")) return (atoi(e) >> (4 * which)) & 15;    // a digit per product
#endif
    const double S = (double)s.T * s.k;
    const double used = s.E * -std::expm1(-S / s.E), r = S / used;         // experts with rows, as if the picks were independent
    const double mb = row_tiles(r, kBM), ms = row_tiles(r, kSmallBM);
    const double nb = used * mb * cdiv(N, kBN), ns = used * ms * cdiv(N, kSmallBN);
    const int cus = num_cus();
    const double big = std::ceil(nb / cus) * (kBN + 0.4 * r / mb);
    if (nb <= cus && ns > cus && r < 60) return TILE_BIG;
    const double small = (ns <= cus ? 0.6 : std::ceil(ns / (2 * cus))) * (which == 0 ? 0.95 : 0.9) * 2 * (kSmallBN + 0.4 * r / ms);
    return small < big ? TILE_SMALL : TILE_BIG;
}

}  // namespace

int num_cus() {
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t p;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess)
            n = p.multiProcessorCount;
        if (n <= 0) n = 256;
    }
    return n;
}

bool mfma_ffn_supported(const unipool_shape& s) {
    // the tile table is built by one workgroup with a thread per expert; the weight-gradient kernel
    // keeps the per-layer row ranges of an expert in LDS
    return s.dtype == UNIPOOL_BF16 && s.d_model % 64 == 0 && s.d_ff % 64 == 0 && s.E <= kMaxTableExperts;
}

bool mfma_router_supported(const unipool_shape& s) {
    // the logits of other pools take the float kernel, which keeps the index-order sums they always had
    return s.dtype == UNIPOOL_BF16 && s.d_model % 64 == 0 && s.E % 8 == 0;
}

hipError_t mfma_logits(const unipool_shape& s, const void* x, const void* w, float* z, hipStream_t st) {
    GemmArgs a = {};
    a.X = (const bf16*)x; a.ldx = s.d_model;
    a.W = (const bf16*)w; a.w_stride = 0; a.ldw = s.d_model;
    a.K = s.d_model; a.N = s.E;
    a.out0 = z; a.ldo = s.E;
    a.flat_rows = s.T; a.flat_bm = kSmallBM;
    // 128 columns where they hold the pool or where all tiles run at once, 256 otherwise, which read x half as often (all of
    // the entry point, us, 256 / 128: 64 experts, 8192 tokens, d 832 26 / 23; 512, 1000, 320 43 / 34; 200, 20000, 832 42 / 45)
    return s.E <= kSmallBN || cdiv(s.T, kSmallBM) * cdiv(s.E, kSmallBN) <= num_cus()
               ? run_xw<TILE_SMALL, true, EPI_F32>(a, st) : run_xw<TILE_BIG, true, EPI_F32>(a, st);
}

// Gate and up projections in tiles of form `tile`; the table of `down` is built along with theirs.
static hipError_t ffn_gate_up(const unipool_shape& s, const void* x_perm, const int32_t* offsets, const void* wgu, void* a_out,
                              void* b_out, void* h_out, int32_t* tile_meta, int32_t* extra, int tile, int down, hipStream_t st,
                              const int32_t* slot_of_row) {
    const int d = s.d_model, f = s.d_ff;
    hipError_t e = build_tiles(s, offsets, tile, down, tile_meta, extra, st);
    if (e != hipSuccess) return e;
    GemmArgs a = {};
    a.X = (const bf16*)x_perm; a.ldx = d;
    a.W = (const bf16*)wgu; a.w_stride = debug_w_stride(2LL * f * d); a.ldw = d;
    a.K = d; a.N = f;
    a.tile_meta = tile_meta; a.out0 = a_out; a.out1 = b_out; a.out2 = h_out; a.ldo = f;
    a.up_rows = f;
    a.gather = slot_of_row; a.gather_div = s.k;
    return run_grouped<true, EPI_SWIGLU_FWD>(a, tile, st);
}

hipError_t mfma_ffn_gate_up(const unipool_shape& s, const void* x_perm, const int32_t* offsets,
                            const void* wgu, void* a_out, void* b_out, void* h_out, int32_t* tile_meta,
                            int32_t* extra, hipStream_t st) {
    const int tile = tile_form(s, 2 * s.d_ff, 0, extra != nullptr);
    return ffn_gate_up(s, x_perm, offsets, wgu, a_out, b_out, h_out, tile_meta, extra, tile, tile, st, nullptr);
}

hipError_t mfma_ffn_fwd(const unipool_shape& s, const void* x_perm, const int32_t* offsets,
                        const void* wgu, const void* wd, void* a_out, void* b_out, void* h_out,
                        void* y, int32_t* tile_meta, int32_t* extra, hipStream_t st, const int32_t* slot_of_row) {
    const int S = s.T * s.k, d = s.d_model, f = s.d_ff;
    const int tile0 = tile_form(s, 2 * f, 0, extra != nullptr), tile1 = tile_form(s, d, 1, extra != nullptr);
    hipError_t e = ffn_gate_up(s, x_perm, offsets, wgu, a_out, b_out, h_out, tile_meta, extra, tile0, tile1, st, slot_of_row);
    if (e != hipSuccess) return e;
    GemmArgs b = {};
    b.X = (const bf16*)h_out; b.ldx = f;
    b.W = (const bf16*)wd; b.w_stride = debug_w_stride((long long)d * f); b.ldw = f;
    b.K = f; b.N = d;
    b.tile_meta = tile0 == tile1 ? tile_meta : extra; b.launch_slot = 1; b.out0 = y; b.ldo = d;
    if (b.K >= kPairMinK) { b.pair_cnt = pair_counters(tile_meta, s.E, S); b.pair_cap = kPairCap; }
    return run_grouped<true, EPI_STORE>(b, tile1, st);
}

hipError_t mfma_ffn_dgrad(const unipool_shape& s, const void* dy, const void* a_in, const void* b_in,
                          const int32_t* offsets, const void* wgu, const void* wd, void* dx,
                          void* d_act, int32_t* tile_meta, int32_t* extra, hipStream_t st) {
    const int S = s.T * s.k, d = s.d_model, f = s.d_ff;
    const int tile0 = tile_form(s, f, 2, extra != nullptr), tile1 = tile_form(s, d, 3, extra != nullptr);
    hipError_t e = build_tiles(s, offsets, tile0, tile1, tile_meta, extra, st);
    if (e != hipSuccess) return e;
    GemmArgs a = {};   // dH = dY W_down (W_down[e] is [d][f]: reduction index strided), then SwiGLU backward
    a.X = (const bf16*)dy; a.ldx = d;
    a.W = (const bf16*)wd; a.w_stride = debug_w_stride((long long)d * f); a.ldw = f;
    a.K = d; a.N = f;
    a.tile_meta = tile_meta; a.out0 = d_act; a.ldo = 2 * f;
    a.aux_a = (const bf16*)a_in; a.aux_b = (const bf16*)b_in;
    e = run_grouped<false, EPI_SWIGLU_BWD>(a, tile0, st);
    if (e != hipSuccess) return e;
    GemmArgs b = {};   // dX = [dA|dB] W_gate_up (W_gate_up[e] is [2f][d])
    b.X = (const bf16*)d_act; b.ldx = 2 * f;
    b.W = (const bf16*)wgu; b.w_stride = debug_w_stride(2LL * f * d); b.ldw = d;
    b.K = 2 * f; b.N = d;
    b.tile_meta = tile0 == tile1 ? tile_meta : extra; b.launch_slot = 1; b.out0 = dx; b.ldo = d;
    if (b.K >= kPairMinK) { b.pair_cnt = pair_counters(tile_meta, s.E, S); b.pair_cap = kPairCap; }
    return run_grouped<false, EPI_STORE>(b, tile1, st);
}

// Sizes of both gradients of a.n_layers layers, and the form of their launch.
static PtqForm set_wgrad_sizes(const unipool_shape& s, PtqLaunch& a) {
    const int d = s.d_model, f = s.d_ff;
    a.E = s.E;
    a.first.mdim = 2 * f; a.first.ndim = d;            // d_w_gate_up[e][n][c] = sum d_act[row][n] * x_perm[row][c]
    a.first.out_stride = 2LL * f * d;
    a.second.mdim = d; a.second.ndim = f;              // d_w_down[e][c][n] = sum dy[row][c] * h[row][n]
    a.second.out_stride = (long long)d * f;
    // Smaller gradients are still in the last-level cache (256 MB) when the next layer adds to them.  One layer's whole
    // backward call, k = 2, plain / streamed, us: 16 experts of 768 x 1024 (151 MB), 256 tokens 106 / 124, 4096 tokens
    // 214 / 207; 14 experts of 1024 x 1024 (176 MB) 147 / 138 and 224 / 208; 64 experts of 768 x 2048 (1.2 GB) 669 / 608
    // and 770 / 712.
    const bool stream = 12ll * s.E * d * f > (160ll << 20);
    return ptq_form(a, (double)a.n_layers * s.T * s.k / s.E, stream);
}

static hipError_t ffn_wgrad(const unipool_shape& s, PtqLaunch a, float* dwgu, float* dwd, hipStream_t st) {
    const PtqForm form = set_wgrad_sizes(s, a);
    a.first.out = dwgu;
    a.second.out = dwd;
    return run_ptq(a, form, st);
}

int mfma_tile_forms(const unipool_shape& s, bool extra, int n_layers, int accumulate) {
    const int N[4] = {2 * s.d_ff, s.d_model, s.d_ff, s.d_model};
    int forms = 0;
    for (int which = 0; which < 4; which++)
        if (tile_form(s, N[which], which, extra) == TILE_SMALL) forms |= UNIPOOL_SMALL_GATE_UP << which;
    PtqLaunch a = {};
    a.n_layers = n_layers; a.accumulate = accumulate;
    const PtqForm form = set_wgrad_sizes(s, a);
    return forms | (form.small ? UNIPOOL_SMALL_WGRAD : 0) | (form.two_launches ? UNIPOOL_WGRAD_TWO_LAUNCHES : 0) |
           (form.stream ? UNIPOOL_WGRAD_STREAMED : 0);
}

hipError_t mfma_ffn_wgrad(const unipool_shape& s, int n_layers, const void* const* x_perm_l,
                          const void* const* d_act_l, const void* const* h_l,
                          const void* const* dy_l, const int32_t* const* offsets_l,
                          float* dwgu, float* dwd, int accumulate, hipStream_t st) {
    PtqLaunch a = {};
    a.off = offsets_l; a.n_layers = n_layers; a.accumulate = accumulate;
    a.first.P = d_act_l; a.first.Q = x_perm_l;
    a.second.P = dy_l; a.second.Q = h_l;
    return ffn_wgrad(s, a, dwgu, dwd, st);
}

hipError_t mfma_ffn_wgrad_layer(const unipool_shape& s, const void* x_perm, const void* d_act, const void* h, const void* dy,
                                const int32_t* offsets, float* dwgu, float* dwd, hipStream_t st) {
    PtqLaunch a = {};
    a.off1 = offsets; a.n_layers = 1; a.accumulate = 1;
    a.first.P1 = d_act; a.first.Q1 = x_perm;
    a.second.P1 = dy; a.second.Q1 = h;
    return ffn_wgrad(s, a, dwgu, dwd, st);
}

bool mfma_route_bwd_supported(const unipool_shape& s, const void* x, const void* w, const void* dx) {
    // Pools that are a multiple of 8 have their operands aligned to 16 bytes.  Others may come at any address: the float
    // kernel reads those value by value; it also takes up to 256 tokens, where its launches are the shorter ones (all of
    // the entry point, us, this path / the float one: 3 experts, d 256, 16 tokens 16.5 / 13.1; 90 experts, d 832, 256 tokens
    // 19.2 / 14.5, 512 tokens 19.3 / 16.4, 1024 tokens 19.7 / 22.5; 500 experts, d 1536, 256 tokens 25.7 / 26.9, 512 tokens
    // 27.2 / 38.1).
    if (s.dtype != UNIPOOL_BF16) return false;
    if (s.E % 8 == 0) return true;
    return s.T > 256 && (((uintptr_t)x | (uintptr_t)w | (uintptr_t)dx) & 15) == 0;
}

hipError_t mfma_route_bwd_mm(const unipool_shape& s, const void* x, const void* w, const void* dz,
                             float* dw, void* dx, int dx_accumulate, const float* dsigma_part, float* d_sigma,
                             float* wpart, hipStream_t st) {
    const int d = s.d_model, E = s.E, T = s.T, ez = dz_stride(s);
    // d_w_router = dz^T x: the token axis is cut into chunks whose partial products are summed in a fixed order;
    // as many chunks as give every CU one output tile in a single round, of 256 tokens at least, or 128 where the partial
    // products are small (all of the entry point, us, 256 / 128: 16 experts, d 768, 3001 tokens 24 / 22; 64 experts, d 768,
    // 8192 tokens 32 / 34)
    const int chunk_min = ez <= 32 ? 128 : 256;
    const int tiles_per_chunk = cdiv(ez, 256) * cdiv(d, 256);
    const int nchunks = max(1, min(min(kRouteBwdSplit, cdiv(T, chunk_min)), num_cus() / tiles_per_chunk));
    PtqLaunch a = {};
    a.n_layers = 1;
    PtqArgs& p = a.first;
    p.P1 = dz; p.Q1 = x;
    p.chunk_rows = cdiv(cdiv(T, nchunks), 32) * 32;
    p.total_rows = T;
    const int used = cdiv(T, p.chunk_rows);
    a.E = used;
    p.mdim = ez; p.ndim = d;
    p.out = wpart; p.out_stride = (long long)ez * d;
    // 128 x 128 tiles for pools that they do not cut and for short calls (all of the entry point, us, 256 / 128: 64 experts,
    // d 768, 8192 tokens 32 / 28; 512, 320, 1000 32 / 25; 192, 1536, 32768 115 / 122)
    hipError_t e = ez <= 128 || T <= 4096 ? run_ptq_form<4, false, true>(a, st) : run_ptq_form<8, false, true>(a, st);
    if (e != hipSuccess) return e;
    const size_t n = (size_t)E * d;                 // a multiple of 64, as d is
    const int n_dsigma = cdiv(T, dz_tokens_per_block(s));
    if (((uintptr_t)dw & 15) == 0)
        reduce_partials_kernel<f32x4><<<(unsigned)((n / 4 + 255) / 256) + 1, 256, 0, st>>>(
            wpart, used, (size_t)ez * d, n, dw, dsigma_part, n_dsigma, d_sigma);
    else
        reduce_partials_kernel<float><<<(unsigned)((n + 255) / 256) + 1, 256, 0, st>>>(
            wpart, used, (size_t)ez * d, n, dw, dsigma_part, n_dsigma, d_sigma);
    // dx (+)= dz W   (W is [E][d]: reduction index strided)
    GemmArgs b = {};
    b.flat_rows = T;
    b.X = (const bf16*)dz; b.ldx = ez;                 // (values between E and ez are zeros)
    b.W = (const bf16*)w; b.w_stride = 0; b.ldw = d;
    b.K = E; b.N = d;
    b.out0 = dx; b.ldo = d;
    // Small tiles: the reduction (E indices) is so short that a tile is mostly its start and its end, which two workgroups
    // to a CU overlap (all of the entry point, us, 256 x 256 / 128 x 128 tiles: 32768 tokens, 192 experts, d 1536 117 / 110;
    // 65536, 192, 1536 223 / 211; 32768, 512, 1024 135 / 131; 131072, 384, 576 320 / 303; 4096, 512, 1024 46 / 38).  Many rounds
    // of wide rows of a large pool are bound by reading dz once per column tile, half as often in large ones: 131072 tokens, 512
    // experts, d 1024 444 / 458; 262144 844 / 870; 131072, 512, 1536 590 / 607; 65536, 448, 2048 368 / 375; but 131072, 256, 1024
    // 312 / 305, 65536, 512, 1024 (4 rounds) 237 / 235, 524288, 512, 256 888 / 873.
    const bool big = E >= 448 && E % kBK == 0 && d >= 1024 && (long long)cdiv(T, kBM) * cdiv(d, kBN) >= 8ll * num_cus();
    if (big) {
        b.flat_bm = kBM;
        return dx_accumulate ? run_xw<TILE_BIG, false, EPI_STORE, false, true>(b, st) : run_xw<TILE_BIG, false, EPI_STORE>(b, st);
    }
    b.flat_bm = kSmallBM;
    if (dx_accumulate)
        return E % kBK != 0 ? run_xw<TILE_SMALL, false, EPI_STORE, true, true>(b, st)
                            : run_xw<TILE_SMALL, false, EPI_STORE, false, true>(b, st);
    return E % kBK != 0 ? run_xw<TILE_SMALL, false, EPI_STORE, true>(b, st) : run_xw<TILE_SMALL, false, EPI_STORE>(b, st);
}

}  // namespace unipool

#ifdef UNIPOOL_PHASE_TIMES
// Copies the phase sums to the host ([1024][8] values) and clears them.
extern "C" int unipool_debug_phase_times(unsigned long long* out) {
    hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(unipool::g_phase_times), sizeof(unsigned long long) * 8192);
    if (e != hipSuccess) return (int)e;
    static unsigned long long zeros[8192];
    return (int)hipMemcpyToSymbol(HIP_SYMBOL(unipool::g_phase_times), zeros, sizeof(zeros));
}
#endif
