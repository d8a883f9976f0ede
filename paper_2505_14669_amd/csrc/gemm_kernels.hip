// MXFP4 x MXFP4 -> fp32 GEMM on the gfx950 block-scaled matrix cores (Section 4.4, "Stage 2":
// D = (A x SFA)(B x SFB)^T with one E8M0 scale per 32 elements along K).
//
// v_mfma_scale_f32_16x16x128_f8f6f4 operand layout (FP4, cbsz = blgp = 4), measured on gfx950:
//   A: lane l holds row l%16, K-elements 32*(l/16) .. +31 as 128 bits, element j in bits [4j,4j+4)
//      -- exactly the packed row-major code bytes, so a fragment is one 16-byte LDS read;
//   B: the same with the output column in place of the row;
//   scale: one byte per lane (selected by op_sel from a 32-bit register) = the E8M0 scale of that
//      lane's 32 K-elements, i.e. one MX group per lane per instruction;
//   D: lane l, register r -> row 4*(l/16) + r, column l%16.
// The 256 x 256 kernel uses it, the smaller tiles v_mfma_scale_f32_32x32x64_f8f6f4 (lane l: row or column l%32, K-elements 32*(l/32) ..
// +31; D: row 8*(r/4) + 4*(l/32) + r%4, column l%32).  Why 16 x 16 x 128 on the large tiles (same rate, same operand bytes per wave
// tile): there the chip is power-limited, and the deeper instruction reads and writes each fp32 accumulator once per 128 K-elements instead of once per 64.
// Registers only, quantized normal data, 128 x 128 wave tiles: 7.09 PFLOP/s at 1.79 GHz against 6.38 at 1.59 GHz; both give the same bits (compared over 25 binades of scales).
// The tiled scale layout (see scale_tile_offset) stores, for each block of 32 rows and 256
// K-elements, dword 32 h + row with the scales of groups h, 2 + h, 4 + h, 6 + h.  16 x 16 x 128: lane l reads the dword of its row and h =
// (l/16) % 2 once per K-quad (128 contiguous bytes twice per wave), and its group of the quad's first and second K-step is byte
// l/32 and byte 2 + l/32.  32 x 32 x 64: lane l reads dword l of the tile, byte s for K-step s.  The paper's separate scale-rearrangement step does not exist here.
//
// Kernels: gemm_mxfp4_stream_kernel (256 x 256 tiles) and gemm_mxfp4_stream_tile_kernel (128 x 256 and 128 x 128 tiles
// for small problems): one block per compute unit streams its tiles through a ring of K-quads (256 elements) in LDS, of 128 x 128 tiles
// also two (gemm_mxfp4_twin_kernel).  The wide kernels are for Hadamard blocks of 256, the past kernels for bf16 results of 256 MB and more.  All work through a batch of one or two products per launch (GemmBatch).
// What bounds them besides power is the way of the operands into the LDS: a cache line is 128 bytes, so a ring of 128-element
// stages (64 bytes of codes per row) fetched every line twice.  K-quads, whole lines, one barrier per quad and reads and loads spread
// evenly over the matrix-core instructions, 16 x 16 x 128 on the large tiles and 32 x 32 x 64 on the small ones, took against that design
// (layer steps, us): 16384 x 4096 x 11008 1434 -> 1378, 16384 x 4096 x 4096 620 -> 601, 2336 x 1376 x 3168 78.7 -> 71.5, 4096 x 2048 x 2048
// 91.2 -> 85.1, forward 1003 x 2048 x 5632 25.6 -> 23.9.  (16 x 16 x 128 on the old stages: 0-4 % slower.)
#include "gemm_common.h"
#include "launchers.h"
#include "pair_level.h"

namespace quartet {

// Test / tuning override of the kernel choice (quartet_debug_set_gemm_plan): -1 / 0 = the size heuristics below.
static int g_forced_variant = -1;
static int g_forced_band = 0;

// quartet_profile_clock: device counters the streaming kernel adds each block's run time to (null: off)
static uint64_t* g_clock_counters = nullptr;

void set_clock_counters(uint64_t* device_counters) { g_clock_counters = device_counters; }

constexpr int kTwoPerCu = 3;          // variant: 128 x 128 tiles, two blocks per compute unit
constexpr int kTwoPerCuCode = 22;     // its number outside

void set_gemm_plan(int variant, int band_height) {
    g_forced_variant = variant == kTwoPerCuCode ? kTwoPerCu : variant;
    g_forced_band = band_height;
}

// One product of a launch of the streaming kernels, and the one or two products a launch works through: a
// block walks tiles of the first product, then of the second (TileWalk; Algorithm 1 Backward: the two gradient
// products do not depend on each other; in one launch the second starts where the first leaves compute units idle and
// there is one ramp-up and one drain instead of two).
struct GemmProblem {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* b_codes;
    const uint8_t* b_scales;
    void* d;
    const uint32_t* mask;
    uint32_t m, n, k, ldd;
    float alpha;
    uint32_t tiles_m, tiles_n, band_height, total_tiles;
};
struct GemmBatch {
    GemmProblem p[2];
    uint32_t extra_tiles, late;     // the second product's tiles that the last `late` blocks take in rounds of their own, see TileWalk
    uint32_t past;                  // fp32 results are stored past the memory-side cache (store_tile_rows8); of bf16 ones by kernels of their own
};

// The tiles of block b of G: b, b + G, ... of the first product, then, with the blocks counted from r = its tiles % G on, tiles of the
// second.  The G - r = late blocks from r on have one tile of the first product fewer than the others, and its tiles may take several
// times as long as the second's: the first extra_tiles of those go to the late blocks alone, `late` a round, the others to all
// blocks, G a round.  The launcher picks extra_tiles (pair_level).  sel: product, tile: number in it; past the end in the second product.
struct TileWalk {
    uint32_t sel, tile;
};
#define WALK_START(W)                                                                                   \
    {                                                                                                   \
        W.sel = blockIdx.x >= first_tiles ? 1u : 0u;                                                    \
        W.tile = W.sel ? second_start : blockIdx.x;                                                     \
    }
#define WALK_NEXT(W)                                                                                    \
    {                                                                                                   \
        if (W.sel) {                                                                                    \
            W.tile += W.tile < extra_tiles ? late : G;                                                  \
        } else {                                                                                        \
            W.tile += G;                                                                                \
            if (W.tile >= first_tiles) { W.sel = 1u; W.tile = second_start; }                           \
        }                                                                                               \
    }

// Byte selector that turns a lane's raw scale dword of a K-quad (with 0x7F7F7F7F as the other source of v_perm_b32) into its scale
// operand: byte 0 for the quad's first K-step, byte 2 for its second.  group0: the quad's first group; groups from gk on do not
// exist, their codes are zero and their scale is 2^0.
__device__ __forceinline__ uint32_t scale_selector(uint32_t lane, uint32_t group0, uint32_t gk) {
    const uint32_t hi = lane >> 5, g = group0 + (lane >> 4);
    return (g < gk ? hi : 4u) | ((g + 4u < gk ? 2u + hi : 4u) << 16);
}

// ---------------------------------------------------------------------------------------------
// Streaming variant: one block per compute unit walks its tiles (TileWalk), and the ring of LDS
// stages never drains between them: the loads of the next tile's first stages are issued during the last stages
// of the current one, so a tile's first matrix-core instruction follows the previous tile's result stores directly.
// The epilogue uses a scratch of its own (16 KB beside the 136 KB ring).
// WIDE: Hadamard blocks of 256 columns (store_tile_rows8): sizes are multiples of the tile.  PAST16: bf16 results past the memory-side cache: a
// branch per pass, as fp32 results have it, costs bf16 launches 0.5-1.6 % (layer step 2336 x 1376 x 3168 58.3 -> 59.2 us).
template <bool OUT_BF16, bool FUSED, bool WIDE, bool PAST16 = false>
__device__ __forceinline__ void stream_large_tiles(const GemmBatch& batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    constexpr uint32_t TM = 4, TN = 4, BM = 256, BN = 256;
    constexpr uint32_t CODES = (BM + BN) * 8;            // 16-byte chunks of codes per K-quad
    constexpr uint32_t QUAD = CODES + 256;               // + 16 scale tiles of 256 B
    constexpr uint32_t EPI = 4u * 256u;                  // 16-byte chunks of epilogue scratch (4 KB per wave)
    __shared__ v4i_t lds[2u * QUAD + EPI];

    // measurement support: shader-clock and constant-clock ticks of this block's run (wave-uniform branch)
    uint64_t clk_t0 = 0, clk_w0 = 0;
    if (clock_counters) {
        clk_t0 = __builtin_readcyclecounter();
        clk_w0 = __builtin_amdgcn_s_memrealtime();
    }

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t l16 = lane & 15u, quarter = lane >> 4;
    const uint32_t G = gridDim.x, first_tiles = batch.p[0].total_tiles, second_tiles = batch.p[1].total_tiles;
    const uint32_t extra_tiles = batch.extra_tiles, late = batch.late;
    const uint32_t second_start = blockIdx.x + late >= G ? blockIdx.x + late - G : extra_tiles + late + blockIdx.x;
    const uint32_t wm0 = (wave >> 1) * 128u, wn0 = (wave & 1u) * 128u;
    const bool scales_of_a = wave < 2u;
    const uint32_t past = OUT_BF16 ? (uint32_t)PAST16 : batch.past;

// tile origin of tile number V of product Q (XCD-aware order, bands of band_height tile rows); V >= its tiles: M0 = m (no rows)
#define STREAM_TILE(Q, V, M0, N0)                                                                       \
    {                                                                                                   \
        const uint32_t v_ = (V), tt_ = (Q).total_tiles;                                                 \
        if (v_ < tt_) {                                                                                 \
            const uint32_t per_ = tt_ >> 3, rem_ = tt_ & 7u, GM_ = (Q).band_height;                     \
            const uint32_t tiles_m_ = (Q).tiles_m, tiles_n_ = (Q).tiles_n;                              \
            const uint32_t xcd_ = v_ & 7u;                                                              \
            const uint32_t tile_ = xcd_ * per_ + (xcd_ < rem_ ? xcd_ : rem_) + (v_ >> 3);               \
            const uint32_t band_ = tile_ / (GM_ * tiles_n_);                                            \
            const uint32_t band_rows_ = (tiles_m_ - band_ * GM_) < GM_ ? (tiles_m_ - band_ * GM_) : GM_; \
            const uint32_t in_band_ = tile_ - band_ * GM_ * tiles_n_;                                   \
            M0 = (band_ * GM_ + in_band_ % band_rows_) * BM;                                            \
            N0 = (in_band_ / band_rows_) * BN;                                                          \
        } else {                                                                                        \
            M0 = (Q).m; N0 = (Q).n;                                                                     \
        }                                                                                               \
    }
    // issue cursor: the tile and K-quad the next LDS-direct loads belong to
    // (its product's inner dimension decides the offsets: kb = bytes per code row, kq = K-quads per tile)
    // A tile does not start at K = 0: the tiles of XCD class c (tile number mod 8; an XCD's compute units hold tiles of
    // one class at a time and must stay in step to share panels in their L2) start c/8 of the way along K, in whole K-quads,
    // and wrap around: ikq is the K-quad the cursor's local quad iq stands for.  Otherwise every compute unit of the
    // chip asks for the same few hundred bytes of its operand rows at the same time, and with a row pitch of a few KB the
    // memory channels behind the L2s serve that unevenly (measured: 1-2 % of the K = 4096 products' time).  fp32 sums are
    // formed in a rotated order then, the same for a tile wherever it runs.  Only for K a multiple of 256: a ragged last
    // K-quad keeps its place at the end.
    // A load instruction brings 8 rows x 128 bytes (whole cache lines: with 16 rows x 64 bytes every line crosses from the L2 twice).
    TileWalk iw;
    uint32_t iq = 0u;
    WALK_START(iw)
    v4i_t res_a, res_b, res_s;
    uint32_t kb, kq, goff, gstep, soff, ikq;
    const uint32_t drow = wave * 8u + (lane >> 3);
    const uint32_t dcol = (lane & 7u) ^ ((drow >> 1) & 7u);
#define STREAM_ISSUE_SETUP()                                                                            \
    {                                                                                                   \
        uint32_t m0_, n0_;                                                                              \
        const GemmProblem& q_ = batch.p[iw.sel];                                                        \
        const uint32_t lv_ = iw.tile;                                                                   \
        STREAM_TILE(q_, lv_, m0_, n0_)                                                                  \
        const uint32_t k_ = q_.k;                                                                       \
        const uint32_t kq_ = (k_ + 255u) >> 8;  /* scale tiles per 32 rows */                           \
        kq = kq_ ? kq_ : 1u;                                                                            \
        kb = k_ >> 1;                                                                                   \
        ikq = ((k_ & 255u) == 0u) ? ((lv_ & 7u) * kq) >> 3 : 0u;                                        \
        goff = drow * kb + dcol * 16u;          /* + j*32*kb, + quad*128 */                             \
        gstep = 32u * kb;                                                                               \
        soff = (((wave & 1u) * 4u + (lane >> 4)) * kq_) * 256u + (lane & 15u) * 16u;    /* + quad*256 */ \
        const uint32_t rows_a_ = (q_.m - m0_) < BM ? (q_.m - m0_) : BM, rows_b_ = (q_.n - n0_) < BN ? (q_.n - n0_) : BN; \
        res_a = make_rsrc_words(q_.a_codes + (size_t)m0_ * kb, rows_a_ * kb);                           \
        res_b = make_rsrc_words(q_.b_codes + (size_t)n0_ * kb, rows_b_ * kb);                           \
        const uint32_t srow0_ = scales_of_a ? m0_ : n0_, srows_ = scales_of_a ? rows_a_ : rows_b_;      \
        res_s = make_rsrc_words((scales_of_a ? q_.a_scales : q_.b_scales) + (size_t)(srow0_ >> 5) * kq_ * 256u, \
                                ((srows_ + 31u) >> 5) * kq_ * 256u);                                    \
    }
    STREAM_ISSUE_SETUP()

    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)&lds[0];
    // the lane's 16-byte chunk of a 128-byte code row in the quad's first and second K-step (chunk c of row r lies at c ^ (r/2)%8)
    const uint32_t chunk0 = quarter ^ (l16 >> 1), chunk1 = chunk0 ^ 4u;
    const uint32_t fa_pos0 = ((wm0 + l16) * 8u + chunk0) * 16u, fb_pos0 = ((BM + wn0 + l16) * 8u + chunk0) * 16u;
    const uint32_t fa_pos1 = ((wm0 + l16) * 8u + chunk1) * 16u, fb_pos1 = ((BM + wn0 + l16) * 8u + chunk1) * 16u;
    const uint8_t* lds_bytes = reinterpret_cast<const uint8_t*>(lds);
    const uint32_t srow = (quarter & 1u) * 32u + l16;
    const uint32_t sa_pos = CODES * 16u + ((wm0 >> 5) * 64u + srow) * 4u, sb_pos = CODES * 16u + ((8u + (wn0 >> 5)) * 64u + srow) * 4u;
    const uint32_t sel_full = scale_selector(lane, 0u, 8u);

    // fragments: the wave's 8 row blocks of A and 8 column blocks of B, 16 x 128 elements each, of a quad's first and second K-step
    uint32_t sa[2 * TM], sb[2 * TN], ra_n[2 * TM], rb_n[2 * TN];
    v4i_t fa0[2 * TM], fb0[2 * TN], fa1[2 * TM], fb1[2 * TN];

// load J (0..7: A rows, 8..15: B rows, 16: scale tiles) of the issue cursor's quad into ring slot SLOT
#define STREAM_ISSUE(SLOT, J)                                                                           \
    {                                                                                                   \
        const uint32_t slot_ = lds0 + ((SLOT) * QUAD + wave * 64u) * 16u;                               \
        if ((J) < 16u) {                                                                                \
            const uint32_t base_ = (ikq * 128u + dcol * 16u < kb) ? goff + ikq * 128u : kOutOfRange;    \
            lds_direct_load16((J) < 8u ? res_a : res_b, base_ + ((J) & 7u) * gstep, slot_ + (J) * 4096u); \
        } else {                                                                                        \
            lds_direct_load16(res_s, soff + ikq * 256u, slot_ + CODES * 16u);                           \
        }                                                                                               \
    }
// the quad is issued: move the cursor on (to the next tile of this block after the tile's last quad)
#define STREAM_ISSUE_ADVANCE()                                                                          \
    {                                                                                                   \
        ++iq;                                                                                           \
        ++ikq;                                                                                          \
        if (ikq == kq) ikq = 0u;                                                                        \
        if (iq == kq) {                                                                                 \
            iq = 0u;                                                                                    \
            WALK_NEXT(iw)                                                                               \
            STREAM_ISSUE_SETUP()                                                                        \
        }                                                                                               \
    }
// LDS positions of the lane's part of the first fragments and scales in ring slot SLOT, kept in one register each (the rest is
// immediate offsets; left to itself the compiler forms an address per read)
#define STREAM_AT(NAME, SLOT, POS) uint32_t NAME = (SLOT) * QUAD * 16u + (POS); asm volatile("" : "+v"(NAME));
// fragment R of a K-step in the order the instructions need them: A 0, B 0..7, A 1..7
#define STREAM_FRAG(FA, FB, AT_A, AT_B, R)                                                              \
    {                                                                                                   \
        if ((R) >= 1u && (R) <= 8u) FB[((R) + 7u) & 7u] = *reinterpret_cast<const v4i_t*>(lds_bytes + (AT_B) + (((R) + 7u) & 7u) * 2048u); \
        else FA[((R) + 8u) & 7u] = *reinterpret_cast<const v4i_t*>(lds_bytes + (AT_A) + (((R) + 8u) & 7u) * 2048u); \
    }
#define STREAM_FENCE() __builtin_amdgcn_sched_barrier(0);

    constexpr uint32_t DRAIN = 0x0070u;                // every LDS-direct load has landed and no LDS read is outstanding
    constexpr uint32_t DRAIN_BUT_STORES = 0xC07Fu;     // the same when 64 younger stores are on their way (63 operations may be left)
#pragma unroll
    for (uint32_t j = 0; j < 17u; ++j) STREAM_ISSUE(0u, j)
    STREAM_ISSUE_ADVANCE()
    __builtin_amdgcn_s_waitcnt(DRAIN);
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (uint32_t j = 0; j < 17u; ++j) STREAM_ISSUE(1u, j)
    STREAM_ISSUE_ADVANCE()
#pragma unroll
    for (uint32_t r = 0; r < 16u; ++r) STREAM_FRAG(fa0, fb0, fa_pos0, fb_pos0, r)
// Scale dwords of a K-quad, in two steps: the raw dwords are read from ring slot SLOT behind the barrier and the next
// quad's first fragments, and turned into operands (of local quad QUADN of a tile whose product has GK groups along K) only behind
// the current quad's last matrix-core instruction.
#define STREAM_SCALES_READ_A(SLOT)                                                                      \
    {                                                                                                   \
        STREAM_AT(at_, SLOT, sa_pos)                                                                    \
        const uint32_t* s_ = reinterpret_cast<const uint32_t*>(lds_bytes + at_);                        \
        _Pragma("unroll") for (uint32_t i = 0; i < 2u * TM; ++i) ra_n[i] = s_[i / 2u * 64u + i % 2u * 16u]; \
    }
#define STREAM_SCALES_READ_B(SLOT)                                                                      \
    {                                                                                                   \
        STREAM_AT(at_, SLOT, sb_pos)                                                                    \
        const uint32_t* s_ = reinterpret_cast<const uint32_t*>(lds_bytes + at_);                        \
        _Pragma("unroll") for (uint32_t j = 0; j < 2u * TN; ++j) rb_n[j] = s_[j / 2u * 64u + j % 2u * 16u]; \
    }
#define STREAM_SCALES_USE(QUADN, GK)                                                                    \
    {                                                                                                   \
        uint32_t sel_ = sel_full;                                                                       \
        if (((QUADN) + 1u) * 8u > (GK)) sel_ = scale_selector(lane, (QUADN) * 8u, (GK));   /* wave-uniform: only a ragged last K-quad */ \
        _Pragma("unroll") for (uint32_t i = 0; i < 2u * TM; ++i) sa[i] = __builtin_amdgcn_perm(0x7F7F7F7Fu, ra_n[i], sel_); \
        _Pragma("unroll") for (uint32_t j = 0; j < 2u * TN; ++j) sb[j] = __builtin_amdgcn_perm(0x7F7F7F7Fu, rb_n[j], sel_); \
        mfma_scales_written(sa, sb);                                                                    \
    }
    TileWalk cw;                                         // the tile being computed
    WALK_START(cw)
    STREAM_SCALES_READ_A(0u)
    STREAM_SCALES_READ_B(0u)
    STREAM_SCALES_USE(0u, batch.p[cw.sel].k >> 5)
// One K-quad: two K-steps of 64 matrix-core instructions; SL = its ring slot.  The fragments of a K-step are read one by one during the
// step before it.  The quad's one barrier stands between its steps: every wave has read its last fragment of the slot, so the
// quad after the next is loaded into it during the second step, and every load of the next quad (issued a whole quad earlier) has
// landed.  Reads and loads are spread over the instructions: bunched in a quarter of the step they made the matrix cores wait
// for the LDS.  STORES: the previous tile's result stores, younger than the loads waited for, may still be under way.
#define STREAM_MF(STEP, I, J)                                                                           \
    if (STEP) mfma_fp4<1>(fa1[I], fb1[J], acc[I][J], sa[I], sb[J]);                                     \
    else mfma_fp4<0>(fa0[I], fb0[J], acc[I][J], sa[I], sb[J]);                                          \
    STREAM_FENCE()
// instruction number N of a step and what follows it: fragment reads of the next K-step behind every third, and in the second step
// the loads behind the instructions in between
#define STREAM_AFTER0(N)                                                                                \
    if ((N) % 3u == 0u && (N) < 48u) { STREAM_FRAG(fa1, fb1, a1_, b1_, (N) / 3u) STREAM_FENCE() }
#define STREAM_AFTER1(N)                                                                                \
    if ((N) % 3u == 0u && (N) < 48u) { STREAM_FRAG(fa0, fb0, an_, bn_, (N) / 3u) STREAM_FENCE() }       \
    if ((N) % 3u == 1u && (N) < 51u) { STREAM_ISSUE(SL_, (N) / 3u) STREAM_FENCE() }                     \
    if ((N) == 48u) { STREAM_SCALES_READ_A(so_) STREAM_FENCE() }                                        \
    if ((N) == 51u) { STREAM_SCALES_READ_B(so_) STREAM_FENCE() }
#define STREAM_ROW(STEP, I)                                                                             \
    STREAM_MF(STEP, I, 0) STREAM_AFTER##STEP((I) * 8u) STREAM_MF(STEP, I, 1) STREAM_AFTER##STEP((I) * 8u + 1u) \
    STREAM_MF(STEP, I, 2) STREAM_AFTER##STEP((I) * 8u + 2u) STREAM_MF(STEP, I, 3) STREAM_AFTER##STEP((I) * 8u + 3u) \
    STREAM_MF(STEP, I, 4) STREAM_AFTER##STEP((I) * 8u + 4u) STREAM_MF(STEP, I, 5) STREAM_AFTER##STEP((I) * 8u + 5u) \
    STREAM_MF(STEP, I, 6) STREAM_AFTER##STEP((I) * 8u + 6u) STREAM_MF(STEP, I, 7) STREAM_AFTER##STEP((I) * 8u + 7u)
#define STREAM_BODY(SL, STORES, NEXT_QUAD, NEXT_GK)                                                     \
    {                                                                                                   \
        const uint32_t SL_ = (SL), so_ = SL_ ^ 1u;                                                      \
        STREAM_AT(a1_, SL_, fa_pos1) STREAM_AT(b1_, SL_, fb_pos1)                                       \
        STREAM_AT(an_, so_, fa_pos0) STREAM_AT(bn_, so_, fb_pos0)                                       \
        STREAM_ROW(0, 0) STREAM_ROW(0, 1) STREAM_ROW(0, 2) STREAM_ROW(0, 3)                             \
        STREAM_ROW(0, 4) STREAM_ROW(0, 5) STREAM_ROW(0, 6) STREAM_ROW(0, 7)                             \
        if (STORES) __builtin_amdgcn_s_waitcnt(DRAIN_BUT_STORES);                                       \
        else __builtin_amdgcn_s_waitcnt(DRAIN);                                                         \
        __builtin_amdgcn_s_barrier();                                                                   \
        STREAM_FENCE()                                                                                  \
        STREAM_ROW(1, 0) STREAM_ROW(1, 1) STREAM_ROW(1, 2) STREAM_ROW(1, 3)                             \
        STREAM_ROW(1, 4) STREAM_ROW(1, 5) STREAM_ROW(1, 6)                                              \
        STREAM_ISSUE_ADVANCE()                                                                          \
        STREAM_FENCE()                                                                                  \
        STREAM_ROW(1, 7)                                                                                \
        STREAM_SCALES_USE(NEXT_QUAD, NEXT_GK)                                                           \
        STREAM_FENCE()                                                                                  \
    }

    v4f acc[2 * TM][2 * TN];
    float* wbuf = reinterpret_cast<float*>(&lds[2u * QUAD]) + wave * 1024u;
    uint32_t sl = 0u;                                      // ring slot of the current quad
    bool stores = false;                                   // the previous tile's 64 result stores are younger than the loads to wait for
    while (cw.sel == 0u || cw.tile < second_tiles) {
        const uint32_t csel = cw.sel, clv = cw.tile;
        const uint32_t ck = batch.p[csel].k, gk = ck >> 5, quads = ck ? (ck + 255u) >> 8 : 1u;
        // the tile's last quad reads the first scales of the block's next tile, which may belong to the other product
        WALK_NEXT(cw)
        const uint32_t gk_after = batch.p[cw.sel].k >> 5;
        mfma_clear_accumulators(acc);                      // (the first quad apart, with the constant 0 in their place, spills)
        __builtin_amdgcn_sched_barrier(0);
        for (uint32_t qd = 0u; qd < quads; ++qd, sl ^= 1u) {
            const bool last = qd + 1u == quads;            // the next quad is the next tile's first
            STREAM_BODY(sl, stores, last ? 0u : qd + 1u, last ? gk_after : gk)
            stores = false;
        }
        mfma_results_written();
        __builtin_amdgcn_sched_barrier(0);
        // The ring already holds the next tile's first quad and is receiving its second, and fa0 / fb0 / sa / sb hold its first
        // fragments and scales.  The vector-memory counter retires in order: the next tile's first barrier waits for loads older than
        // the result stores below, its second one for the stores as well.
        const GemmProblem& q = batch.p[csel];
        uint32_t m0, n0;
        STREAM_TILE(q, clv, m0, n0)
        const uint32_t m = q.m, n = q.n, ldd = q.ldd;
        const uint32_t* __restrict__ mask = q.mask;
        const uint32_t row_base = m0 + wm0, col_base = n0 + wn0;
        const bool full = (ldd & 3u) == 0u && row_base + TM * 32u <= m && col_base + TN * 32u <= n && (!FUSED || mask != nullptr);
        if constexpr (WIDE) store_tile_rows8<TM, TN, OUT_BF16, FUSED, true, true>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        else if (full) store_tile_rows8<TM, TN, OUT_BF16, FUSED, true>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        else store_tile_rows8<TM, TN, OUT_BF16, FUSED, false>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        stores = WIDE || full;                             // 16 passes of four stores each; a ragged tile may have skipped some
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the quads issued past the last tile (zero-filled) have landed before the LDS is given back
    if (clock_counters && tid == 0) {
        const uint64_t t1 = __builtin_readcyclecounter(), w1 = __builtin_amdgcn_s_memrealtime();
        atomicAdd(reinterpret_cast<unsigned long long*>(clock_counters), (unsigned long long)(t1 - clk_t0));
        atomicAdd(reinterpret_cast<unsigned long long*>(clock_counters) + 1, (unsigned long long)(w1 - clk_w0));
    }
#undef STREAM_TILE
#undef STREAM_ISSUE_SETUP
#undef STREAM_ISSUE
#undef STREAM_ISSUE_ADVANCE
#undef STREAM_AT
#undef STREAM_FRAG
#undef STREAM_AFTER0
#undef STREAM_AFTER1
#undef STREAM_FENCE
#undef STREAM_SCALES_READ_A
#undef STREAM_SCALES_READ_B
#undef STREAM_SCALES_USE
#undef STREAM_MF
#undef STREAM_ROW
#undef STREAM_BODY
}

template <bool OUT_BF16, bool FUSED>
__global__ void __launch_bounds__(256)
gemm_mxfp4_stream_kernel(GemmBatch batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    stream_large_tiles<OUT_BF16, FUSED, false>(batch, nb, clock_counters);
}

template <bool FUSED>
__global__ void __launch_bounds__(256)
gemm_mxfp4_past_kernel(GemmBatch batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    stream_large_tiles<true, FUSED, false, true>(batch, nb, clock_counters);
}

__global__ void __launch_bounds__(256)
gemm_mxfp4_past_wide_kernel(GemmBatch batch, uint64_t* __restrict__ clock_counters) {
    stream_large_tiles<true, true, true, true>(batch, 8u, clock_counters);
}

template <bool OUT_BF16>
__global__ void __launch_bounds__(256)
gemm_mxfp4_wide_kernel(GemmBatch batch, uint64_t* __restrict__ clock_counters) {
    stream_large_tiles<OUT_BF16, true, true>(batch, 8u, clock_counters);
}

// ---------------------------------------------------------------------------------------------
// The streaming design for other tile shapes: wave tile (TM*32) x (TN*32), block tile (64 TM) x (64 TN), for problems
// whose 256 x 256 tiles would leave compute units idle.  Same issue cursor, same epilogue; the instruction order is generated from the
// tile shape.  A quad of these tiles lasts 0.3-0.6 us, less than a load's way from memory, so the ring has S = 3 or 4 slots (what
// fits): during the first three K-steps (64 elements) of quad q go out the loads of quad q + S - 1.  The quad's one barrier stands
// before its last K-step, whose fragments every wave has read by then.  That leaves the slot of a tile's last quad free until the
// next tile begins: it serves as the epilogue's scratch.
// Instructions of 32 x 32 x 64 (two sets of fragments, even and odd K-steps): these problems are bound by what a wave can issue and by
// the L2, not by power, and the smaller instruction of the 256 x 256 kernel means twice as many of them for the same work.  Measured
// against 16 x 16 x 128 (us, fp32 results): 128 x 128 tiles 2048 x 2048 x 4096 14.6 / 16.0, 4096 x 4096 x 1024 21.0 / 22.8, 4096^3 47.4 / 49.2;
// 128 x 256 tiles 18.1 / 20.5, 19.8 / 21.0, 41.2 / 42.3; same bits.
// PER_CU = 2: two blocks share a compute unit (each with two slots and epilogue scratch of its own, 80 KB), so one multiplies while the
// other waits for its loads or stores its results.  A quad's slot is filled again behind the quad's own barrier, and the loads have
// three quarters of a quad to land: with several tiles per compute unit that is less than what the epilogues cost one block alone.
// Pairs of layers (tokens, in, out), one block / two (us): 608 x 8832 x 3424 63.6 / 52.7, 4800 x 1824 x 2112 48.9 / 43.6, 9600 x 576 x 576 32.4 /
// 36.0 (a tile or two per compute unit: the deeper ring); single products 10327 x 992 x 800 21.1 / 17.9, 4926 x 6496 x 10144 230 / 251.
template <int TM, int TN, int PER_CU, bool OUT_BF16, bool FUSED, bool WIDE = false, bool PAST16 = false>
__device__ __forceinline__ void stream_tiles(const GemmBatch& batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    constexpr uint32_t BM = 64 * TM, BN = 64 * TN;
    static_assert(BM % 128 == 0 && BN % 128 == 0, "a wave's four scale tiles must belong to one operand");
    constexpr uint32_t CODES = (BM + BN) * 8;            // 16-byte chunks of codes per K-quad
    constexpr uint32_t QUAD = CODES + 256;               // + room for 16 scale tiles of 256 B (one KB per wave)
    constexpr uint32_t S = PER_CU == 2 ? 2u : BN == 256 ? 3u : 4u;   // ring slots
    constexpr bool LATE = S == 2u;                       // a quad's slot is filled again behind its own barrier
    constexpr uint32_t LA = BM / 32, LB = BN / 32, NL = LA + LB;   // LDS-direct loads of codes per wave per quad
    constexpr uint32_t NT = (BM + BN) / 32;              // scale tiles per K-quad: A's, then B's
    constexpr int NM = TM * TN, R = TM + TN;             // matrix-core instructions and fragment reads per K-step (64 elements)
    constexpr uint32_t EPI = LATE ? 4u * TN * 64u : 0u;  // 16-byte chunks of epilogue scratch beside the ring
    __shared__ v4i_t lds[S * QUAD + EPI];
    static_assert(PER_CU * sizeof(lds) <= 160u * 1024u, "the blocks of a compute unit share its LDS");

    // measurement support: shader-clock and constant-clock ticks of this block's run (wave-uniform branch)
    uint64_t clk_t0 = 0, clk_w0 = 0;
    if (clock_counters) {
        clk_t0 = __builtin_readcyclecounter();
        clk_w0 = __builtin_amdgcn_s_memrealtime();
    }

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lrow = lane & 31u, lhalf = lane >> 5;
    const uint32_t G = gridDim.x, first_tiles = batch.p[0].total_tiles, second_tiles = batch.p[1].total_tiles;
    const uint32_t extra_tiles = batch.extra_tiles, late = batch.late;
    const uint32_t second_start = blockIdx.x + late >= G ? blockIdx.x + late - G : extra_tiles + late + blockIdx.x;
    const uint32_t wm0 = (wave >> 1) * (TM * 32u), wn0 = (wave & 1u) * (TN * 32u);
    // scale tiles 4 wave .. 4 wave + 3 of [A's | B's] are this wave's to fetch (waves past the last tile fetch nothing real:
    // their load is out of range and delivers zeros, which keeps every wave's count of loads the same)
    const bool has_scales = 4u * wave < NT, scales_of_a = 4u * wave < BM / 32u;
    const uint32_t stile0 = scales_of_a ? 4u * wave : 4u * wave - BM / 32u;
    const uint32_t past = OUT_BF16 ? (uint32_t)PAST16 : batch.past;

// tile origin of tile number V of product Q (as in the 256 x 256 kernel)
#define TILE_ORIGIN(Q, V, M0, N0)                                                                       \
    {                                                                                                   \
        const uint32_t v_ = (V), tt_ = (Q).total_tiles;                                                 \
        if (v_ < tt_) {                                                                                 \
            const uint32_t per_ = tt_ >> 3, rem_ = tt_ & 7u, GM_ = (Q).band_height;                     \
            const uint32_t tiles_m_ = (Q).tiles_m, tiles_n_ = (Q).tiles_n;                              \
            const uint32_t xcd_ = v_ & 7u;                                                              \
            const uint32_t tile_ = xcd_ * per_ + (xcd_ < rem_ ? xcd_ : rem_) + (v_ >> 3);               \
            const uint32_t band_ = tile_ / (GM_ * tiles_n_);                                            \
            const uint32_t band_rows_ = (tiles_m_ - band_ * GM_) < GM_ ? (tiles_m_ - band_ * GM_) : GM_; \
            const uint32_t in_band_ = tile_ - band_ * GM_ * tiles_n_;                                   \
            M0 = (band_ * GM_ + in_band_ % band_rows_) * BM;                                            \
            N0 = (in_band_ / band_rows_) * BN;                                                          \
        } else {                                                                                        \
            M0 = (Q).m; N0 = (Q).n;                                                                     \
        }                                                                                               \
    }
    TileWalk iw;                                         // issue cursor: the tile and K-quad the next loads belong to
    uint32_t iq = 0u;
    WALK_START(iw)
    v4i_t res_a, res_b, res_s;
    uint32_t kb, kq, goff, gstep, soff;                  // of the cursor's product
    const uint32_t drow = wave * 8u + (lane >> 3);
    const uint32_t dcol = (lane & 7u) ^ ((drow >> 1) & 7u);
#define ISSUE_SETUP()                                                                                   \
    {                                                                                                   \
        uint32_t m0_, n0_;                                                                              \
        const GemmProblem& q_ = batch.p[iw.sel];                                                        \
        const uint32_t lv_ = iw.tile;                                                                   \
        TILE_ORIGIN(q_, lv_, m0_, n0_)                                                                  \
        const uint32_t k_ = q_.k, kq_ = (k_ + 255u) >> 8;                                               \
        kq = kq_ ? kq_ : 1u;                                                                            \
        kb = k_ >> 1;                                                                                   \
        goff = drow * kb + dcol * 16u;          /* + j*32*kb, + quad*128 */                             \
        gstep = 32u * kb;                                                                               \
        soff = ((stile0 + (lane >> 4)) * kq_) * 256u + (lane & 15u) * 16u;   /* + quad*256 */           \
        const uint32_t rows_a_ = (q_.m - m0_) < BM ? (q_.m - m0_) : BM, rows_b_ = (q_.n - n0_) < BN ? (q_.n - n0_) : BN; \
        res_a = make_rsrc_words(q_.a_codes + (size_t)m0_ * kb, rows_a_ * kb);                           \
        res_b = make_rsrc_words(q_.b_codes + (size_t)n0_ * kb, rows_b_ * kb);                           \
        const uint32_t srow0_ = scales_of_a ? m0_ : n0_, srows_ = scales_of_a ? rows_a_ : rows_b_;      \
        res_s = make_rsrc_words((scales_of_a ? q_.a_scales : q_.b_scales) + (size_t)(srow0_ >> 5) * kq_ * 256u, \
                                has_scales ? ((srows_ + 31u) >> 5) * kq_ * 256u : 0u);                  \
    }
    ISSUE_SETUP()

    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)&lds[0];
    // the lane's 16-byte chunk 2 s + lhalf of a 128-byte code row in K-step s (chunk c of row r lies at c ^ (r/2)%8)
    const uint32_t swz = lhalf ^ ((lrow >> 1) & 7u);
    const uint32_t fa_pos = ((wm0 + lrow) * 8u + swz) * 16u, fb_pos = ((BM + wn0 + lrow) * 8u + swz) * 16u;   // K-step s: ^ 32 s
    const uint32_t sa_pos = CODES * 16u + ((wm0 >> 5) * 64u + lane) * 4u, sb_pos = CODES * 16u + ((BM / 32u + (wn0 >> 5)) * 64u + lane) * 4u;
    const uint8_t* lds_bytes = reinterpret_cast<const uint8_t*>(lds);

    uint32_t sa[TM], sb[TN], ra_n[TM], rb_n[TN];
    uint4 fa[2][TM], fb[2][TN];                          // fragments of even and odd K-steps

// code load J (0 .. LA-1: A rows, LA .. NL-1: B rows) or the scale tiles (J == NL) of the cursor's quad into ring slot SLOT
#define ISSUE(SLOT, J)                                                                                  \
    {                                                                                                   \
        const uint32_t slot_ = lds0 + ((SLOT) * QUAD + wave * 64u) * 16u;                               \
        if ((uint32_t)(J) < NL) {                                                                       \
            const uint32_t base_ = (iq * 128u + dcol * 16u < kb) ? goff + iq * 128u : kOutOfRange;      \
            const uint32_t jj_ = (uint32_t)(J) < LA ? (uint32_t)(J) : (uint32_t)(J) - LA;               \
            lds_direct_load16((uint32_t)(J) < LA ? res_a : res_b, base_ + jj_ * gstep, slot_ + (uint32_t)(J) * 4096u); \
        } else {                                                                                        \
            lds_direct_load16(res_s, soff + iq * 256u, slot_ + CODES * 16u);                            \
        }                                                                                               \
    }
#define ISSUE_ADVANCE()                                                                                 \
    {                                                                                                   \
        ++iq;                                                                                           \
        if (iq == kq) {                                                                                 \
            iq = 0u;                                                                                    \
            WALK_NEXT(iw)                                                                               \
            ISSUE_SETUP()                                                                               \
        }                                                                                               \
    }
// fragment number RR of K-step STEP of the quad in slot SLOT, in the order the instructions need them: A0, B0 .. B(TN-1), A1 ..
#define READ_FRAG(SLOT, STEP, RR)                                                                       \
    {                                                                                                   \
        const int rr_ = (RR);                                                                           \
        if (rr_ >= 1 && rr_ <= TN) fb[(STEP) & 1][rr_ - 1] = *reinterpret_cast<const uint4*>(lds_bytes + (SLOT) * QUAD * 16u + (fb_pos ^ ((STEP) * 32u)) + (rr_ - 1) * 4096); \
        else if (rr_ < R) fa[(STEP) & 1][rr_ == 0 ? 0 : rr_ - TN] = *reinterpret_cast<const uint4*>(lds_bytes + (SLOT) * QUAD * 16u + (fa_pos ^ ((STEP) * 32u)) + (rr_ == 0 ? 0 : rr_ - TN) * 4096); \
    }
#define FENCE() __builtin_amdgcn_sched_barrier(0);
#define READ_SCALES(SLOT)                                                                               \
    {                                                                                                   \
        const uint32_t* s_a_ = reinterpret_cast<const uint32_t*>(lds_bytes + (SLOT) * QUAD * 16u + sa_pos); \
        const uint32_t* s_b_ = reinterpret_cast<const uint32_t*>(lds_bytes + (SLOT) * QUAD * 16u + sb_pos); \
        _Pragma("unroll") for (uint32_t i = 0; i < TM; ++i) ra_n[i] = s_a_[i * 64u];                    \
        _Pragma("unroll") for (uint32_t j = 0; j < TN; ++j) rb_n[j] = s_b_[j * 64u];                    \
    }
#define USE_SCALES(QUADN, GK)                                                                           \
    {                                                                                                   \
        uint32_t keep_ = 0xFFFFFFFFu;                                                                   \
        if (((QUADN) + 1u) * 8u > (GK)) {     /* wave-uniform: only a ragged last K-quad */             \
            const uint32_t steps_ = ((GK) + 1u - lhalf) >> 1, done_ = (QUADN) * 4u;                     \
            const uint32_t nv_ = steps_ > done_ ? (steps_ - done_ < 4u ? steps_ - done_ : 4u) : 0u;     \
            keep_ = nv_ >= 4u ? 0xFFFFFFFFu : ((1u << (8u * nv_)) - 1u);                                \
        }                                                                                               \
        _Pragma("unroll") for (uint32_t i = 0; i < TM; ++i) sa[i] = (ra_n[i] & keep_) | (0x7F7F7F7Fu & ~keep_); \
        _Pragma("unroll") for (uint32_t j = 0; j < TN; ++j) sb[j] = (rb_n[j] & keep_) | (0x7F7F7F7Fu & ~keep_); \
    }

    // vector-memory operations that may be under way at a quad's barrier: the loads of the quads behind the next one, and once after a
    // tile's end its result stores, which are younger than the next quad's loads
    constexpr uint32_t FIRST = LATE ? 2u : S - 1u, AHEAD0 = (FIRST - 1u) * (NL + 1u);   // quads loaded before the first barrier
    constexpr uint32_t AHEAD = (S - 2u) * (NL + 1u), AHEAD_ST = AHEAD + TM * 4u * TN;
    static_assert(AHEAD_ST < 64u, "the counter has six bits");
    constexpr uint32_t WAIT0 = 0x0070u | (AHEAD0 & 15u) | ((AHEAD0 >> 4) << 14);
    constexpr uint32_t WAIT = 0x0070u | (AHEAD & 15u) | ((AHEAD >> 4) << 14);      // and no LDS read is outstanding
    constexpr uint32_t WAIT_ST = 0x0070u | (AHEAD_ST & 15u) | ((AHEAD_ST >> 4) << 14);
#pragma unroll
    for (uint32_t s0 = 0; s0 < FIRST; ++s0) {
#pragma unroll
        for (uint32_t j = 0; j <= NL; ++j) ISSUE(s0, j)
        ISSUE_ADVANCE()
    }
    __builtin_amdgcn_s_waitcnt(WAIT0);
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) READ_FRAG(0u, 0, r)
    TileWalk cw;                                         // the tile being computed
    WALK_START(cw)
    READ_SCALES(0u)
    USE_SCALES(0u, batch.p[cw.sel].k >> 5)

// the instruction of a quad behind which load L goes out: spread over the first three K-steps, with two slots over the last one
#define ISSUE_AT(L) (LATE ? 3 * NM + (L) * NM / ((int)NL + 1) : (L) * 3 * NM / ((int)NL + 1))
// one K-quad in slot SL; SL1: the next quad's slot, SLI: the slot being filled (SL itself behind the barrier with two slots)
#define QUAD_BODY(SL, SL1, SLI, STORES, NEXT_QUAD, NEXT_GK)                                             \
    {                                                                                                   \
        _Pragma("unroll") for (int idx = 0; idx < 4 * NM; ++idx) {                                      \
            const int st_ = idx / NM, ij_ = idx % NM, I_ = ij_ / TN, J_ = ij_ % TN;                     \
            if (st_ == 0) acc[I_][J_] = mfma_fp4_32<0>(fa[0][I_], fb[0][J_], acc[I_][J_], sa[I_], sb[J_]); \
            if (st_ == 1) acc[I_][J_] = mfma_fp4_32<1>(fa[1][I_], fb[1][J_], acc[I_][J_], sa[I_], sb[J_]); \
            if (st_ == 2) acc[I_][J_] = mfma_fp4_32<2>(fa[0][I_], fb[0][J_], acc[I_][J_], sa[I_], sb[J_]); \
            if (st_ == 3) acc[I_][J_] = mfma_fp4_32<3>(fa[1][I_], fb[1][J_], acc[I_][J_], sa[I_], sb[J_]); \
            asm volatile("" : "+a"(acc[I_][J_]));                                                       \
            FENCE()                                                                                     \
            if (st_ < 2 && ij_ < R) { READ_FRAG(SL, st_ + 1, ij_) FENCE() }                             \
            if (st_ == 2 && 2 * ij_ < R) { READ_FRAG(SL, 3, 2 * ij_) READ_FRAG(SL, 3, 2 * ij_ + 1) FENCE() } \
            _Pragma("unroll") for (int l_ = 0; l_ <= (int)NL; ++l_)                                     \
                if (ISSUE_AT(l_) == idx) { ISSUE(SLI, l_) FENCE() }                                     \
            if (idx == 3 * NM - 1) {                                                                    \
                if (!LATE) ISSUE_ADVANCE()                                                              \
                if (STORES) __builtin_amdgcn_s_waitcnt(WAIT_ST);                                        \
                else __builtin_amdgcn_s_waitcnt(WAIT);                                                  \
                __builtin_amdgcn_s_barrier();                                                           \
                FENCE()                                                                                 \
            }                                                                                           \
            if (R < NM && st_ == 3 && ij_ < R) { READ_FRAG(SL1, 0, ij_) FENCE() }                       \
            if (R >= NM && st_ == 3 && 2 * ij_ < R) { READ_FRAG(SL1, 0, 2 * ij_) READ_FRAG(SL1, 0, 2 * ij_ + 1) FENCE() } \
            if (idx == 3 * NM + (R < NM ? R : (R + 1) / 2)) { READ_SCALES(SL1) FENCE() }                \
            if (LATE && idx == 4 * NM - 1) { ISSUE_ADVANCE() FENCE() }                                  \
        }                                                                                               \
        USE_SCALES(NEXT_QUAD, NEXT_GK)                                                                  \
        FENCE()                                                                                         \
    }

    v16f acc[TM][TN];
    uint32_t sl = 0u;                                      // ring slot of the current quad
    auto slot_after = [](uint32_t s) { return s + 1u == S ? 0u : s + 1u; };
    auto slot_before = [](uint32_t s) { return s == 0u ? S - 1u : s - 1u; };
    bool stores = false;                                   // the previous tile's result stores are younger than the loads to wait for
    while (cw.sel == 0u || cw.tile < second_tiles) {
        const uint32_t csel = cw.sel, clv = cw.tile;
        const uint32_t ck = batch.p[csel].k, gk = ck >> 5, quads = ck ? (ck + 255u) >> 8 : 1u;
        // the tile's last quad reads the first scales of the block's next tile, which may belong to the other product
        WALK_NEXT(cw)
        const uint32_t gk_after = batch.p[cw.sel].k >> 5;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        uint32_t sl1 = slot_after(sl);
        QUAD_BODY(sl, sl1, LATE ? sl : slot_before(sl), stores, quads > 1u ? 1u : 0u, quads > 1u ? gk : gk_after)
        for (uint32_t qd = 1u; qd < quads; ++qd) {
            const bool last = qd + 1u == quads;            // the next quad is the next tile's first
            sl = sl1;
            sl1 = slot_after(sl);
            QUAD_BODY(sl, sl1, LATE ? sl : slot_before(sl), false, last ? 0u : qd + 1u, last ? gk_after : gk)
        }
        __builtin_amdgcn_sched_barrier(0);
        // scratch: the last quad's slot, where every wave is past its last read and the next loads go out behind the barrier below
        float* wbuf = reinterpret_cast<float*>(&lds[(LATE ? S : sl) * QUAD]) + wave * (TN * 256u);
        sl = sl1;
        const GemmProblem& q = batch.p[csel];
        uint32_t m0, n0;
        TILE_ORIGIN(q, clv, m0, n0)
        const uint32_t m = q.m, n = q.n, ldd = q.ldd;
        const uint32_t* __restrict__ mask = q.mask;
        const uint32_t row_base = m0 + wm0, col_base = n0 + wn0;
        const bool full = (ldd & 3u) == 0u && row_base + TM * 32u <= m && col_base + TN * 32u <= n && (!FUSED || mask != nullptr);
        if constexpr (WIDE) store_tile_rows8<TM, TN, OUT_BF16, FUSED, true, true>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        else if (full) store_tile_rows8<TM, TN, OUT_BF16, FUSED, true>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        else store_tile_rows8<TM, TN, OUT_BF16, FUSED, false>(acc, wbuf, q.d, ldd, mask, q.alpha, row_base, col_base, m, n, lane, nb, past);
        stores = WIDE || full;                             // every store was issued; a ragged tile may have skipped some
        if (!LATE) {
            __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the quads issued past the last tile (zero-filled) have landed before the LDS is given back
    if (clock_counters && tid == 0) {
        const uint64_t t1 = __builtin_readcyclecounter(), w1 = __builtin_amdgcn_s_memrealtime();
        atomicAdd(reinterpret_cast<unsigned long long*>(clock_counters), (unsigned long long)(t1 - clk_t0));
        atomicAdd(reinterpret_cast<unsigned long long*>(clock_counters) + 1, (unsigned long long)(w1 - clk_w0));
    }
#undef TILE_ORIGIN
#undef ISSUE_SETUP
#undef ISSUE
#undef ISSUE_ADVANCE
#undef READ_FRAG
#undef FENCE
#undef READ_SCALES
#undef USE_SCALES
#undef ISSUE_AT
#undef QUAD_BODY
}

template <int TM, int TN, bool OUT_BF16, bool FUSED>
__global__ void __launch_bounds__(256)
gemm_mxfp4_stream_tile_kernel(GemmBatch batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    stream_tiles<TM, TN, 1, OUT_BF16, FUSED>(batch, nb, clock_counters);
}

template <bool OUT_BF16>
__global__ void __launch_bounds__(256)
gemm_mxfp4_wide_tile_kernel(GemmBatch batch, uint64_t* __restrict__ clock_counters) {
    stream_tiles<2, 4, 1, OUT_BF16, true, true>(batch, 8u, clock_counters);
}

template <bool OUT_BF16, bool FUSED>
__global__ void __launch_bounds__(256, 2)
gemm_mxfp4_twin_kernel(GemmBatch batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    stream_tiles<2, 2, 2, OUT_BF16, FUSED>(batch, nb, clock_counters);
}

template <bool FUSED>
__global__ void __launch_bounds__(256, 2)
gemm_mxfp4_past_twin_kernel(GemmBatch batch, uint32_t nb, uint64_t* __restrict__ clock_counters) {
    stream_tiles<2, 2, 2, true, FUSED, false, true>(batch, nb, clock_counters);
}

static int stream_blocks() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n >= 8)
            cus = n & ~7;
        else
            cus = 8;
    }
    return cus;
}

// Results of a launch that the memory-side cache (256 MB) cannot hold beside its operands are stored past it: they would only push those and
// what follows out.  Less is stored through the L2 and stays there for its reader.  Through the L2 / past the cache (us), layer steps
// (tokens, in, out): fp32 16384 x 2048 x 4096 (y 256 MB) 357 / 344, 16384 x 4096 x 4096 572 / 534, 8192 x 7936 x 1024 (gradients 279 MB) 229 / 219; bf16
// 16384 x 2048 x 8192 (y 256 MB) 605 / 592, 16384 x 8192 x 1024 (gradients 272 MB) 447 / 430, 12544 x 10752 x 2048 659 / 637.  A forward pass of 256 MB that is
// repeated alone is 1-10 % slower past the cache (fp32 8192 x 2048 x 8192 107 / 117), from 264 MB on 0-6 % faster.  For bf16 on the kernels that such
// launches take; 128 x 256 tiles, which take 1 in 1000 of them, and forced 128 x 128 ones with one block per compute unit stay with the L2.
static uint32_t stored_past(const GemmBatch& batch, bool bf16) {
    const double results = (double)batch.p[0].m * batch.p[0].n + (double)batch.p[1].m * batch.p[1].n;
    return results * (bf16 ? 2.0 : 4.0) >= 256.0 * 1024.0 * 1024.0 ? 1u : 0u;
}

// tile grid and band height of one product for block tiles of bm x bn
static GemmProblem make_problem(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* b_codes, const uint8_t* b_scales,
                                int64_t m, int64_t n, int64_t k, float alpha, void* d, int64_t ldd, const uint32_t* mask,
                                int64_t bm, int64_t bn) {
    GemmProblem q;
    q.a_codes = a_codes; q.a_scales = a_scales; q.b_codes = b_codes; q.b_scales = b_scales;
    q.d = d; q.mask = mask;
    q.m = (uint32_t)m; q.n = (uint32_t)n; q.k = (uint32_t)k; q.ldd = (uint32_t)ldd;
    q.alpha = alpha;
    q.tiles_m = (uint32_t)((m + bm - 1) / bm); q.tiles_n = (uint32_t)((n + bn - 1) / bn);
    q.band_height = (bm == 256 && bn == 256 && q.tiles_n >= 40u && (q.tiles_m & 1u) == 0u) ? 2u : 4u;
    if (g_forced_band > 0) q.band_height = (uint32_t)g_forced_band;
    q.total_tiles = q.tiles_m * q.tiles_n;
    return q;
}

template <bool OUT_BF16, bool FUSED>
static void launch_stream_batch_t(const GemmBatch& batch, uint32_t nb, hipStream_t st) {
    const uint32_t total = batch.p[0].total_tiles + batch.p[1].total_tiles, cus = (uint32_t)stream_blocks();
    const dim3 grid(total < cus ? total : cus);
    if (OUT_BF16 && batch.past) hipLaunchKernelGGL((gemm_mxfp4_past_kernel<FUSED>), grid, dim3(256), 0, st, batch, nb, g_clock_counters);
    else hipLaunchKernelGGL((gemm_mxfp4_stream_kernel<OUT_BF16, FUSED>), grid, dim3(256), 0, st, batch, nb, g_clock_counters);
}

template <bool OUT_BF16, bool FUSED>
static void launch_stream_t(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* b_codes,
                            const uint8_t* b_scales, int64_t m, int64_t n, int64_t k, float alpha, void* d,
                            int64_t ldd, const uint32_t* mask, uint32_t nb, hipStream_t st) {
    GemmBatch batch;
    batch.p[0] = make_problem(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, 256, 256);
    batch.p[1] = GemmProblem{};      // no second product
    batch.past = stored_past(batch, OUT_BF16);
    batch.extra_tiles = batch.late = 0u;
    launch_stream_batch_t<OUT_BF16, FUSED>(batch, nb, st);
}

template <int TM, int TN, int PER_CU, bool OUT_BF16, bool FUSED>
static void launch_stream_tile_batch_t(const GemmBatch& batch, uint32_t nb, hipStream_t st) {
    const uint32_t total = batch.p[0].total_tiles + batch.p[1].total_tiles, room = PER_CU * (uint32_t)stream_blocks();
    const dim3 grid(total < room ? total : room);
    if (PER_CU == 2 && OUT_BF16 && batch.past) hipLaunchKernelGGL((gemm_mxfp4_past_twin_kernel<FUSED>), grid, dim3(256), 0, st, batch, nb, g_clock_counters);
    else if constexpr (PER_CU == 2) hipLaunchKernelGGL((gemm_mxfp4_twin_kernel<OUT_BF16, FUSED>), grid, dim3(256), 0, st, batch, nb, g_clock_counters);
    else hipLaunchKernelGGL((gemm_mxfp4_stream_tile_kernel<TM, TN, OUT_BF16, FUSED>), grid, dim3(256), 0, st, batch, nb, g_clock_counters);
}

template <int TM, int TN, int PER_CU, bool OUT_BF16, bool FUSED>
static void launch_stream_tile_t(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* b_codes,
                                 const uint8_t* b_scales, int64_t m, int64_t n, int64_t k, float alpha, void* d,
                                 int64_t ldd, const uint32_t* mask, uint32_t nb, hipStream_t st) {
    GemmBatch batch;
    batch.p[0] = make_problem(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, 64 * TM, 64 * TN);
    batch.p[1] = GemmProblem{};      // no second product
    batch.past = stored_past(batch, OUT_BF16);
    batch.extra_tiles = batch.late = 0u;
    launch_stream_tile_batch_t<TM, TN, PER_CU, OUT_BF16, FUSED>(batch, nb, st);
}

// Variants: 0 = 256x256 tiles (hand-scheduled K-quad), 1 = 128x256 tiles, 2 = 128x128 tiles (schedule generated from the
// tile shape), kTwoPerCu = 128x128 tiles with two blocks per compute unit; blocks stream their tiles through a ring of K-quads, two
// K-steps per trip with the scale byte picked by op_sel.  set_gemm_plan overrides the size heuristic (tests reach every variant
// through it).
// fused != 0: D = alpha * H_along_n((A B^T) . mask) with Hadamard blocks of nb = 1, 2 or 4 groups of 32 columns (mask may
// be null = all ones), n % (32 nb) == 0.
//
// The tile shape is the one with the smallest estimated time: launch and first loads, the share of the chip that starts, the
// busiest compute unit's K-quads and its tiles' epilogues (weighed with the mean: the last round runs on a chip that is partly idle), or
// what the memory takes for the results if that is more.  Fitted to the products of 330 layers' backward passes (tokens 256 .. 16384, in and
// out 256 .. 11008) and of 400 forward or serving calls (m 8 .. 16384), both result types, every shape timed behind the conversions that
// write its operands: the shape chosen costs 1.0 % (pairs) and 1.1 % (singles) more than the best one on average, 7 / 5 % at the 95th
// percentile.  Measured, 256 x 256 / 128 x 256 / 128 x 128 / 128 x 128 with two blocks per compute unit (us): pairs (dW, dx) of layers (tokens,
// in, out) 4608 x 2432 x 6016 107 / 104 / 105 / 95, 13696 x 2816 x 832 101 / 69 / 77 / 80; single products 4253 x 3648 x 5408 59.7 / 62.3 / 72.8 /
// 69.2, 2860 x 4448 x 320 18.2 / 17.2 / 16.2 / 13.2.
struct StreamCost {
    double start, per_quad, per_tile, per_fill, per_result, busiest;     // us; per_result: of 10^6 results; busiest: weight against the mean
};
static const StreamCost kStreamSingle[4] = {{1.42, 1.590, 5.39, 11.7, 0.803, 1.00}, {3.04, 0.904, 3.60, 4.40, 0.752, 1.00},
                                            {3.20, 0.609, 1.94, 1.95, 0.718, 1.00}, {1.54, 0.677, 1.03, 2.33, 0.591, 0.80}};
static const StreamCost kStreamPair[4] = {{0.00, 1.520, 10.1, 19.8, 1.505, 1.00}, {3.06, 0.897, 6.46, 2.03, 1.351, 1.00},
                                          {4.26, 0.582, 4.19, 0.00, 0.128, 0.62}, {0.00, 0.638, 0.84, 5.04, 1.247, 1.00}};
constexpr int64_t kTileM[4] = {256, 128, 128, 128}, kTileN[4] = {256, 256, 128, 128};

// *extra: the late blocks' rounds.  Two blocks b and b + half of a compute unit take turns at its matrix cores: their loads add up.
static double stream_estimate(int variant, int products, const int64_t* m, const int64_t* n, const int64_t* k, int64_t cus, int64_t* extra) {
    const StreamCost& c = (products == 1 ? kStreamSingle : kStreamPair)[variant];
    int64_t tiles[2] = {0, 0};
    double cost[2] = {0.0, 1.0}, results = 0.0, sum = 0.0;
    for (int p = 0; p < products; ++p) {
        tiles[p] = ((m[p] + kTileM[variant] - 1) / kTileM[variant]) * ((n[p] + kTileN[variant] - 1) / kTileN[variant]);
        cost[p] = c.per_quad * (double)(k[p] > 256 ? (k[p] + 255) / 256 : 1) + c.per_tile;
        sum += (double)tiles[p] * cost[p];
        results += (double)m[p] * (double)n[p];
    }
    const int64_t total = tiles[0] + tiles[1], used = total < cus ? total : cus;
    const int64_t room = variant == kTwoPerCu ? 2 * cus : cus, blocks = total < room ? total : room, half = blocks / 2;
    PairLevel l = pair_level(tiles, cost, blocks);
    *extra = l.extra;
    // Where the second product cannot fill the rounds that would level the loads, the estimate does not count on extra ones: the constants, fitted
    // so, are low for launches that few long tiles dominate.  140 such layers, every shape timed: the one chosen costs 0.6 % more than the best
    // one on average, with the extra rounds counted 1.0 % (10848 x 288 x 544: 45.1 us in place of 35.8).
    if ((int64_t)(cost[0] / cost[1]) - 1 > pair_most_extra(tiles, blocks)) l = pair_loads(tiles, cost, blocks, 0);
    double busiest = l.busiest();
    if (variant == kTwoPerCu) {
        // a tile per compute unit: the deeper ring of one block; products narrower than a tile: not measured
        if (total <= cus || n[0] < 128 || (products == 2 && n[1] < 128)) return 1e30;
        const double mixed = l.early_load + l.late_load;
        busiest = l.early == 0 ? 2.0 * l.late_load : l.early > half ? 2.0 * l.early_load : 0.0;
        if (l.early > 0 && mixed > busiest) busiest = mixed;
        if (l.early > 0 && l.early < half && 2.0 * l.late_load > busiest) busiest = 2.0 * l.late_load;
    }
    const double mean = sum / (double)used, weight = busiest > 4.0 * mean ? 1.0 : c.busiest;     // (a few long tiles alone: theirs is the time)
    const double work = weight * busiest + (1.0 - weight) * mean + c.per_fill * (double)used / (double)cus;
    const double memory = c.per_result * 1e-6 * results;
    return c.start + (work > memory ? work : memory);
}

// the variant for one product or a pair, and its estimated time
static int pick_variant(int products, const int64_t* m, const int64_t* n, const int64_t* k, int cus, double* estimate) {
    int variant = -1;
    for (int v = 0; v < 4; ++v) {
        if (g_forced_variant >= 0 && g_forced_variant != v) continue;
        int64_t extra;
        const double t = stream_estimate(v, products, m, n, k, cus, &extra);
        if (variant < 0 || t < *estimate) { *estimate = t; variant = v; }
    }
    return variant;
}

// Problems that the split kernels (gemm_split_kernels.hip) finish sooner: few rows, small layers, long inner dimensions with few
// tiles.  Compares their estimate with that of the streaming kernels, in favour of the latter by 12 % (one product, two waves) or
// 35 % (two products; four waves, whose estimate is low for 64 x 64 tiles), which cost least over the calls the estimates were fitted to.  Measured, streaming against split (us): 630 x 1312 x 2944 11.7 / 7.0;
// 2910 x 384 x 1056 7.6 / 7.2; 469 x 1792 x 1728 8.3 / 6.5; on the other side 2538 x 864 x 384 8.1 / 10.2; four waves 339 x 2624 x 5600 15.5 / 9.2 and
// 377 x 4096 x 3936 12.8 / 13.9, 950 x 1696 x 5664 16.5 / 18.1; pairs of layers 736 x 928 x 800 10.5 / 8.2, 2176 x 1024 x 864 11.8 / 14.7.  For
// one product the choice depends on m, n and k alone, so fused and plain products of one size run on the same side.
static bool use_split(int products, const int64_t* m, const int64_t* n, const int64_t* k, int cus, double streaming, int* shape) {
    if (g_forced_variant >= 0) return false;
    // A block per tile, and a launch has fewer than 2^32 threads: with 32 x 32 tiles of up to four waves, 2^24 tiles at most
    int64_t tiles = 0;
    for (int p = 0; p < products; ++p) tiles += ((m[p] + 31) / 32) * ((n[p] + 31) / 32);
    if (tiles >= ((int64_t)1 << 24)) return false;
    const bool four = split_waves(products == 2 && k[1] > k[0] ? k[1] : k[0]) == 4;
    return best_split_shape(products, m, n, k, cus, shape) < (four || products == 2 ? 0.65 : 0.88) * streaming;
}

// The kernel for one product or a pair, plain (nb = 0) or with the gradient epilogue of Hadamard blocks of nb groups.
struct GemmPlan {
    bool split;
    int shape;          // split: tile shape (see launch_gemm_split); otherwise the streaming variant
};
static GemmPlan plan_gemm(int products, const int64_t* m, const int64_t* n, const int64_t* k, uint32_t nb, int cus) {
    double estimate = 0.0;
    int shape = 0, variant = pick_variant(products, m, n, k, cus, &estimate);
    if (nb >= 4u && variant >= 2) {
        // A block of 128 columns needs the 128-column wave tile.  (256 x 256 where the estimates put it before 128 x 256 is not sooner: 40 layers
        // each with blocks of 128 and 256, 1.00 and 0.98 of its speed on average.)
        variant = 1;
        // In a pair the split kernels are weighed against the tiles that run; against those that cannot, backward passes of layers with blocks
        // of 128 took (tokens, in, out; us) 384 x 3456 x 256 21.6 for 13.9, 6016 x 384 x 640 40.2 for 26.5, 1280 x 640 x 2560 30.0 for 22.8.  One
        // product stays on the side where the plain product of its sizes runs: their results are the same bits.
        int64_t extra;
        if (products == 2) estimate = stream_estimate(1, 2, m, n, k, cus, &extra);
    }
    if (nb != 8u && use_split(products, m, n, k, cus, estimate, &shape)) return {true, split_shape_for(shape, nb)};
    return {false, variant};
}

int gemm_plan_code(int products, const int64_t* m, const int64_t* n, const int64_t* k, uint32_t nb, int cus) {
    const GemmPlan plan = plan_gemm(products, m, n, k, nb, cus);
    const int64_t k_max = products == 2 && k[1] > k[0] ? k[1] : k[0];
    return plan.split ? 100 * split_waves(k_max) + plan.shape : plan.shape == kTwoPerCu ? kTwoPerCuCode : plan.shape;
}

hipError_t launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* b_codes,
                       const uint8_t* b_scales, int64_t m, int64_t n, int64_t k, float alpha, void* d,
                       int d_bf16, int64_t ldd, int fused, const uint32_t* mask, uint32_t nb, hipStream_t st) {
    if (m == 0 || n == 0) return hipSuccess;
    const GemmPlan plan = plan_gemm(1, &m, &n, &k, fused ? nb : 0u, stream_blocks());
    if (plan.split) {
        const GemmArgs g = {a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask};
        return launch_gemm_split(g, nullptr, d_bf16, fused, nb, plan.shape, st);
    }
    const int variant = plan.shape;
#define QUARTET_DISPATCH(FN, ...)                                                                     \
    do {                                                                                              \
        if (d_bf16) { if (fused) FN<__VA_ARGS__ true, true>(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, nb, st); \
                      else FN<__VA_ARGS__ true, false>(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, nb, st); }   \
        else { if (fused) FN<__VA_ARGS__ false, true>(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, nb, st);      \
               else FN<__VA_ARGS__ false, false>(a_codes, a_scales, b_codes, b_scales, m, n, k, alpha, d, ldd, mask, nb, st); }         \
    } while (0)
    if (variant == 1) QUARTET_DISPATCH(launch_stream_tile_t, 2, 4, 1, );
    else if (variant == 2) QUARTET_DISPATCH(launch_stream_tile_t, 2, 2, 1, );
    else if (variant == kTwoPerCu) QUARTET_DISPATCH(launch_stream_tile_t, 2, 2, 2, );
    else QUARTET_DISPATCH(launch_stream_t, );
#undef QUARTET_DISPATCH
    return hipGetLastError();
}

// Hadamard blocks of 256 columns: the kernels that apply their epilogue take whole tiles of 256 x 256 (hence of 128 x 256) only, which is
// what every layer with such blocks has, and results and masks aligned as the C entry requires them (a guard: nothing else comes here).  Against two products on the kernels that are soonest for them, fp32 results in the
// workspace and two epilogue kernels, layer steps (tokens, in, out; us): 256 x 1024 x 512 32.5 -> 24.5, 1024 x 768 x 1280 48 -> 34, 4096 x 4096 x
// 2048 145 -> 112, 8192 x 2048 x 5632 288 -> 268, 1024 x 10752 x 7936 496 -> 330, 14336 x 1792 x 7680 541 -> 499.
static bool wide_fits(const GemmArgs& g, int d_bf16) {
    return g.m % 256 == 0 && g.n % 256 == 0 && g.ldd % 4 == 0 && g.mask != nullptr && (reinterpret_cast<uintptr_t>(g.d) & (d_bf16 ? 7u : 15u)) == 0;
}
static void launch_wide(const GemmBatch& batch, bool large, int d_bf16, hipStream_t st) {
    const uint32_t total = batch.p[0].total_tiles + batch.p[1].total_tiles, cus = (uint32_t)stream_blocks();
    const dim3 grid(total < cus ? total : cus), block(256);
    if (large && d_bf16 && batch.past) hipLaunchKernelGGL(gemm_mxfp4_past_wide_kernel, grid, block, 0, st, batch, g_clock_counters);
    else if (large && d_bf16) hipLaunchKernelGGL((gemm_mxfp4_wide_kernel<true>), grid, block, 0, st, batch, g_clock_counters);
    else if (large) hipLaunchKernelGGL((gemm_mxfp4_wide_kernel<false>), grid, block, 0, st, batch, g_clock_counters);
    else if (d_bf16) hipLaunchKernelGGL((gemm_mxfp4_wide_tile_kernel<true>), grid, block, 0, st, batch, g_clock_counters);
    else hipLaunchKernelGGL((gemm_mxfp4_wide_tile_kernel<false>), grid, block, 0, st, batch, g_clock_counters);
}

// Two gradient products in one launch (both with the fused epilogue, results of one type).  One tile shape serves both.  Hadamard
// blocks of 256 columns (nb = 8): hipErrorNotSupported, and nothing is launched, for what those kernels do not take; the caller sees to it that
// there is no empty product.
hipError_t launch_gemm_grad_pair(const GemmArgs& g0, const GemmArgs& g1, int d_bf16, uint32_t nb, hipStream_t st) {
    const bool empty0 = g0.m == 0 || g0.n == 0, empty1 = g1.m == 0 || g1.n == 0;
    if (nb == 8u && (empty0 || empty1)) return hipErrorNotSupported;
    if (empty0 || empty1) {
        hipError_t e = launch_gemm(g0.a_codes, g0.a_scales, g0.b_codes, g0.b_scales, g0.m, g0.n, g0.k, g0.alpha, g0.d, d_bf16, g0.ldd,
                                   1, g0.mask, nb, st);
        if (e != hipSuccess) return e;
        return launch_gemm(g1.a_codes, g1.a_scales, g1.b_codes, g1.b_scales, g1.m, g1.n, g1.k, g1.alpha, g1.d, d_bf16, g1.ldd, 1,
                           g1.mask, nb, st);
    }
    const int64_t ms[2] = {g0.m, g1.m}, ns[2] = {g0.n, g1.n}, ks[2] = {g0.k, g1.k};
    const GemmPlan plan = plan_gemm(2, ms, ns, ks, nb, stream_blocks());
    if (nb == 8u && !(wide_fits(g0, d_bf16) && wide_fits(g1, d_bf16))) return hipErrorNotSupported;
    if (plan.split) return launch_gemm_split(g0, &g1, d_bf16, 1, nb, plan.shape, st);
    const int variant = plan.shape;
    GemmBatch batch;
    batch.p[0] = make_problem(g0.a_codes, g0.a_scales, g0.b_codes, g0.b_scales, g0.m, g0.n, g0.k, g0.alpha, g0.d, g0.ldd, g0.mask,
                              kTileM[variant], kTileN[variant]);
    batch.p[1] = make_problem(g1.a_codes, g1.a_scales, g1.b_codes, g1.b_scales, g1.m, g1.n, g1.k, g1.alpha, g1.d, g1.ldd, g1.mask,
                              kTileM[variant], kTileN[variant]);
    const int64_t cus = stream_blocks();
    const uint32_t total = batch.p[0].total_tiles + batch.p[1].total_tiles, room = (uint32_t)(variant == kTwoPerCu ? 2 * cus : cus), blocks = total < room ? total : room;
    int64_t extra;
    stream_estimate(variant, 2, ms, ns, ks, cus, &extra);
    batch.past = stored_past(batch, d_bf16 != 0);
    batch.late = blocks - batch.p[0].total_tiles % blocks;
    batch.extra_tiles = (uint32_t)extra * batch.late;
#define QUARTET_PAIR(FN, ...)                                                                           \
    do { if (d_bf16) FN<__VA_ARGS__ true, true>(batch, nb, st); else FN<__VA_ARGS__ false, true>(batch, nb, st); } while (0)
    if (nb == 8u) launch_wide(batch, variant == 0, d_bf16, st);
    else if (variant == 1) QUARTET_PAIR(launch_stream_tile_batch_t, 2, 4, 1, );
    else if (variant == 2) QUARTET_PAIR(launch_stream_tile_batch_t, 2, 2, 1, );
    else if (variant == kTwoPerCu) QUARTET_PAIR(launch_stream_tile_batch_t, 2, 2, 2, );
    else QUARTET_PAIR(launch_stream_batch_t, );
#undef QUARTET_PAIR
    return hipGetLastError();
}

}  // namespace quartet
