// MXFP4 x MXFP4 -> fp32 GEMM for problems that do not fill the chip with the streaming kernels' tiles: few rows (serving), small
// layers.  Same operands, epilogues and results as gemm_kernels.hip.
//
// What bounds these problems is latency, not matrix-core or memory rate: a 128 x 128 tile of the streaming kernel walks the whole
// inner dimension in one block, stage after stage through its LDS ring, while most compute units have no tile.  Here a block of
// NW waves owns one small tile and its waves share the inner dimension: wave w takes the K-quads (256 elements) w, w + NW, ...,
// through an LDS ring of its own (two quads of LDS-direct loads, whole 128-byte lines; no barrier in the loop), and the partial
// sums meet in LDS.  The order of a result's sum depends on k and the number of waves alone, not on the tile shape, and the number of
// waves on k (of a pair on the larger k), so fused and plain products give the same bits.
#include "gemm_common.h"
#include "launchers.h"

namespace quartet {

struct SplitProblem {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* b_codes;
    const uint8_t* b_scales;
    void* d;
    const uint32_t* mask;
    uint32_t m, n, k, ldd;
    float alpha;
    uint32_t tiles_m, total_tiles;
    FastDiv by_tiles_m;
};
struct SplitBatch {
    SplitProblem p[2];
};

// 4 bytes per lane to LDS byte address lds_base + 4 * lane (see lds_direct_load16)
__device__ __forceinline__ void lds_direct_load4(v4i_t rsrc, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_base), "v"(voff), "s"(rsrc) : "memory");
}

// The last part of the epilogue: chunk c (4 columns) of all TN 32-column slices of result row grow, held in vv by one of the eight
// lanes of that row (lane i of the eight: c = i ^ (i & 4 ? 3 : 0)), the mask already applied.  With FUSED the gradient epilogue
// (the steps of store_tile_rows8; as a function shared with it this cost the streaming kernels 30 spilled scalar registers and
// 4 % of a fused product's time), then the scale and the store.
template <int TN, bool OUT_BF16, bool FUSED>
__device__ __forceinline__ void finish_row_chunk(float (&vv)[TN][4], void* d, uint32_t ldd, float alpha, uint32_t grow,
                                                 uint32_t col_base, uint32_t m, uint32_t n, uint32_t c, uint32_t nb) {
    const float up4 = (c & 1u) ? -1.0f : 1.0f, up8 = (c & 2u) ? -1.0f : 1.0f, up16 = (c & 4u) ? -1.0f : 1.0f;
    const float norm = ((c ^ (c >> 1) ^ (c >> 2)) & 1u) ? -block_norm(nb) : block_norm(nb);
    const bool wide = (ldd & 3u) == 0u;
    if (FUSED && nb >= 2u) {
#pragma unroll
        for (uint32_t j = 0; j + 1u < TN; j += 2)
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const float a = vv[j][e], b = vv[j + 1][e];
                vv[j][e] = a + b;
                vv[j + 1][e] = a - b;
            }
    }
    if (FUSED && nb >= 4u && TN >= 4) {
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j)
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const float a = vv[j][e], b = vv[(j + 2u) % TN][e];
                vv[j][e] = a + b;
                vv[(j + 2u) % TN][e] = a - b;
            }
    }
#pragma unroll
    for (uint32_t j = 0; j < TN; ++j) {
        const uint32_t gcol = col_base + j * 32u;
        float v0 = vv[j][0], v1 = vv[j][1], v2 = vv[j][2], v3 = vv[j][3];
        if (FUSED) {
            const float a0 = v0 + v1, a1 = v0 - v1, a2 = v2 + v3, a3 = v2 - v3;
            v0 = a0 + a2; v2 = a0 - a2; v1 = a1 + a3; v3 = a1 - a3;
            QUARTET_BUTTERFLIES_ACROSS(v0, v1, v2, v3, up4, up8, up16);
            v0 = epilogue_norm(v0, norm); v1 = epilogue_norm(v1, norm); v2 = epilogue_norm(v2, norm); v3 = epilogue_norm(v3, norm);
        }
        v0 = v0 * alpha; v1 = v1 * alpha; v2 = v2 * alpha; v3 = v3 * alpha;
        if (grow >= m) continue;
        const uint32_t col = gcol + 4u * c;
        const size_t at = (size_t)grow * ldd + col;
        if (OUT_BF16) {
            uint16_t* dst = static_cast<uint16_t*>(d) + at;
            const uint32_t h0 = f32_to_bf16_rne(v0), h1 = f32_to_bf16_rne(v1), h2 = f32_to_bf16_rne(v2), h3 = f32_to_bf16_rne(v3);
            if (wide && col + 4u <= n) {
                *reinterpret_cast<uint2*>(dst) = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
            } else {
                if (col < n) dst[0] = (uint16_t)h0;
                if (col + 1u < n) dst[1] = (uint16_t)h1;
                if (col + 2u < n) dst[2] = (uint16_t)h2;
                if (col + 3u < n) dst[3] = (uint16_t)h3;
            }
        } else {
            float* dst = static_cast<float*>(d) + at;
            if (wide && col + 4u <= n) {
                *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
            } else {
                if (col < n) dst[0] = v0;
                if (col + 1u < n) dst[1] = v1;
                if (col + 2u < n) dst[2] = v2;
                if (col + 3u < n) dst[3] = v3;
            }
        }
    }
}

template <int TM, int TN, int NW, bool OUT_BF16, bool FUSED>
__global__ void __launch_bounds__(64 * NW)
gemm_mxfp4_split_kernel(SplitBatch batch, uint32_t nb) {
    constexpr uint32_t BM = 32 * TM, BN = 32 * TN, T = TM + TN;
    // a ring slot: T row blocks of 32 rows x 128 bytes (16-byte chunk c of row r at position c ^ (r / 2) % 8: the 16 lanes of a
    // fragment read fall on different banks), then their T scale tiles of 256 bytes
    constexpr uint32_t SLOT = T * (4096u + 256u), LOADS = T * 5u;
    constexpr uint32_t D = TN < 4 ? 2u : 1u;           // slots per wave (four column blocks: what fits)
    constexpr uint32_t RING = D * SLOT * NW, PART = BM * BN * 4u * NW;
    __shared__ __align__(16) uint8_t lds[RING > PART ? RING : PART];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lrow = lane & 31u, lhalf = lane >> 5;
    // consecutive tiles of one XCD share their columns of B (blocks go to the XCDs in turn)
    const bool second = blockIdx.x >= batch.p[0].total_tiles;
    // Field by field: all arguments are on their way at once, then one product's are picked.  By index three scalar loads waited for each
    // other, and a division, before the first operand load.  With that out (us): 24 x 4096 x 11008 quantized and multiplied 10.38 -> 10.19, a
    // 256 x 512 x 512 layer step, with the same in the row quantizers' paired launch, 15.93 -> 15.47.
#define PICK(F) (second ? batch.p[1].F : batch.p[0].F)
    const SplitProblem q = {PICK(a_codes), PICK(a_scales), PICK(b_codes), PICK(b_scales), PICK(d), PICK(mask), PICK(m), PICK(n), PICK(k), PICK(ldd),
                            PICK(alpha), PICK(tiles_m), PICK(total_tiles), {PICK(by_tiles_m.mul), PICK(by_tiles_m.shift)}};
#undef PICK
    const uint32_t v = second ? blockIdx.x - batch.p[0].total_tiles : blockIdx.x;
    const uint32_t per = q.total_tiles >> 3, rem = q.total_tiles & 7u, xcd = v & 7u;
    const uint32_t tile = xcd * per + (xcd < rem ? xcd : rem) + (v >> 3);
    const uint32_t tile_n = fast_div(tile, q.by_tiles_m), m0 = (tile - tile_n * q.tiles_m) * BM, n0 = tile_n * BN;
    const uint32_t m = q.m, n = q.n, kb = q.k >> 1, gk = q.k >> 5, kq = (q.k + 255u) >> 8;

    // rows past the matrix read as zeros; chunks past k inside a row are cut off per lane
    const uint32_t rows_a = (m - m0) < BM ? (m - m0) : BM, rows_b = (n - n0) < BN ? (n - n0) : BN;
    const v4i_t res_a = make_rsrc_words(q.a_codes + (size_t)m0 * kb, rows_a * kb), res_b = make_rsrc_words(q.b_codes + (size_t)n0 * kb, rows_b * kb);
    const v4i_t res_sa = make_rsrc_words(q.a_scales + (size_t)(m0 >> 5) * kq * 256u, ((rows_a + 31u) >> 5) * kq * 256u);
    const v4i_t res_sb = make_rsrc_words(q.b_scales + (size_t)(n0 >> 5) * kq * 256u, ((rows_b + 31u) >> 5) * kq * 256u);
    const uint32_t ring = (uint32_t)(size_t)(lds_ptr_t)lds + wave * D * SLOT;
    // a load instruction covers 8 rows; the rows 8 i + lane / 8 of a row block differ in (row / 2) % 8 by 4 i
    const uint32_t srow = lane >> 3, c0 = (lane & 7u) ^ (srow >> 1);
    auto issue = [&](uint32_t quad, uint32_t slot) {
        const uint32_t to = ring + slot * SLOT;
        const bool quad_in = quad < kq;                // wave-uniform
#pragma unroll
        for (uint32_t t = 0; t < T; ++t) {
            const v4i_t& res = t < TM ? res_a : res_b;
            const uint32_t rb = t < TM ? t : t - TM;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t at = quad * 128u + (c0 ^ (4u * (i & 1u))) * 16u;
                lds_direct_load16(res, at < kb ? (rb * 32u + i * 8u + srow) * kb + at : kOutOfRange, to + t * 4096u + i * 1024u);
            }
            lds_direct_load4(t < TM ? res_sa : res_sb, quad_in ? (rb * kq + quad) * 256u + lane * 4u : kOutOfRange, to + T * 4096u + t * 256u);
        }
    };
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    issue(wave, 0u);
    if (D == 2u) issue(wave + NW, 1u);
    uint32_t slot = 0u;
    for (uint32_t quad = wave; quad < kq; quad += NW, slot = D - 1u - slot) {
        constexpr uint32_t KEEP = (D - 1u) * LOADS, WAIT = 0x0F70u | (KEEP & 15u) | ((KEEP >> 4) << 14);   // the next quad's loads stay in flight
        __builtin_amdgcn_s_waitcnt(WAIT);
        const uint8_t* from = lds + (wave * D + slot) * SLOT;
        uint4 f[T][4];
        uint32_t sc[T];
#pragma unroll
        for (uint32_t t = 0; t < T; ++t) {
            sc[t] = *reinterpret_cast<const uint32_t*>(from + T * 4096u + t * 256u + lane * 4u);
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s)
                f[t][s] = *reinterpret_cast<const uint4*>(from + t * 4096u + lrow * 128u + (((2u * s + lhalf) ^ (lrow >> 1)) & 7u) * 16u);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the slot's contents are in registers
        issue(quad + D * NW, slot);                   // past the last quad: out of range (zeros)
        if (quad * 8u + 8u > gk) {                     // wave-uniform: scale bytes of groups past k become 2^0 (their codes are zero)
            const uint32_t steps = (gk + 1u - lhalf) >> 1, done = quad * 4u;
            const uint32_t nv = steps > done ? (steps - done < 4u ? steps - done : 4u) : 0u;
            const uint32_t keep = nv >= 4u ? 0xFFFFFFFFu : ((1u << (8u * nv)) - 1u);
#pragma unroll
            for (uint32_t t = 0; t < T; ++t) sc[t] = (sc[t] & keep) | (0x7F7F7F7Fu & ~keep);
        }
#define SPLIT_STEP(S)                                                                                   \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                      \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                                  \
            acc[i][j] = mfma_fp4_32<S>(f[i][S], f[TM + j][S], acc[i][j], sc[i], sc[TM + j]);
        SPLIT_STEP(0) SPLIT_STEP(1) SPLIT_STEP(2) SPLIT_STEP(3)
#undef SPLIT_STEP
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                // the zero-filled quads past the end have landed: the ring can be reused
    __syncthreads();

    // partial sums: row r of the tile at r * BN floats
    float* part = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (uint32_t r = 0; r < 16; ++r)
                part[wave * BM * BN + ((uint32_t)i * 32u + (r >> 2) * 8u + lhalf * 4u + (r & 3u)) * BN + (uint32_t)j * 32u + lrow] = acc[i][j][r];
    __syncthreads();
    // eight lanes per row, each with one 4-column chunk of all slices of the row
    const uint32_t c = (tid & 7u) ^ ((tid & 4u) ? 3u : 0u);
#pragma unroll
    for (uint32_t row = tid >> 3; row < BM; row += 8u * NW) {   // wave-uniform: a wave's eight rows are all inside or all outside
        const uint32_t grow = m0 + row;
        float vv[TN][4];
#pragma unroll
        for (uint32_t j = 0; j < TN; ++j) {
            float4 t[NW];
#pragma unroll
            for (uint32_t w = 0; w < NW; ++w) t[w] = *reinterpret_cast<const float4*>(&part[w * BM * BN + row * BN + j * 32u + 4u * c]);
#pragma unroll
            for (uint32_t w = 1; w < NW; ++w) { t[0].x += t[w].x; t[0].y += t[w].y; t[0].z += t[w].z; t[0].w += t[w].w; }
            vv[j][0] = t[0].x; vv[j][1] = t[0].y; vv[j][2] = t[0].z; vv[j][3] = t[0].w;
            if (FUSED) {
                const uint32_t gcol = n0 + j * 32u;
                const uint32_t mw = (q.mask && grow < m && gcol < n) ? q.mask[(size_t)grow * (n >> 5) + (gcol >> 5)] : 0xFFFFFFFFu;
                const int32_t bits = (int32_t)(mw >> (4u * c));
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) vv[j][e] = u2f(f2u(vv[j][e]) & (uint32_t)((bits << (31 - (int)e)) >> 31));
            }
        }
        finish_row_chunk<TN, OUT_BF16, FUSED>(vv, q.d, q.ldd, q.alpha, grow, n0, m, n, c, nb);
    }
}

static SplitProblem split_problem(const GemmArgs& g, uint32_t bm, uint32_t bn) {
    SplitProblem q;
    q.a_codes = g.a_codes; q.a_scales = g.a_scales; q.b_codes = g.b_codes; q.b_scales = g.b_scales;
    q.d = g.d; q.mask = g.mask;
    q.m = (uint32_t)g.m; q.n = (uint32_t)g.n; q.k = (uint32_t)g.k; q.ldd = (uint32_t)g.ldd;
    q.alpha = g.alpha;
    q.tiles_m = (q.m + bm - 1u) / bm;
    q.total_tiles = q.tiles_m * ((q.n + bn - 1u) / bn);
    q.by_tiles_m = make_fast_div(q.tiles_m);
    return q;
}

template <int TM, int TN, int NW>
static void launch_split(const GemmArgs& g0, const GemmArgs* g1, int d_bf16, int fused, uint32_t nb, hipStream_t st) {
    SplitBatch batch;
    batch.p[0] = split_problem(g0, 32 * TM, 32 * TN);
    batch.p[1] = g1 ? split_problem(*g1, 32 * TM, 32 * TN) : SplitProblem{};
    const dim3 grid(batch.p[0].total_tiles + batch.p[1].total_tiles), block(64 * NW);
    if (d_bf16) {
        if (fused) hipLaunchKernelGGL((gemm_mxfp4_split_kernel<TM, TN, NW, true, true>), grid, block, 0, st, batch, nb);
        else hipLaunchKernelGGL((gemm_mxfp4_split_kernel<TM, TN, NW, true, false>), grid, block, 0, st, batch, nb);
    } else {
        if (fused) hipLaunchKernelGGL((gemm_mxfp4_split_kernel<TM, TN, NW, false, true>), grid, block, 0, st, batch, nb);
        else hipLaunchKernelGGL((gemm_mxfp4_split_kernel<TM, TN, NW, false, false>), grid, block, 0, st, batch, nb);
    }
}

// Estimated time in us of a launch that works through the given products on tiles of (32 TM) x (32 TN) with NW waves: launch and
// first loads, the serial quads of a wave, and per tile a compute unit holds (at least one) a fixed part and the quads' trip
// through its LDS.  Fitted to 120 shapes, m 1 .. 4096, n and k 256 .. 11008 (rms error 10 %).
struct SplitShape {
    int id;
    int64_t bm, bn;
    double start, per_step, per_tile, per_tile_quad;
};
static const SplitShape kSplitShapes2[3] = {   // two waves
    {11, 32, 32, 2.67, 0.066, 0.45, 0.101}, {12, 32, 64, 2.74, 0.050, 0.79, 0.170}, {22, 64, 64, 2.25, 0.089, 1.79, 0.229}};
static const SplitShape kSplitShapes4[3] = {   // four waves
    {11, 32, 32, 2.46, 0.0, 0.92, 0.092}, {12, 32, 64, 1.49, 0.0, 2.42, 0.142}, {22, 64, 64, 0.93, 0.0, 3.73, 0.204}};
// Waves that share k.  Four from here on: with a tile per compute unit or less they are sooner (two / four waves, us: 24 x 4096 x 11008 8.1 / 5.7,
// 200 x 4096 x 4096 8.2 / 7.4; below the line 24 x 4096 x 2816 5.2 / 5.2).  With more tiles than compute units two waves would still be
// (24 x 11008 x 4096 5.5 / 5.5, x 8192 10.1 / 10.7; 64 x 11008 x 4096 7.5 / 9.0): the rule does not look at the number of tiles.
constexpr int64_t kFourWaveQuads = 12;

int split_waves(int64_t k) { return (k + 255) / 256 >= kFourWaveQuads ? 4 : 2; }

// a wave's lanes must hold whole Hadamard blocks: 64 columns need two column blocks per tile, 128 need four
int split_shape_for(int shape, uint32_t nb) { return nb == 4u ? 14 : nb == 2u && shape == 11 ? 12 : shape; }

double best_split_shape(int products, const int64_t* m, const int64_t* n, const int64_t* k, int compute_units, int* shape) {
    int64_t quads = 0;
    for (int p = 0; p < products; ++p) quads = quads > (k[p] + 255) / 256 ? quads : (k[p] + 255) / 256;
    const bool four = split_waves(256 * quads) == 4;
    double best = -1.0;
    for (const SplitShape& s : four ? kSplitShapes4 : kSplitShapes2) {
        double t = s.start + s.per_step * (double)((quads + (four ? 3 : 1)) / (four ? 4 : 2)), tiles_all = 0.0, load = 0.0;
        for (int p = 0; p < products; ++p) {
            const double tiles = (double)((m[p] + s.bm - 1) / s.bm) * (double)((n[p] + s.bn - 1) / s.bn) / (double)compute_units;
            tiles_all += tiles;
            load += tiles * (s.per_tile + s.per_tile_quad * (double)((k[p] + 255) / 256));
        }
        t += tiles_all >= 1.0 ? load : load / tiles_all;
        if (best < 0.0 || t < best) { best = t; *shape = s.id; }
    }
    return best;
}

hipError_t launch_gemm_split(const GemmArgs& g0, const GemmArgs* g1, int d_bf16, int fused, uint32_t nb, int shape, hipStream_t st) {
    const int64_t k = g1 && g1->k > g0.k ? g1->k : g0.k;
#define QUARTET_SPLIT(NW)                                                                               \
    switch (shape) {                                                                                    \
    case 11: launch_split<1, 1, NW>(g0, g1, d_bf16, fused, nb, st); break;                              \
    case 12: launch_split<1, 2, NW>(g0, g1, d_bf16, fused, nb, st); break;                              \
    case 14: launch_split<1, 4, NW>(g0, g1, d_bf16, fused, nb, st); break;                              \
    default: launch_split<2, 2, NW>(g0, g1, d_bf16, fused, nb, st); break;                              \
    }
    if (split_waves(k) == 4) QUARTET_SPLIT(4)
    else QUARTET_SPLIT(2)
#undef QUARTET_SPLIT
    return hipGetLastError();
}

}  // namespace quartet
