// Pieces shared by the matrix-core GEMM kernels: buffer resources, LDS-direct loads and the epilogue
// that takes a wave's accumulator tile through LDS to full-line stores.
#pragma once
#include "device_common.h"

namespace quartet {

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = f2u(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Raw buffer resource over [base, base + bytes): loads past the end return zero, which is how ragged
// tile edges are handled without per-load predicates.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

constexpr uint32_t kOutOfRange = 0x80000000u;   // byte offset no resource here reaches

typedef int v4i_t __attribute__((ext_vector_type(4)));

// acc += A B^T with the operands' scales in byte 0 (STEP = 0) or byte 2 (STEP = 1) of sa and sb.  Written out so that the accumulator
// stays where it is (the builtin's result is not tied to its input, and the register allocator then moves 16 x 16 accumulators
// between both register files in the loop).  The compiler does not see a matrix-core instruction in this and keeps no wait states around it: the code that
// writes an operand or reads an accumulator with vector instructions does (the three functions below; a test looks through the
// built kernels).  LDS reads that fill fragments are waited for as everywhere.
template <int STEP>
__device__ __forceinline__ void mfma_fp4(const v4i_t& a, const v4i_t& b, v4f& acc, uint32_t sa, uint32_t sb) {
    if (STEP == 0)
        asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                     : "+a"(acc) : "v"(a), "v"(b), "v"(sa), "v"(sb));
    else
        asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel:[0,0,0] op_sel_hi:[1,1,0] cbsz:4 blgp:4"
                     : "+a"(acc) : "v"(a), "v"(b), "v"(sa), "v"(sb));
}
// Two wait states between a vector instruction's result and a matrix-core instruction that reads it.  The empty statements make
// every scale one that is needed in their place: the instructions that form it stand before the s_nop and cannot be sunk behind it.
template <int M, int N>
__device__ __forceinline__ void mfma_scales_written(uint32_t (&sa)[M], uint32_t (&sb)[N]) {
#pragma unroll
    for (int i = 0; i < M; ++i) asm volatile("" : "+v"(sa[i]));
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+v"(sb[j]));
    asm volatile("s_nop 1" ::: "memory");
}
// All accumulators to 0, register by register: these instructions keep their place, the compiler's own are repeated or sunk to right
// before the first use.
template <int M, int N>
__device__ __forceinline__ void mfma_clear_accumulators(v4f (&acc)[M][N]) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) { float z; asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(z)); acc[i][j][r] = z; }
    asm volatile("s_nop 1" ::: "memory");
}
// the last matrix-core instruction (eight passes at most) has written its accumulator
__device__ __forceinline__ void mfma_results_written() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// c + A B^T of 32 x 32 x 64 (FP4), scales in byte S of sa and sb; the compiler keeps the wait states
template <int S>
__device__ __forceinline__ v16f mfma_fp4_32(const uint4& a, const uint4& b, v16f c, uint32_t sa, uint32_t sb) {
    const v8i va = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const v8i vb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vb, c, 4, 4, S, (int)sa, S, (int)sb);
}

// Plain epilogue of a kernel whose ring is free when it ends (the MXFP8 twin): the wave's accumulator tile goes through
// LDS one 32-column slice at a time and comes back with 8 consecutive lanes holding the 32 columns of one row (4 each):
// a store instruction then writes 8 whole 128-byte lines.  wbuf: this wave's LDS scratch of TM*32 rows x kEpiStride floats.
constexpr uint32_t kEpiStride = 32;   // floats per LDS row, no padding: the LDS has 64 banks and serves a 16-byte read 16 lanes (two rows here) at a time, so neighbouring rows must sit 32 banks apart (counters: every read took twice its cycles with rows of 36 or 40 floats)

template <int TM, int TN, bool OUT_BF16>
__device__ __forceinline__ void store_tile(v16f (&acc)[TM][TN], float* wbuf, void* d, uint32_t ldd, float alpha,
                                           uint32_t row_base, uint32_t col_base, uint32_t m, uint32_t n, uint32_t lane) {
    constexpr uint32_t ITERS = TM * 4;   // 8 rows per pass
    const uint32_t lrow = lane & 31u, lhalf = lane >> 5;
    const uint32_t sub = lane >> 3, c = lane & 7u;
    const bool wide = (ldd & 3u) == 0u;   // every 4-column chunk starts 16-byte (fp32) / 8-byte (bf16) aligned
#pragma unroll
    for (uint32_t j = 0; j < TN; ++j) {
        const uint32_t gcol = col_base + j * 32u;
#pragma unroll
        for (uint32_t i = 0; i < TM; ++i)
#pragma unroll
            for (uint32_t r = 0; r < 16; ++r)
                wbuf[(i * 32u + (r >> 2) * 8u + lhalf * 4u + (r & 3u)) * kEpiStride + lrow] = acc[i][j][r];
        float4 slice[ITERS];   // all reads in flight before the first use: one wave per SIMD hides no LDS latency
#pragma unroll
        for (uint32_t it = 0; it < ITERS; ++it)
            slice[it] = *reinterpret_cast<const float4*>(&wbuf[(it * 8u + sub) * kEpiStride + 4u * c]);
#pragma unroll
        for (uint32_t it = 0; it < ITERS; ++it) {
            const uint32_t grow = row_base + it * 8u + sub;
            const float v0 = slice[it].x * alpha, v1 = slice[it].y * alpha, v2 = slice[it].z * alpha, v3 = slice[it].w * alpha;
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
}

// One butterfly stage between a lane and its DPP partner for the four values of a chunk, one instruction per value: both
// lanes form partner * t + own (t = +-1, so the fused multiply-add rounds exactly like the addition): t = +1 in the lower
// lane gives a + b, t = -1 in the upper lane gives -(a - b).  A lane's values therefore carry the sign (-1)^(number of
// stages in which it was the upper one); the partners of every stage have been upper equally often before it, so the signs
// cancel inside each stage, and the normalization constant takes the final sign back (epilogue_norm).  Rounding is symmetric
// in sign: the bits are those of a + b and a - b.
// The instruction is written out (the compiler keeps a separate lane move in front of a fused multiply-add).  A DPP
// operand must not be read in the two issue slots after a vector instruction wrote it: hence the s_nop in front, and the
// three stages of the four values in one block, where every value is read four instructions after it was written.
#define QUARTET_DPP_TAIL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define QUARTET_BUTTERFLY_STAGE(CTRL_TEXT, T)                           \
    "v_fmac_f32_dpp %0, %0, " T " " CTRL_TEXT QUARTET_DPP_TAIL            \
    "v_fmac_f32_dpp %1, %1, " T " " CTRL_TEXT QUARTET_DPP_TAIL            \
    "v_fmac_f32_dpp %2, %2, " T " " CTRL_TEXT QUARTET_DPP_TAIL            \
    "v_fmac_f32_dpp %3, %3, " T " " CTRL_TEXT QUARTET_DPP_TAIL
// strides 4, 8, 16 of a 32-column slice held as four values in each of eight lanes: partners lane ^ 1, lane ^ 2, 7 - lane.
// volatile: the block reads other lanes, so it must stay where all lanes of a row group are active (not be moved into the
// predicated store that uses its results).
#define QUARTET_BUTTERFLIES_ACROSS(v0, v1, v2, v3, t4, t8, t16)                        \
    asm volatile("s_nop 1\n\t"                                                              \
        QUARTET_BUTTERFLY_STAGE("quad_perm:[1,0,3,2]", "%4")                            \
        QUARTET_BUTTERFLY_STAGE("quad_perm:[2,3,0,1]", "%5")                            \
        QUARTET_BUTTERFLY_STAGE("row_half_mirror", "%6")                                \
        : "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3) : "v"(t4), "v"(t8), "v"(t16))
// v * (+-norm) with the lane's sign taken back; the added +0 turns a zero of either sign into +0, which is what sums and
// differences of the unsigned values give (x - x = +0, and no -0 enters: masked elements and empty sums are +0).
__device__ __forceinline__ float epilogue_norm(float v, float signed_norm) { return __builtin_fmaf(v, signed_norm, 0.0f); }

// Epilogue of the streaming kernels: the wave's accumulator tile leaves in passes of 8 rows x TN*32 columns (on the FULL path with one
// store per pass and 32-column slice exactly: a lane's chunks do not touch, so the compiler cannot put two into one, and the kernels
// count on it) through a scratch of the wave's own (outside the ring, so the ring keeps streaming the next tile); every store instruction writes
// 8 whole 128-byte lines.  With FUSED the gradient epilogue of Algorithm 1 Backward, D = alpha * H_along_n(acc . M), is
// applied on the way: mask select, the stages that combine whole 32-column groups and butterflies of stride 1 and 2 inside
// the lane, strides 4, 8, 16 between the 8 lanes that hold a row's slice (QUARTET_BUTTERFLIES_ACROSS: lane i holds 4-column
// chunk i ^ (i & 4 ? 3 : 0), which makes the partners lane ^ 1, lane ^ 2 and 7 - lane, all reachable by DPP), the
// normalization, then the scale: the same fp32 operations in the same order as the stand-alone epilogue kernel.
// acc: the wave's (TM*32) x (TN*32) tile.  A pass takes eight rows of it into LDS; a lane reads back chunk c (4 columns) of all
// 32-column slices of LDS row `sub`, so Hadamard blocks of 32, 64 and 128 columns are handled alike (group-combining stages inside
// the lane, then the 32-point stages of each slice).  The LDS has 64 banks and serves a 16-byte read 16 lanes at a time (rows 2a and
// 2a+1 here) and a 4-byte write 32 lanes at a time; row r lies at r * TN*32 floats, its columns XORed so that both keep apart:
//   v16f [TM][TN] (v_mfma_scale_f32_32x32x64_f8f6f4: lane l, register r -> row 8*(r/4) + 4*(l/32) + r%4, column l%32): pass P takes
//     registers 4*(P%4) .. +3 of the accumulators of tile row P/4, rows 8 P .. 8 P + 7 in order; columns XORed with 32*((r ^ r/4)%2).
//   v4f [2 TM][2 TN] (v_mfma_scale_f32_16x16x128_f8f6f4: lane l, register r -> row 4*(l/16) + r, column l%16): pass P takes registers
//     2*(P%2) and 2*(P%2) + 1 of the accumulators of tile row P/2, that is the rows 4*q + 2*(P%2) + e of it (q = 0..3, e = 0, 1), LDS row
//     2*q + e; columns XORed with 32*(r%2) and 16*((r/2)%2).
// WIDE (FULL only, waves of 128 columns): Hadamard blocks of 256 columns, which span the tiles of two neighbouring waves (wave ^ 1).  The
// stage that pairs columns 128 apart comes behind the stages in the lane: the waves put their values into their scratches, meet, read
// each other's and meet again before the scratch takes the next pass's rows.  Every wave of the block must come here, as often as
// the others.
template <int TM, int TN, bool OUT_BF16, bool FUSED, bool FULL, bool WIDE = false, typename ACC, int AM, int AN>
__device__ __forceinline__ void store_tile_rows8(ACC (&acc)[AM][AN], float* wbuf, void* d, uint32_t ldd,
                                                 const uint32_t* mask, float alpha, uint32_t row_base,
                                                 uint32_t col_base, uint32_t m, uint32_t n, uint32_t lane, uint32_t nb, uint32_t past) {
    static_assert(TN == 2 || TN == 4, "the slice swap of odd rows pairs the slices up");
    constexpr bool A32 = sizeof(ACC) == sizeof(v16f);
    static_assert(AM == (A32 ? TM : 2 * TM) && AN == (A32 ? TN : 2 * TN), "the accumulators must make up the tile");
    constexpr uint32_t PASSES = TM * 4, W = TN * 32;
    const uint32_t sub = lane >> 3, c = (lane & 7u) ^ ((lane & 4u) ? 3u : 0u);
    const float up4 = (c & 1u) ? -1.0f : 1.0f, up8 = (c & 2u) ? -1.0f : 1.0f, up16 = (c & 4u) ? -1.0f : 1.0f;
    const float norm = ((c ^ (c >> 1) ^ (c >> 2)) & 1u) ? -block_norm(nb) : block_norm(nb);
    const bool wide = FULL || (ldd & 3u) == 0u;
    const uint32_t mask_ld = n >> 5;
    const uint32_t lhalf = lane >> 5, wq = lane >> 4;
    float* wr = wbuf + lhalf * 4u * W + (lane & 31u);                        // v16f: + e*W + ((j ^ e ^ lhalf) % 2 swapped) * 32
    // v4f: column block j (16 columns) of LDS row 2q + e at block j ^ (q % 2) ^ 2e: an even block moves up by q % 2, an odd one down
    float* wr_even = wbuf + 2u * wq * W + (lane & 15u) + (wq & 1u) * 16u;
    float* wr_odd = wbuf + 2u * wq * W + (lane & 15u) - (wq & 1u) * 16u;
    const uint32_t rswz = A32 ? (sub ^ (sub >> 2)) & 1u : sub & 1u;
    const float* rd = wbuf + sub * W + 4u * (A32 ? c : c ^ (((sub >> 1) & 1u) * 4u));   // + ((j ^ rswz) * 32)
    // the row that pass p leaves in LDS row sub: + row_step(p)
    const uint32_t row_of_sub = row_base + (A32 ? sub : 4u * (sub >> 1) + (sub & 1u));
    auto row_step = [](uint32_t p) { return A32 ? p * 8u : (p >> 1) * 16u + (p & 1u) * 2u; };
    uint32_t mw[PASSES][TN];
    if (FUSED) {
        const bool mvec = FULL && TN == 4 && (mask_ld & 3u) == 0u && (reinterpret_cast<uintptr_t>(mask) & 15u) == 0u;   // wave-uniform
#pragma unroll
        for (uint32_t p = 0; p < PASSES; ++p) {
            const uint32_t grow = row_of_sub + row_step(p);
            if (mvec) {
                const uint4 w4 = *reinterpret_cast<const uint4*>(&mask[(size_t)grow * mask_ld + (col_base >> 5)]);
                mw[p][0] = w4.x; mw[p][1] = w4.y; mw[p][2] = w4.z; mw[p][3] = w4.w;
            } else {
#pragma unroll
                for (uint32_t j = 0; j < TN; ++j) {
                    const uint32_t gcol = col_base + j * 32u;
                    if (FULL) mw[p][j] = mask[(size_t)grow * mask_ld + (gcol >> 5)];
                    else mw[p][j] = (mask && grow < m && gcol < n) ? mask[(size_t)grow * mask_ld + (gcol >> 5)] : 0xFFFFFFFFu;
                }
            }
        }
    }
    if (FUSED) {     // the masks are here before the first store: the compiler does not count the stores below and would wait for them too
#pragma unroll
        for (uint32_t p = 0; p < PASSES; ++p)
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j) asm volatile("" : "+v"(mw[p][j]));
    }
    auto write_pass = [&](uint32_t p) __attribute__((always_inline)) {
        if constexpr (A32) {
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) wr[e * W + ((j ^ ((e & 1u) ^ lhalf)) * 32u)] = acc[p >> 2][j][(p & 3u) * 4u + e];
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 2u * TN; ++j)
#pragma unroll
                for (uint32_t e = 0; e < 2; ++e) ((j & 1u) ? wr_odd : wr_even)[e * W + (j ^ (2u * e)) * 16u] = acc[p >> 1][j][(p & 1u) * 2u + e];
        }
    };
    write_pass(0u);
#pragma unroll
    for (uint32_t p = 0; p < PASSES; ++p) {
        float4 sl[TN];
#pragma unroll
        for (uint32_t j = 0; j < TN; ++j) sl[j] = *reinterpret_cast<const float4*>(&rd[(j ^ rswz) * 32u]);
        if (!WIDE && p + 1u < PASSES) write_pass(p + 1u);     // behind the reads in the wave's LDS queue: LDS operations of a wave run in order
        const uint32_t grow = row_of_sub + row_step(p);
        float vv[TN][4];
#pragma unroll
        for (uint32_t j = 0; j < TN; ++j) {
            vv[j][0] = sl[j].x; vv[j][1] = sl[j].y; vv[j][2] = sl[j].z; vv[j][3] = sl[j].w;
            if (FUSED) {
                const int32_t bits = (int32_t)(mw[p][j] >> (4u * c));
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    vv[j][e] = __uint_as_float(__float_as_uint(vv[j][e]) & (uint32_t)((bits << (31 - (int)e)) >> 31));
            }
        }
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
        if constexpr (WIDE) {
            static_assert(FUSED && FULL && TN == 4, "two waves' 128 columns each, nothing ragged");
            const bool upper = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 1u) != 0u;
            float4* mine = reinterpret_cast<float4*>(wbuf) + lane;
            const float4* theirs = reinterpret_cast<const float4*>(upper ? wbuf - TN * 256u : wbuf + TN * 256u) + lane;
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j) mine[j * 64u] = make_float4(vv[j][0], vv[j][1], vv[j][2], vv[j][3]);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            float4 o[TN];
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j) o[j] = theirs[j * 64u];
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (p + 1u < PASSES) write_pass(p + 1u);
            const float t = upper ? -1.0f : 1.0f;      // own + theirs below, theirs - own above
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j) {
                vv[j][0] = __builtin_fmaf(vv[j][0], t, o[j].x); vv[j][1] = __builtin_fmaf(vv[j][1], t, o[j].y);
                vv[j][2] = __builtin_fmaf(vv[j][2], t, o[j].z); vv[j][3] = __builtin_fmaf(vv[j][3], t, o[j].w);
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < TN; ++j) {
            float v0 = vv[j][0], v1 = vv[j][1], v2 = vv[j][2], v3 = vv[j][3];
            if (FUSED) {
                const float a0 = v0 + v1, a1 = v0 - v1, a2 = v2 + v3, a3 = v2 - v3;
                v0 = a0 + a2; v2 = a0 - a2; v1 = a1 + a3; v3 = a1 - a3;
                QUARTET_BUTTERFLIES_ACROSS(v0, v1, v2, v3, up4, up8, up16);
                v0 = epilogue_norm(v0, norm); v1 = epilogue_norm(v1, norm); v2 = epilogue_norm(v2, norm); v3 = epilogue_norm(v3, norm);
            }
            vv[j][0] = v0 * alpha; vv[j][1] = v1 * alpha; vv[j][2] = v2 * alpha; vv[j][3] = v3 * alpha;
        }
        if (!FULL && grow >= m) continue;
        // past (a launch whose results the memory-side cache cannot hold): non-temporal; otherwise through the L2.  Against plain stores,
        // whose lines the L2 evicts and writes back while the next tiles load (us): forward 1003 x 2048 x 5632 22.1 -> 21.1; layer steps 2336 x
        // 1376 x 3168 64.8 -> 63.7, 16384 x 4096 x 4096 563 -> 547, 16384 x 4096 x 11008 1328 -> 1306.  A branch per pass, not per store;
        // for bf16 `past` is a constant.
        if (FULL && past) {
#pragma unroll
            for (uint32_t j = 0; j < TN; ++j) {
                const size_t at = (size_t)grow * ldd + col_base + j * 32u + 4u * c;
                if (OUT_BF16) {
                    const uint32_t h0 = f32_to_bf16_rne(vv[j][0]), h1 = f32_to_bf16_rne(vv[j][1]), h2 = f32_to_bf16_rne(vv[j][2]), h3 = f32_to_bf16_rne(vv[j][3]);
                    const v2u_t v = {h0 | (h1 << 16), h2 | (h3 << 16)};
                    __builtin_nontemporal_store(v, reinterpret_cast<v2u_t*>(static_cast<uint16_t*>(d) + at));
                } else {
                    const v4f v = {vv[j][0], vv[j][1], vv[j][2], vv[j][3]};
                    __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(static_cast<float*>(d) + at));
                }
            }
            continue;
        }
#pragma unroll
        for (uint32_t j = 0; j < TN; ++j) {
            const uint32_t col = col_base + j * 32u + 4u * c;
            const size_t at = (size_t)grow * ldd + col;
            const float v0 = vv[j][0], v1 = vv[j][1], v2 = vv[j][2], v3 = vv[j][3];
            if (OUT_BF16) {
                uint16_t* dst = static_cast<uint16_t*>(d) + at;
                const uint32_t h0 = f32_to_bf16_rne(v0), h1 = f32_to_bf16_rne(v1), h2 = f32_to_bf16_rne(v2), h3 = f32_to_bf16_rne(v3);
                if (FULL || (wide && col + 4u <= n)) {
                    store_through8(dst, h0 | (h1 << 16), h2 | (h3 << 16));
                } else {
                    if (col < n) dst[0] = (uint16_t)h0;
                    if (col + 1u < n) dst[1] = (uint16_t)h1;
                    if (col + 2u < n) dst[2] = (uint16_t)h2;
                    if (col + 3u < n) dst[3] = (uint16_t)h3;
                }
            } else {
                float* dst = static_cast<float*>(d) + at;
                if (FULL || (wide && col + 4u <= n)) {
                    store_through16(dst, make_uint4(f2u(v0), f2u(v1), f2u(v2), f2u(v3)));
                } else {
                    if (col < n) dst[0] = v0;
                    if (col + 1u < n) dst[1] = v1;
                    if (col + 2u < n) dst[2] = v2;
                    if (col + 3u < n) dst[3] = v3;
                }
            }
        }
    }
}


__device__ __forceinline__ v4i_t make_rsrc_words(const void* base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    v4i_t r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    return r;
}

// 16 bytes per lane from the buffer resource at byte offset voff (past the end: zeros) to LDS byte
// address lds_base + 16 * lane.  lds_base must be wave-uniform.  Completion is counted by vmcnt.
template <bool STREAM = false>   // STREAM: non-temporal, for data that is touched once
__device__ __forceinline__ void lds_direct_load16(v4i_t rsrc, uint32_t voff, uint32_t lds_base) {
    if (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                     :: "s"(lds_base), "v"(voff), "s"(rsrc) : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds_base), "v"(voff), "s"(rsrc) : "memory");
}

}  // namespace quartet
