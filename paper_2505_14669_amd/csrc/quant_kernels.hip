// Fused Hadamard + MXFP4 quantizer kernels for gfx950 (Algorithm 1, "Stage 1" of Section 4.4).
//
// One lane owns one group of 32 values end to end: the five butterfly stages, the group
// reduction (sum of squares or absmax), the scale and the 32 codes all stay in that lane's
// registers, so nothing crosses lanes and the fp32 operation order is fixed (Hadamard blocks of
// 64, 128 or 256 elements add the stages that combine whole groups in front: their groups sit in
// neighbouring lanes).  HBM traffic is wave-coalesced on both sides:
//   row mode        : a wave loads 4 KB (64 groups) with 16-byte lane-contiguous loads, swizzles it
//                     through LDS so each lane gets its own 64 bytes; codes leave as one 16-byte
//                     store per lane.
//   transposed mode : a block owns 256 source rows (one K-quad of the output).  Large bf16 matrices: lanes read 2 adjacent
//                     columns per row (256 B per wave row) into registers and the codes are gathered in LDS; otherwise (small
//                     matrices, wide Hadamard blocks, MXFP4 sources) the rows go through LDS and eight neighbouring lanes hold
//                     the eight groups of a column.  Both write whole 128-byte lines of codes.
#include "device_common.h"
#include "gemm_common.h"
#include "launchers.h"

namespace quartet {

// Eight values -> eight E2M1 codes in one dword: round-to-nearest-even of v/scale (scale a power
// of two), saturating at +-6, element j in bits [4j, 4j+4).
__device__ __forceinline__ uint32_t rtn_pack8(const float* v, float scale) {
    uint32_t w = 0u;
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[0], v[1], scale, 0);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[2], v[3], scale, 1);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[4], v[5], scale, 2);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[6], v[7], scale, 3);
    return w;
}

__device__ __forceinline__ void flip_signs(float (&v)[32], uint32_t sign_word) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = u2f(f2u(v[i]) ^ (((sign_word >> i) & 1u) << 31));
}

// Hadamard blocks of 64, 128 or 256 elements (nb = 2, 4, 8 groups): the groups of a K-quad sit in eight consecutive lanes,
// lane sub = lane % 8 holding group j of the K-quad.  Groups that a group-combining stage pairs up differ in one bit of j;
// j = sub ^ (sub & 4 ? 3 : 0) makes the partners sub ^ 1, sub ^ 2 and 7 - sub, which DPP reaches inside the arithmetic
// instruction.
__device__ __forceinline__ uint32_t kquad_group_of(uint32_t sub) { return sub ^ ((sub & 4u) ? 3u : 0u); }

// sign word of group j of its Hadamard block (nb groups) for a lane
__device__ __forceinline__ uint32_t lane_sign_word(const SrParams& p, uint32_t j) {
    uint32_t sw = p.sign_words[0];
#pragma unroll
    for (uint32_t q = 1; q < 8; ++q) sw = ((j & (p.nb - 1u)) == q) ? p.sign_words[q] : sw;
    return sw;
}

// 0xFFFFFFFF if bit i of w is set, else 0
__device__ __forceinline__ uint32_t bit_mask(uint32_t w, uint32_t i) { return (uint32_t)__builtin_amdgcn_sbfe((int)w, i, 1u); }

#define QUARTET_STAGE_ALL(CTRL_TEXT, v, t)                                                          \
    _Pragma("unroll") for (int i_ = 0; i_ < 32; i_ += 4)                                             \
        QUARTET_STAGE4_DPP(CTRL_TEXT, v[i_], v[i_ + 1], v[i_ + 2], v[i_ + 3], t);

// Group-combining stages of a Hadamard block of nb = 2, 4 or 8 groups held by lanes as above, the 32-point stages and the
// normalization.  A group-combining stage leaves -(a - b) in the upper lane and the normalization takes the sign back (see
// cross_lane_stage); zeros come out as +0.
__device__ __forceinline__ void rotate_block_lanes(float (&v)[32], uint32_t j, uint32_t nb) {
    const float t1 = (j & 1u) ? -1.0f : 1.0f, t2 = (j & 2u) ? -1.0f : 1.0f, t4 = (j & 4u) ? -1.0f : 1.0f;
    QUARTET_STAGE_ALL("quad_perm:[1,0,3,2]", v, t1)
    if (nb > 2u) { QUARTET_STAGE_ALL("quad_perm:[2,3,0,1]", v, t2) }
    if (nb > 4u) { QUARTET_STAGE_ALL("row_half_mirror", v, t4) }
    fwht32_unscaled(v);
    const float c = block_norm_signed(nb, j);
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = __builtin_fmaf(v[i], c, 0.0f);
}

// Encode one rotated group held in v[]: scale, codes, mask.  q_base = (linear output position of
// element 0)/16 is the Philox call index of the group's first 16 elements.
template <int MODE>
__device__ __forceinline__ void encode_group(float (&v)[32], const SrParams& p, uint32_t stream, uint64_t q_base,
                                             uint4& codes, uint32_t& scale_byte, uint32_t& mask_word) {
    uint32_t c[4] = {0u, 0u, 0u, 0u};
    if (MODE == kFwd) {
        // QuEST: scale from the group RMS, round to nearest, remember what clipped
        float t[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) t[i] = v[i] * v[i];
#pragma unroll
        for (int n = 16; n >= 1; n >>= 1) {
#pragma unroll
            for (int i = 0; i < n; ++i) t[i] = t[2 * i] + t[2 * i + 1];
        }
        uint32_t E = (f2u(t[0]) >> 23) & 0xFFu;
        int e = (E == 0u) ? 0 : (((int)E - 133) >> 1);   // floor((log2 ss - 6) / 2)
        uint32_t b = (uint32_t)(e + 127);
        float scale = u2f(b << 23);                        // 2^e
        float thr = u2f(0x40C00000u + ((uint32_t)e << 23)); // 6 * 2^e
        uint32_t m = 0u;
#pragma unroll
        for (int i = 31; i >= 0; --i) m = (m << 1) | (__builtin_fabsf(v[i]) <= thr ? 1u : 0u);
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = rtn_pack8(&v[8 * i], scale);
        scale_byte = b;
        mask_word = m;
    } else {
        // AbsMax power-of-two scale, 3/4 range matching, RTN or SR (nothing clips)
        float mx = 0.0f;
#pragma unroll
        for (int i = 0; i < 32; ++i) mx = __builtin_fmaxf(mx, __builtin_fabsf(v[i]));
        uint32_t E = (f2u(mx) >> 23) & 0xFFu;
        uint32_t b = (E == 0u) ? 127u : (E >= 2u ? E - 2u : 0u);
        float mult = u2f((254u - b) << 23) * 0.75f;        // 3/4 * 2^-e, exact
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = v[i] * mult;
        if (MODE == kBwdRtn) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = rtn_pack8(&v[8 * i], 1.0f);
        } else {
#pragma unroll
            for (int call = 0; call < 2; ++call) {
                uint64_t q = q_base + (uint64_t)call;
                uint32_t w[4];
                philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), stream, 0u, p.key0, p.key1, w);
                c[2 * call] = sr_pack8(&v[16 * call], w[0], w[1]);
                c[2 * call + 1] = sr_pack8(&v[16 * call + 8], w[2], w[3]);
            }
        }
        scale_byte = b;
        mask_word = 0xFFFFFFFFu;
    }
    codes = make_uint4(c[0], c[1], c[2], c[3]);
}

// Sign bit of element i of the randomized rotation's sign vector as a float's sign bit (wave-uniform: scalar arithmetic).
__device__ __forceinline__ uint32_t sign_bit(uint32_t sign_word, uint32_t i) { return ((sign_word >> i) & 1u) << 31; }

// Eight bf16 values (elements first .. first+7 of a group) to fp32 with the sign vector applied on the way.  An even
// element is x << 16 plus its sign bit: adding 0x80000000 flips the top bit, and shift-and-add is one instruction where
// shift and XOR are two; an odd element is one three-input bit operation either way.
__device__ __forceinline__ void unpack_bf16x8_signed(const uint4& q, float* v, uint32_t sign_word, uint32_t first) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        v[2 * j] = u2f((w[j] << 16) + sign_bit(sign_word, first + 2u * j));
        v[2 * j + 1] = u2f((w[j] & 0xFFFF0000u) ^ sign_bit(sign_word, first + 2u * j + 1u));
    }
}

__device__ __forceinline__ void unpack_bf16x8(const uint4& q, float* v) {
    v[0] = u2f(q.x << 16); v[1] = u2f(q.x & 0xFFFF0000u);
    v[2] = u2f(q.y << 16); v[3] = u2f(q.y & 0xFFFF0000u);
    v[4] = u2f(q.z << 16); v[5] = u2f(q.z & 0xFFFF0000u);
    v[6] = u2f(q.w << 16); v[7] = u2f(q.w & 0xFFFF0000u);
}

// Codes and masks of a matrix [rows x 32 gk] go through the L2 and stay in the memory-side cache (256 MB), where the product that
// follows finds them; from 64 MB of codes on they go past it, where they would displace more than they bring.  Against non-temporal
// stores for all (us): forward 1003 x 2048 x 5632 23.3 -> 22.1; layer steps 4096 x 2048 x 2048 76.8 -> 71.2, 2336 x 1376 x 3168 69.9 ->
// 64.8, 8192 x 5632 x 2048 249.6 -> 238.7, 16384 x 4096 x 4096 580 -> 563.  The quantizers alone on rotating buffers, through the L2 / past it
// (GB/s): 16384 x 4096 forward 6110 / 5770, stochastic transposed 4610 / 4550; 16384 x 11008 4770 / 5600, 4700 / 5250.
__device__ __forceinline__ bool codes_past_cache(uint32_t rows, uint32_t gk) { return (uint64_t)rows * gk >= (64u << 20) / 16u; }
__device__ __forceinline__ void store_codes(void* p, const uint4& q, bool past) {
    if (past) store_stream16(p, q);
    else store_through16(p, q);
}
__device__ __forceinline__ void store_mask(void* p, uint32_t m, bool past) {
    if (past) store_stream4(p, m);
    else store_through4(p, m);
}

// ------------------------------------------------------------------ row mode
// Block = 8 rows x 32 groups (four 256-element K-quads, 2 KB of bf16 per row).  Wave w owns rows
// 2w, 2w+1; lane l the group l%32 of row l/32.  Loads are lane-contiguous 16-byte chunks, swizzled
// through LDS so each lane ends up with its own group's 64 bytes.  Codes leave as 512 contiguous
// bytes per row, mask words as 128; the 256 scale bytes of the block are exchanged through LDS and
// leave as whole 32-byte runs of the scale tiles (8 rows x one dword), never as single bytes.
// BIG: the Hadamard block spans p.nb = 2, 4 or 8 groups; they sit in consecutive lanes (a row's groups
// start at a multiple of 8 in every block), so the group-combining stages are lane exchanges.
// bid: the block's number in its matrix; stage (16 KB), s_scale (256 B): the block's LDS
template <int MODE, bool MASK, bool BIG>
__device__ __forceinline__ void quant_row_tile(const uint16_t* __restrict__ x, uint32_t rows, uint32_t gk, int64_t ldx,
                                               uint4* __restrict__ codes, uint8_t* __restrict__ scales, uint32_t* __restrict__ mask,
                                               const SrParams& p, uint32_t stream, uint32_t k_blocks, FastDiv div_k_blocks, uint32_t bid,
                                               uint4 (*stage)[256], uint32_t* s_scale) {
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    // consecutive blocks walk along K inside the same 8 rows, so the blocks in flight cover one
    // contiguous stretch of the input
    const uint32_t row_set = fast_div(bid, div_k_blocks);
    const uint32_t row0 = row_set * 8u, kq0 = (bid - row_set * k_blocks) * 4u, kqs = (gk + 7u) >> 3;
    // The block's rows through a buffer resource that ends with the last element of its last row:
    // rows past the matrix read as zeros without a predicate.  Groups past k inside a row read
    // whatever lies there (the row's padding or the next row); their results are never stored.
    const uint32_t rows_here = (rows - row0) < 8u ? (rows - row0) : 8u;
    const __amdgpu_buffer_rsrc_t res_x = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(x + (size_t)row0 * ldx), 0, (int)(((rows_here - 1u) * (uint32_t)ldx + gk * 32u) * 2u), 0x00020000);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        uint32_t c = 64u * j + lane;                       // 16-byte chunk inside the wave's 2 rows x 2 KB
        const uint32_t voff = ((wave * 2u + (c >> 7)) * (uint32_t)ldx + kq0 * 256u + (c & 127u) * 8u) * 2u;
        v4u_t q = __builtin_amdgcn_raw_buffer_load_b128(res_x, (int)voff, 0, 2 /* non-temporal */);
        stage[wave][(c & ~3u) | ((c & 3u) ^ ((c >> 4) & 3u))] = make_uint4(q.x, q.y, q.z, q.w);
    }
    __syncthreads();
    float v[32];
    // BIG: the lane's group inside the wave's 64
    const uint32_t gw = BIG ? (lane & ~7u) | kquad_group_of(lane & 7u) : lane;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        uint4 q = stage[wave][4u * gw + (j ^ ((gw >> 2) & 3u))];
        if (MODE != kFwd && !BIG) unpack_bf16x8_signed(q, &v[8 * j], p.sign_word, 8u * j);
        else unpack_bf16x8(q, &v[8 * j]);
    }
    const uint32_t row_local = wave * 2u + (gw >> 5), gi = gw & 31u;
    const uint32_t row = row0 + row_local, g = kq0 * 8u + gi;
    uint4 out;
    uint32_t sb, mw;
    if (BIG) {
        if (MODE != kFwd) flip_signs(v, lane_sign_word(p, gi & 7u));
        rotate_block_lanes(v, gi & 7u, p.nb);
    } else {
        fwht32(v);
    }
    encode_group<MODE>(v, p, stream, ((uint64_t)row * gk + g) * 2u, out, sb, mw);
    // scale byte of (row, group gi) -> position of the tiled layout inside the block's 256 bytes:
    // [K-quad gi/8][h = gi%2][row_local][p = (gi%8)/2]
    reinterpret_cast<uint8_t*>(s_scale)[(((gi >> 3) * 2u + (gi & 1u)) * 8u + row_local) * 4u + ((gi & 7u) >> 1)] = (uint8_t)sb;
    if (row < rows && g < gk) {
        const size_t gidx = (size_t)row * gk + g;
        const bool past = codes_past_cache(rows, gk);
        store_codes(&codes[gidx], out, past);
        if (MASK) store_mask(&mask[gidx], mw, past);
    }
    __syncthreads();
    if (threadIdx.x < 64u) {
        const uint32_t t = threadIdx.x, kql = t >> 4, h = (t >> 3) & 1u, rl = t & 7u;
        const uint32_t r = row0 + rl, kq = kq0 + kql;
        if (r < rows && kq * 8u + h < gk) {
            uint8_t* dst = scales + scale_tile_offset(r, kq * 8u + h, kqs);   // dword of (row, h) in tile kq
            const uint32_t w = s_scale[t];
            if (kq * 8u + 8u <= gk) {
                *reinterpret_cast<uint32_t*>(dst) = w;
            } else {                                         // ragged last K-quad: only the bytes that exist
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    if (kq * 8u + 2u * q + h < gk) dst[q] = (uint8_t)(w >> (8u * q));
            }
        }
    }
}

template <int MODE, bool MASK, bool BIG>
__global__ void __launch_bounds__(256)
quant_row_kernel(const uint16_t* __restrict__ x, uint32_t rows, uint32_t gk, int64_t ldx,
                 uint4* __restrict__ codes, uint8_t* __restrict__ scales, uint32_t* __restrict__ mask,
                 SrParams p, uint32_t k_blocks, FastDiv div_k_blocks) {
    __shared__ uint4 stage[4][256];
    __shared__ uint32_t s_scale[64];
    quant_row_tile<MODE, MASK, BIG>(x, rows, gk, ldx, codes, scales, mask, p, p.stream_id, k_blocks, div_k_blocks, blockIdx.x, stage, s_scale);
}

// Two matrices with the same inner dimension in one launch (Algorithm 1 Forward quantizes X and W, and neither depends
// on the other): blocks [0, split) work on the first, the rest on the second.  A weight-sized matrix alone fills the chip
// for a few microseconds only, most of it ramp-up and drain; behind the activations' blocks it costs its bytes.
struct RowMatrix {
    const uint16_t* x;
    uint32_t rows;
    int64_t ldx;
    uint4* codes;
    uint8_t* scales;
    uint32_t* mask;
};

template <int MODE, bool MASK, bool BIG>
__global__ void __launch_bounds__(256)
quant_row_pair_kernel(RowMatrix a, RowMatrix b, uint32_t split, uint32_t gk, SrParams p, uint32_t k_blocks, FastDiv div_k_blocks) {
    __shared__ uint4 stage[4][256];
    __shared__ uint32_t s_scale[64];
    const bool second = blockIdx.x >= split;
    // field by field: both matrices' arguments are on their way together with split, not behind it (forward 1003 x 2048 x 5632 21.03 -> 20.86 us)
    const RowMatrix m = {second ? b.x : a.x, second ? b.rows : a.rows, second ? b.ldx : a.ldx, second ? b.codes : a.codes,
                         second ? b.scales : a.scales, second ? b.mask : a.mask};
    quant_row_tile<MODE, MASK, BIG>(m.x, m.rows, gk, m.ldx, m.codes, m.scales, m.mask, p, p.stream_id, k_blocks, div_k_blocks,
                                      second ? blockIdx.x - split : blockIdx.x, stage, s_scale);
}

// Store phase of the transposed kernels: the tile's codes, scale bytes and mask words gathered in LDS
// ([local column][group], codes with a 16-byte slot swizzle; columns 16..31 of every 32 swap places in pairs, which
// puts the 16 lanes of a 16-byte LDS access on the 64 banks' 16 different slots) leave as full 128-byte lines of codes,
// 32-byte runs of mask words and whole dwords of the scale tiles.
template <bool MASK>
__device__ __forceinline__ void transposed_store_tile(const uint4* s_codes, const uint8_t* s_scales, const uint32_t* s_mask,
                                                      uint32_t col0, uint32_t grp0, uint32_t rows, uint32_t gk, uint32_t k,
                                                      uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                                      uint32_t* __restrict__ mask) {
    // full 128-byte lines of codes: 8 lanes per output row
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j) {
        uint32_t id = threadIdx.x + 256u * j;
        uint32_t lc = id >> 3, part = id & 7u;
        uint32_t r = col0 + lc, grp = grp0 + part;
        if (r < rows && grp < gk) {
            uint4 q = s_codes[(lc ^ ((lc >> 4) & 1u)) * 8u + (part ^ ((lc >> 1) & 7u))];
            store_codes(codes + (size_t)r * (k >> 1) + (size_t)grp * 16u, q, codes_past_cache(rows, gk));
        }
    }
    if (MASK) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            uint32_t id = threadIdx.x + 256u * j;
            uint32_t lc = id >> 3, part = id & 7u;
            uint32_t r = col0 + lc, grp = grp0 + part;
            if (r < rows && grp < gk) mask[(size_t)r * gk + grp] = s_mask[lc * 8u + part];
        }
    }
    // scales: the block's 8 groups are one K-quad, so each 32-row block of the tile is one 256-byte
    // scale tile; thread t writes dword t%64 of tile t/64 (bytes = groups h, 2+h, 4+h, 6+h of its row)
    const uint32_t t = threadIdx.x, lc = (t >> 6) * 32u + (t & 31u), h = (t >> 5) & 1u;
    const uint32_t r = col0 + lc;
    if (r < rows) {
        uint32_t w = 0u;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) w |= (uint32_t)s_scales[lc * 8u + 2u * q + h] << (8u * q);
        const uint32_t kq = (gk + 7u) >> 3;
        uint32_t* dst = reinterpret_cast<uint32_t*>(scales + scale_tile_offset(r, grp0 + h, kq));
        if (grp0 + 6u + h < gk) {
            *dst = w;
        } else {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (grp0 + 2u * q + h < gk) reinterpret_cast<uint8_t*>(dst)[q] = (uint8_t)(w >> (8u * q));
        }
    }
}

// ------------------------------------------------------------------ transposed mode, bf16 source, whole-chip matrices
// Logical A[rows x k] = S^T where the source S is bf16 [k x ldx], Hadamard block = the group.
// Block tile: 8 groups (256 source rows, one K-quad of the output) x 128 source columns; wave w owns groups 2w, 2w+1; lane l
// owns columns 2l, 2l+1.  Bound by memory (nearest) or vector-ALU issue (stochastic).  Every load reads 256 contiguous bytes of one
// source row into registers, 64 of them in flight per wave: on large matrices that streams faster than the 128-byte pieces
// through LDS of quant_columns_block, which is the better kernel below about 2000 of its waves and for wider Hadamard blocks
// (16384 x 11008, stochastic / nearest: 95 / 83 us here, 100 / 88 there; 4096 x 2048: 8.3 / 6.9 here, 7.6 / 6.5 there; 256 x 512:
// 6.7 / 5.4 here, 3.4 / 3.1 there).
// bx, by: the block's K-quad and column tile; s_codes (16 KB), s_scales (1 KB), s_mask (4 KB): the block's LDS
template <int MODE, bool MASK>
__device__ __forceinline__ void quant_transposed_tile(const uint16_t* __restrict__ src,
                                                      uint32_t rows, uint32_t k, int64_t ldx, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, uint32_t* __restrict__ mask,
                                                      const SrParams& p, uint32_t stream, uint32_t bx, uint32_t by,
                                                      uint4* s_codes, uint8_t* s_scales, uint32_t* s_mask) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    const uint32_t gk = k >> 5;
    const uint32_t col0 = by * 128u;
    const uint32_t grp0 = bx * 8u;
    const uint32_t col = col0 + 2u * lane;                // even; rows is even, so col+1 < rows too
    // the block's corner of the source through a buffer resource that ends with the last column of the
    // last source row
    const uint32_t src_rows = (k - grp0 * 32u) < 256u ? (k - grp0 * 32u) : 256u;
    const uint32_t src_cols = (rows - col0) < 128u ? (rows - col0) : 128u;
    const __amdgpu_buffer_rsrc_t res_x = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(src + (size_t)grp0 * 32u * ldx + col0), 0,
        (int)(((src_rows - 1u) * (uint32_t)ldx + src_cols) * 2u), 0x00020000);

    // all 64 loads of the wave's two groups go out before any arithmetic: the second group's data
    // arrives while the first is rotated and quantized.  Rows past k read as zeros without a predicate
    // (the wave-uniform row offset rides in the scalar offset and takes part in the range check);
    // columns past `rows` inside a source row read whatever lies there, their results are never stored.
    uint32_t raw[2][32];
#pragma unroll
    for (uint32_t rb = 0; rb < 2; ++rb) {
#pragma unroll
        for (uint32_t i = 0; i < 32; ++i)
            raw[rb][i] = __builtin_amdgcn_raw_buffer_load_b32(
                res_x, (int)(4u * lane), (int)(((2u * wave + rb) * 32u + i) * (uint32_t)ldx * 2u), 2 /* non-temporal */);
    }
#pragma unroll
    for (uint32_t rb = 0; rb < 2; ++rb) {
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t gl = 2u * wave + rb;               // group inside the block tile
        const uint32_t grp = grp0 + gl;
        const uint32_t sw = lane & 7u;                    // 16-byte slot swizzle against bank conflicts
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c) {
            float v[32];
#pragma unroll
            for (uint32_t i = 0; i < 32; ++i) {       // with the sign vector applied on the way (forward: sign word 0 in p)
                const uint32_t sbit = MODE != kFwd ? sign_bit(p.sign_word, i) : 0u;
                v[i] = c ? u2f((raw[rb][i] & 0xFFFF0000u) ^ sbit) : u2f((raw[rb][i] << 16) + sbit);
            }
            uint4 q;
            uint32_t sb, m;
            // output position of element 0 of the group: row*k + grp*32, divided by 16
            fwht32(v);
            encode_group<MODE>(v, p, stream, ((uint64_t)(col + c) * k + grp * 32u) >> 4, q, sb, m);
            const uint32_t lc = 2u * lane + c;            // local column
            s_codes[(lc ^ ((lc >> 4) & 1u)) * 8u + (gl ^ sw)] = q;
            s_scales[lc * 8u + gl] = (uint8_t)sb;
            if (MASK) s_mask[lc * 8u + gl] = m;
        }
    }
    __syncthreads();
    transposed_store_tile<MASK>(s_codes, s_scales, s_mask, col0, grp0, rows, gk, k, codes, scales, mask);
}

// ------------------------------------------------------------------ transposed conversions, lanes along the output's groups
// A block covers 256 source rows (the 8 groups of one K-quad of the output) by B = 128, 64 or 32 bytes of each row.  The rows
// go to LDS by LDS-direct loads of 16 bytes per lane (whole pieces of a row, no registers, all of them in flight at once);
// then a lane owns one group of a column: sub = lane % 8 stands for group j of the K-quad (kquad_group_of), lane / 8 for a
// chunk of neighbouring columns, and it reads its chunk of the group's 32 rows back.
//   - The groups of a Hadamard block above 32 sit in neighbouring lanes.
//   - The eight lanes of a chunk hold the 128 contiguous bytes of codes of one output row and K-quad: every 16-byte store
//     instruction writes whole lines.
// STREAM: read non-temporally (large matrices; small ones come out of the caches: 4096 x 2048 7.6 us cached, 8.3 streamed; so do
// large ones where two blocks share a line, see launch_transposed_nb).
// Group j's 32 rows start at j * kquad_pitch(B): the 32 bytes of padding put the rows i of the eight groups, which one read
// instruction addresses, on different banks.
template <uint32_t B> __host__ __device__ constexpr uint32_t kquad_pitch() { return 32u * B + 32u; }
template <uint32_t B, bool STREAM>
__device__ __forceinline__ void stage_kquad_rows(const v4i_t& res, uint32_t pitch, const void* lds) {
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr uint32_t CPR = B / 16u, RPI = 64u / CPR, PER_GROUP = 32u / RPI, PER_WAVE = 2u * PER_GROUP;   // wave w: groups 2w, 2w + 1
    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)const_cast<void*>(lds);
    const uint32_t voff = (lane / CPR) * pitch + (lane % CPR) * 16u;
#pragma unroll
    for (uint32_t t = 0; t < PER_WAVE; ++t) {
        const uint32_t grp = 2u * wave + t / PER_GROUP, part = t % PER_GROUP;
        lds_direct_load16<STREAM>(res, voff + (grp * 32u + part * RPI) * pitch, lds0 + grp * kquad_pitch<B>() + part * 1024u);
    }
}

// The scale bytes of a wave's COLS output rows in one K-quad: a lane has put the bytes of its group into s ([h][row][byte],
// see scale_tile_offset); they leave as whole dwords of a scale tile.  row0 is a multiple of COLS, COLS divides 32.
template <uint32_t COLS>
__device__ __forceinline__ void store_kquad_scales(const uint32_t* s, uint8_t* __restrict__ scales, uint32_t row0, uint32_t rows,
                                                   uint32_t grp0, uint32_t gk, uint32_t lane) {
    const uint32_t h = lane / COLS, r = row0 + lane % COLS;
    if (lane < 2u * COLS && r < rows && grp0 + h < gk) {
        uint8_t* dst = scales + scale_tile_offset(r, grp0 + h, (gk + 7u) >> 3);
        const uint32_t w = s[lane];
        if (grp0 + 6u + h < gk) {
            *reinterpret_cast<uint32_t*>(dst) = w;
        } else {                                       // ragged last K-quad: only the bytes that exist
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (grp0 + 2u * q + h < gk) dst[q] = (uint8_t)(w >> (8u * q));
        }
    }
}

// bf16 source.  Logical A[rows x k] = S^T where the source S is bf16 [k x ldx]; the block covers 32 * CPL columns from col0 on (CPL
// = 2: 128-byte pieces of the source rows; CPL = 1: half of that, for matrices too small to fill the chip), K-quad bx.  STREAM: read
// non-temporally.
// lds: 8 * kquad_pitch<64 CPL>() bytes, s_scale: 64 * CPL dwords.
template <int MODE, bool MASK, bool BIG, uint32_t CPL, bool STREAM>
__device__ __forceinline__ void quant_columns_block(const uint16_t* __restrict__ src, uint32_t rows, uint32_t k, int64_t ldx,
                                                    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                                    uint32_t* __restrict__ mask, const SrParams& p, uint32_t stream, uint32_t bx, uint32_t col0,
                                                    const void* lds, uint32_t* s_scale) {
    constexpr uint32_t B = 64u * CPL;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t chunk = lane >> 3, j = kquad_group_of(lane & 7u);
    const uint32_t gk = k >> 5, grp0 = bx * 8u, grp = grp0 + j;
    // the block's corner of the source through a buffer resource that ends with the last column of the last source row:
    // rows past k read as zeros without a predicate; columns past `rows` inside a source row read whatever lies there,
    // their results are never stored
    const uint32_t src_rows = (k - grp0 * 32u) < 256u ? (k - grp0 * 32u) : 256u;
    const uint32_t src_cols = (rows - col0) < 32u * CPL ? (rows - col0) : 32u * CPL;
    const v4i_t res_x = make_rsrc_words(src + (size_t)grp0 * 32u * ldx + col0, ((src_rows - 1u) * (uint32_t)ldx + src_cols) * 2u);
    stage_kquad_rows<B, STREAM>(res_x, (uint32_t)ldx * 2u, lds);
    const uint32_t sw = BIG && MODE != kFwd ? lane_sign_word(p, j) : 0u;
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    const uint8_t* mine = static_cast<const uint8_t*>(lds) + j * kquad_pitch<B>() + (wave * 8u + chunk) * (2u * CPL);
    uint32_t raw[32];
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) {
        raw[i] = CPL == 2u ? *reinterpret_cast<const uint32_t*>(mine + i * B) : (uint32_t)*reinterpret_cast<const uint16_t*>(mine + i * B);
        if (BIG && MODE != kFwd) raw[i] ^= bit_mask(sw, i) & 0x80008000u;      // the lane's sign vector on both halves
    }
    uint32_t* s = s_scale + wave * 16u * CPL;
#pragma unroll
    for (uint32_t c = 0; c < CPL; ++c) {
        __builtin_amdgcn_sched_barrier(0);            // one column at a time
        float v[32];
#pragma unroll
        for (uint32_t i = 0; i < 32; ++i) {           // unpacked with the sign vector applied on the way (forward: sign word 0)
            const uint32_t sbit = (MODE != kFwd && !BIG) ? sign_bit(p.sign_word, i) : 0u;
            v[i] = c ? u2f((raw[i] & 0xFFFF0000u) ^ sbit) : u2f((raw[i] << 16) + sbit);
        }
        if (BIG) rotate_block_lanes(v, j, p.nb);
        else fwht32(v);
        const uint32_t lc = chunk * CPL + c, r = col0 + wave * 8u * CPL + lc;
        uint4 q;
        uint32_t sb, m;
        // output position of element 0 of the group: row*k + grp*32, divided by 16
        encode_group<MODE>(v, p, stream, ((uint64_t)r * k + grp * 32u) >> 4, q, sb, m);
        reinterpret_cast<uint8_t*>(s)[((j & 1u) * 8u * CPL + lc) * 4u + (j >> 1)] = (uint8_t)sb;
        if (r < rows && grp < gk) {
            store_codes(codes + (size_t)r * (k >> 1) + (size_t)grp * 16u, q, codes_past_cache(rows, gk));
            if (MASK) mask[(size_t)r * gk + grp] = m;
        }
    }
    __builtin_amdgcn_wave_barrier();                  // the bytes are the wave's own and a wave's LDS operations run in order
    store_kquad_scales<8u * CPL>(s, scales, col0 + wave * 8u * CPL, rows, grp0, gk, lane);
}

// Column tile of the block with K-quad bx and nominal column tile by, of n_ct column tiles (a bijection for every bx): with
// a dense source whose row pitch is a multiple of a few KB, the blocks in flight would otherwise all read the same stretch of
// columns of every row, which the memory channels serve unevenly (measured: 5-9 % slower; a source with 128 bytes of padding
// per row does not show it).  Blocks are numbered K-quad first: the blocks that run at the same time then write neighbouring
// 128-byte lines of the same output rows (10 % faster than column-tile first).
__device__ __forceinline__ uint32_t transposed_column_tile(uint32_t bx, uint32_t by, uint32_t n_ct) { return (by + bx) % n_ct; }

// Stochastic: scheduled for two to three waves per SIMD (16384 x 11008: 87.0 us, scheduled for three alone 88.6); nearest: four.
template <int MODE, bool MASK>
__attribute__((amdgpu_waves_per_eu(MODE == kBwdSr ? 2 : 4, MODE == kBwdSr ? 3 : 8)))
__global__ void __launch_bounds__(256)
quant_transposed_kernel(const uint16_t* __restrict__ src,
                        uint32_t rows, uint32_t k, int64_t ldx, uint8_t* __restrict__ codes,
                        uint8_t* __restrict__ scales, uint32_t* __restrict__ mask, SrParams p) {
    __shared__ uint4 s_codes[128 * 8];
    __shared__ uint8_t s_scales[128 * 8];
    __shared__ uint32_t s_mask[128 * 8];
    quant_transposed_tile<MODE, MASK>(src, rows, k, ldx, codes, scales, mask, p, p.stream_id, blockIdx.x,
                                      transposed_column_tile(blockIdx.x, blockIdx.y, gridDim.y), s_codes, s_scales, s_mask);
}

// STREAM false with CPL = 2: the launch may round the K-quads up
template <int MODE, bool MASK, bool BIG, uint32_t CPL, bool STREAM>
__global__ void __launch_bounds__(256, 4)
quant_columns_kernel(const uint16_t* __restrict__ src,
                        uint32_t rows, uint32_t k, int64_t ldx, uint8_t* __restrict__ codes,
                        uint8_t* __restrict__ scales, uint32_t* __restrict__ mask, SrParams p) {
    __shared__ __align__(16) uint8_t stage[8u * kquad_pitch<64u * CPL>()];
    __shared__ uint32_t s_scale[64u * CPL];
    if (CPL == 2u && !STREAM && blockIdx.x >= (k + 255u) >> 8) return;
    quant_columns_block<MODE, MASK, BIG, CPL, STREAM>(src, rows, k, ldx, codes, scales, mask, p, p.stream_id, blockIdx.x,
                                              transposed_column_tile(blockIdx.x, blockIdx.y, gridDim.y) * 32u * CPL, stage, s_scale);
}

// MXFP4 source: re-quantization of a saved MXFP4 tensor S [k x rows] along its other dimension (Algorithm 1 Backward: the
// operands W_q^T and X_q^T).  The block covers 32 * NC source columns from c0 on, K-quad kq of the output; NC = 8, 4, 2: 128, 64, 32
// bytes of codes of every source row (less work per wave for smaller problems).  Codes are decoded two columns at a time.
// lds: 8 * kquad_pitch<16 NC>() bytes and at least 9216, s_scale: 64 * NC dwords.
template <int MODE, bool BIG, uint32_t NC>
__device__ __forceinline__ void requant_columns_block(const uint8_t* __restrict__ src_codes, const uint8_t* __restrict__ src_scales,
                                                      uint32_t rows, uint32_t k, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, const SrParams& p, uint32_t stream, uint32_t kq, uint32_t col0,
                                                      void* lds, uint32_t* s_scale) {
    constexpr uint32_t B = 16u * NC;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t chunk = lane >> 3, j = kquad_group_of(lane & 7u);
    const uint32_t gk = k >> 5, grp0 = kq * 8u, grp = grp0 + j, c0 = col0 + wave * 8u * NC;
    const uint32_t half = rows >> 1, skq = (rows + 255u) >> 8;  // source row pitch in bytes, source K-quads
    // the source codes of the K-quad's rows and the scale tiles of their row blocks, through buffer resources that end with the
    // data: source rows past k read as zeros; columns past `rows` read whatever lies there, the output rows they feed are
    // never stored
    const uint32_t src_rows = (k - grp0 * 32u) < 256u ? (k - grp0 * 32u) : 256u;
    const v4i_t res_c = make_rsrc_words(src_codes + (size_t)grp0 * 32u * half + (col0 >> 1), src_rows * half - (col0 >> 1));
    stage_kquad_rows<B, false>(res_c, half, lds);
    // A lane's 32 scales are one byte of 32 neighbouring dwords of its row block's tile: column group g of the K-quad, dwords of
    // half h = g % 2, byte g / 2 (the same for the whole wave).  The lanes of the four chunks that may share (j, h) form eight
    // of them each, as floats, and share them through LDS.
    const size_t tile0 = ((size_t)grp0 * skq + (c0 >> 8)) * 256u, scale_bytes = (size_t)gk * skq * 256u;
    const size_t scale_left = tile0 < scale_bytes ? scale_bytes - tile0 : 0;
    const __amdgpu_buffer_rsrc_t res_s = make_rsrc(src_scales + tile0, (uint32_t)(scale_left < (size_t)8 * skq * 256u ? scale_left : (size_t)8 * skq * 256u));
    const uint32_t gbyte = (c0 >> 6) & 3u, h = ((c0 + chunk * NC) >> 5) & 1u, h4 = ((c0 >> 5) & 1u) ^ (chunk >> 2);
    const int scale_off = (int)(j * skq * 256u + h4 * 128u + (chunk & 3u) * 32u);
    const v4u_t d0 = __builtin_amdgcn_raw_buffer_load_b128(res_s, scale_off, 0, 0);
    const v4u_t d1 = __builtin_amdgcn_raw_buffer_load_b128(res_s, scale_off, 16, 0);
    const uint32_t sw = BIG ? lane_sign_word(p, j) : p.sign_word;
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    const uint8_t* mine = static_cast<const uint8_t*>(lds) + j * kquad_pitch<B>() + (wave * 8u + chunk) * (NC / 2u);
    uint32_t w[32];
    // the sign vector applied on the codes: all values of a word are element i of their groups (sign-magnitude: decoding the
    // flipped code gives the negated value exactly, zeros included)
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) {
        w[i] = NC == 8u ? *reinterpret_cast<const uint32_t*>(mine + i * B)
             : NC == 4u ? (uint32_t)*reinterpret_cast<const uint16_t*>(mine + i * B) : (uint32_t)mine[i * B];
        w[i] ^= bit_mask(sw, i) & 0x88888888u;
    }
    __syncthreads();                                   // every wave has its codes: their LDS serves the scales from here on
    constexpr uint32_t SROW = 36u;                     // floats per (h, j): 16-byte aligned, the eight j of a read on different banks
    float* fs = static_cast<float*>(lds) + wave * 16u * SROW;
    {
        const uint32_t d[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        float f[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) f[i] = u2f(((d[i] >> (8u * gbyte)) & 0xFFu) << 23);
        float4* dst = reinterpret_cast<float4*>(fs + (h4 * 8u + j) * SROW + (chunk & 3u) * 8u);
        dst[0] = make_float4(f[0], f[1], f[2], f[3]);
        dst[1] = make_float4(f[4], f[5], f[6], f[7]);
    }
    __builtin_amdgcn_wave_barrier();
    const float4* my_scales = reinterpret_cast<const float4*>(fs + (h * 8u + j) * SROW);
    uint32_t* s = s_scale + wave * 16u * NC;
    // of the lane's current column (an output row): linear position / 16 of its group's first element, and its 16 bytes of codes
    const uint32_t r0 = c0 + chunk * NC;
    uint64_t q_base = ((uint64_t)r0 * k + grp * 32u) >> 4;
    uint8_t* dst_codes = codes + (size_t)r0 * (k >> 1) + (size_t)grp * 16u;
    const bool past = codes_past_cache(rows, gk);
    uint8_t* s_byte = reinterpret_cast<uint8_t*>(s) + ((((chunk * NC) >> 5) * 2u + (j & 1u)) * (NC >= 4u ? 32u : 16u) + ((chunk * NC) & 31u)) * 4u + (j >> 1);
#define REQUANT_COLUMN(C, V)                                                                            \
    {                                                                                                   \
        if (BIG) rotate_block_lanes(V, j, p.nb);                                                        \
        else fwht32(V);                                                                                 \
        uint4 q;                                                                                        \
        uint32_t sb, m;                                                                                 \
        encode_group<MODE>(V, p, stream, q_base, q, sb, m);                                              \
        s_byte[(C) * 4u] = (uint8_t)sb;                                                                 \
        if (r0 + (C) < rows && grp < gk) store_codes(dst_codes, q, past);                               \
        q_base += k >> 4;                                                                               \
        dst_codes += k >> 1;                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
// Columns 2 P and 2 P + 1 of the lane's chunk sit in one byte of its words, and one instruction decodes both.  Keeping the second's
// 32 values while the first is quantized takes more than 128 registers (a fourth wave per SIMD) with Philox (PARK: 20 of them
// wait in LDS; this kernel is bound by vector-ALU issue) and with the lanes of a wide Hadamard block (AGAIN: decoded twice).
#define REQUANT_DECODE(P, FIRST, SECOND)                                                                \
    _Pragma("unroll") for (uint32_t i4 = 0; i4 < 8; ++i4) {                                             \
        const float4 s4 = my_scales[i4];                                                                \
        const float sc[4] = {s4.x, s4.y, s4.z, s4.w};                                                   \
        _Pragma("unroll") for (uint32_t e = 0; e < 4; ++e) {                                            \
            const v2f a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4u * i4 + e], sc[e], P);           \
            FIRST[4u * i4 + e] = a[0];                                                                  \
            SECOND[4u * i4 + e] = a[1];                                                                 \
        }                                                                                               \
    }                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);
#define REQUANT_PAIR(P)                                                                                 \
    if (2u * (P) < NC) {                                                                                \
        float v0[32], v1[32];                                                                           \
        REQUANT_DECODE(P, v0, v1)                                                                       \
        if (PARK) {                                                                                     \
            _Pragma("unroll") for (uint32_t i = 0; i < 20; ++i) parked[64u * i] = v1[i];                \
            asm volatile("" ::: "memory");                                                              \
            __builtin_amdgcn_sched_barrier(0);                                                          \
        }                                                                                               \
        REQUANT_COLUMN(2u * (P), v0)                                                                    \
        if (PARK) {                                                                                     \
            asm volatile("" ::: "memory");                                                              \
            _Pragma("unroll") for (uint32_t i = 0; i < 20; ++i) v1[i] = parked[64u * i];                \
        }                                                                                               \
        if (AGAIN) {                                                                                    \
            _Pragma("unroll") for (uint32_t i = 0; i < 32; ++i) asm volatile("" : "+v"(w[i]));          \
            REQUANT_DECODE(P, v0, v1)                                                                   \
        }                                                                                               \
        REQUANT_COLUMN(2u * (P) + 1u, v1)                                                               \
    }
    constexpr bool AGAIN = BIG, PARK = !BIG && MODE == kBwdSr && NC == 8u;
    float* parked = static_cast<float*>(lds) + 4u * 16u * SROW + wave * 20u * 64u + lane;
    static_assert(!PARK || 4u * 16u * SROW * 4u + 4u * 5u * 1024u <= 8u * kquad_pitch<B>(), "the parked values must fit behind the scales");
    __builtin_amdgcn_sched_barrier(0);
    REQUANT_PAIR(0)
    REQUANT_PAIR(1)
    REQUANT_PAIR(2)
    REQUANT_PAIR(3)
#undef REQUANT_PAIR
#undef REQUANT_DECODE
#undef REQUANT_COLUMN
    __builtin_amdgcn_wave_barrier();
    if (NC == 8u) {
        store_kquad_scales<32u>(s, scales, c0, rows, grp0, gk, lane);
        store_kquad_scales<32u>(s + 64, scales, c0 + 32u, rows, grp0, gk, lane);
    } else {
        store_kquad_scales<8u * (NC == 8u ? 4u : NC)>(s, scales, c0, rows, grp0, gk, lane);
    }
}

// SHARED: the grid's first dimension is the K-quads, rounded up to a multiple of 8 (see launch_requant_big); otherwise the columns
template <int MODE, bool BIG, uint32_t NC, bool SHARED>
__global__ void __launch_bounds__(256, 4)
requant_transposed_kernel(const uint8_t* __restrict__ src_codes, const uint8_t* __restrict__ src_scales,
                          uint32_t rows, uint32_t k, uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                          SrParams p) {
    __shared__ __align__(16) uint8_t stage[NC == 2u ? 9216u : 8u * kquad_pitch<16u * NC>()];
    __shared__ uint32_t s_scale[64u * NC];
    const uint32_t kq = SHARED ? blockIdx.x : blockIdx.y, column = SHARED ? blockIdx.y : blockIdx.x;
    if (SHARED && kq >= (k + 255u) >> 8) return;
    requant_columns_block<MODE, BIG, NC>(src_codes, src_scales, rows, k, codes, scales, p, p.stream_id, kq, column * 32u * NC, stage, s_scale);
}

// ------------------------------------------------------------------ the backward pass's operand conversions in one launch
// dy^T quantized along the tokens, X_q and W_q re-quantized along their other dimension, and optionally dy itself along out:
// Algorithm 1 Backward needs all of them before the two gradient products and none depends on another.  Launched one after the
// other, the re-quantizers leave most of the chip idle on weight-sized tensors and every kernel pays its own ramp-up and
// drain.  In one grid the re-quantizer blocks come first (W_q's, then X_q's) and the dy^T tiles fill the CUs as those finish.
// (Spreading the re-quantizer blocks evenly among the tiles was measured slower than launching the kernels one by one: it
// breaks up the order in which neighbouring tiles write their lines.)
struct BwdOperandsMap {
    uint32_t n_rq_w, n_rq;           // re-quantizer blocks of W_q, and of W_q and X_q together: block indices [0, n_rq)
    uint32_t t_gx, t_gy;             // dy^T tiles: K-quads, column tiles
    uint32_t quads;                  // re-quantizer blocks along the columns (of W_q and of X_q: both have `in` columns)
    FastDiv div_t_gx, div_quads;
    uint32_t n_tiles_end;            // blocks [n_rq, n_tiles_end): dy^T tiles; blocks from n_tiles_end on: row tiles of dy (optional)
    uint32_t r_k_blocks;             // row tiles per 8 rows of dy
    FastDiv div_r_k_blocks;
};

// one re-quantized matrix of the launch
struct RequantMatrix {
    const uint8_t* src_codes;
    const uint8_t* src_scales;
    uint32_t rows, k;
    uint8_t* codes;
    uint8_t* scales;
    uint32_t stream_id;
};

// CPL, NC: columns per lane of the dy^T tile and of the re-quantizer waves (less work per wave for smaller problems).
// p: the parameters of all four conversions but for the Philox stream.  Each kind of block is inlined once (W_q's and X_q's
// blocks share one copy: with one each the kernel outgrew the 64 KB instruction cache).
template <int MODE, bool BIG, uint32_t CPL, uint32_t NC>
__global__ void __launch_bounds__(256, 4)
bwd_operands_kernel(const uint16_t* __restrict__ dy, uint32_t t_rows, uint32_t t_k, int64_t t_ldx,
                    uint8_t* __restrict__ t_codes, uint8_t* __restrict__ t_scales, uint32_t t_stream, RequantMatrix w, RequantMatrix x,
                    uint4* __restrict__ r_codes, uint8_t* __restrict__ r_scales, uint32_t r_stream, SrParams p, BwdOperandsMap map) {
    constexpr bool WIDE_TILE = !BIG && CPL == 2u;
    constexpr uint32_t B = 64u * CPL > 16u * NC ? 64u * CPL : 16u * NC;
    __shared__ __align__(16) uint8_t smem[8u * kquad_pitch<B>()];
    __shared__ uint32_t s_scale[64u * (NC > CPL ? NC : CPL)];
    static_assert(sizeof(smem) >= 4 * 256 * 16 && sizeof(s_scale) >= 64 * 4, "the row tile's staging must fit");
    static_assert(!WIDE_TILE || (sizeof(smem) >= 128 * 8 * 16 && sizeof(s_scale) >= 128 * 8), "the dy^T tile's staging must fit");
    const uint32_t b = blockIdx.x;
    if (b < map.n_rq) {
        const bool is_w = b < map.n_rq_w;
        const RequantMatrix& m = is_w ? w : x;
        const uint32_t i = is_w ? b : b - map.n_rq_w;
        const uint32_t kq = fast_div(i, map.div_quads), quad = i - kq * map.quads;
        requant_columns_block<MODE, BIG, NC>(m.src_codes, m.src_scales, m.rows, m.k, m.codes, m.scales, p, m.stream_id, kq, quad * 32u * NC, smem, s_scale);
    } else if (b >= map.n_tiles_end) {
        // Q(dy) in row mode (the first operand of the dx product), for callers that want all four conversions in one launch:
        // dy is [t_k x t_rows] row-major, groups along its rows
        quant_row_tile<MODE, false, BIG>(dy, t_k, t_rows >> 5, t_ldx, r_codes, r_scales, nullptr, p, r_stream, map.r_k_blocks,
                                         map.div_r_k_blocks, b - map.n_tiles_end, reinterpret_cast<uint4 (*)[256]>(smem), s_scale);
    } else {
        const uint32_t tb = b - map.n_rq;
        const uint32_t by = fast_div(tb, map.div_t_gx), bx = tb - by * map.t_gx;
        const uint32_t ct = transposed_column_tile(bx, by, map.t_gy);
        if (WIDE_TILE)
            quant_transposed_tile<MODE, false>(dy, t_rows, t_k, t_ldx, t_codes, t_scales, nullptr, p, t_stream, bx, ct,
                                               reinterpret_cast<uint4*>(smem), reinterpret_cast<uint8_t*>(s_scale), nullptr);
        else
            quant_columns_block<MODE, false, BIG, CPL, CPL == 2u>(dy, t_rows, t_k, t_ldx, t_codes, t_scales, nullptr, p, t_stream, bx, ct * 32u * CPL,
                                                       smem, s_scale);
    }
}

// ------------------------------------------------------------------ MXFP4 -> fp32
__global__ void __launch_bounds__(256)
dequant_kernel(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales, uint32_t n_groups,
               uint32_t gk, FastDiv div_gk, float* __restrict__ out) {
    uint32_t g = blockIdx.x * 256u + threadIdx.x;
    if (g >= n_groups) return;
    uint4 q = reinterpret_cast<const uint4*>(codes)[g];
    const uint32_t row = fast_div(g, div_gk), gi = g - row * gk;
    float s = u2f((uint32_t)scales[scale_tile_offset(row, gi, (gk + 7u) >> 3)] << 23);
    uint32_t w[4] = {q.x, q.y, q.z, q.w};
    float4* dst = reinterpret_cast<float4*>(out + (size_t)g * 32u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v2f a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], s, 0);
        v2f b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], s, 1);
        v2f c = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], s, 2);
        v2f d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], s, 3);
        dst[2 * i] = make_float4(a[0], a[1], b[0], b[1]);
        dst[2 * i + 1] = make_float4(c[0], c[1], d[0], d[1]);
    }
}

// ------------------------------------------------------------------ host-side launchers

template <int MODE, bool MASK>
static void launch_row_big(bool big, dim3 grid, hipStream_t st, const void* x, int64_t rows, uint32_t gk, int64_t ldx,
                           uint8_t* codes, uint8_t* scales, uint32_t* mask, const SrParams& p, uint32_t k_blocks) {
    dim3 block(256);
    if (big)
        hipLaunchKernelGGL((quant_row_kernel<MODE, MASK, true>), grid, block, 0, st, (const uint16_t*)x, (uint32_t)rows,
                           gk, ldx, (uint4*)codes, scales, mask, p, k_blocks, make_fast_div(k_blocks));
    else
        hipLaunchKernelGGL((quant_row_kernel<MODE, MASK, false>), grid, block, 0, st, (const uint16_t*)x, (uint32_t)rows,
                           gk, ldx, (uint4*)codes, scales, mask, p, k_blocks, make_fast_div(k_blocks));
}

template <int MODE>
static hipError_t launch_row(const void* x, int64_t rows, int64_t k, int64_t ldx, uint8_t* codes,
                             uint8_t* scales, uint32_t* mask, const SrParams& p, hipStream_t st) {
    if (rows == 0 || k == 0) return hipSuccess;
    const uint32_t gk = (uint32_t)(k / 32);
    const uint32_t k_blocks = (gk + 31) / 32;
    dim3 grid((uint32_t)((rows + 7) / 8) * k_blocks);
    if (mask) launch_row_big<MODE, true>(p.nb > 1u, grid, st, x, rows, gk, ldx, codes, scales, mask, p, k_blocks);
    else launch_row_big<MODE, false>(p.nb > 1u, grid, st, x, rows, gk, ldx, codes, scales, mask, p, k_blocks);
    return hipGetLastError();
}

// Columns per lane of the re-quantizer waves for a launch that converts `elements` values transposed.  A wave quantizes its columns
// one after the other, 1-1.5 us each, so while the whole launch is shorter than eight of them the waves take fewer columns; fewer
// columns also mean shorter pieces of the source rows (128, 64, 32 bytes), which cost memory efficiency once the chip is full.
// Measured (us, all four conversions of a layer, 8 / 4 / 2 columns, stochastic): 256 x 512 x 512 11.5 / 7.5 / 5.4; 2048^3 (16 M
// elements) 12.5 / 8.9 / 9.1; 4096 x 4096 x 1024 (25 M) 22.9 / 17.6 / 18.5; 8192 x 2048 x 2048 (38 M) 30.0 / 31.4 / -;
// 4096^3 (50 M) 37 / 38 / -.
static uint32_t requant_columns(uint64_t elements) {
    return elements >= ((uint64_t)32 << 20) ? 8u : elements >= ((uint64_t)10 << 20) ? 4u : 2u;
}

template <int MODE, bool MASK>
static void launch_transposed_nb(const void* src, int64_t rows, int64_t k, int64_t ldx, uint8_t* codes, uint8_t* scales,
                                 uint32_t* mask, const SrParams& p, hipStream_t st) {
    const uint32_t kquads = (uint32_t)((k / 32 + 7) / 8);
    const uint16_t* s = (const uint16_t*)src;
    // Blocks of 32 columns (half the work) while the matrix is too small to fill the chip: up to two of their 256 x 32 waves per SIMD where
    // the K-quads are a multiple of 8, 1.25 of them elsewhere.  They read half lines.  The blocks of one K-quad lie kquads apart
    // in the launch and blocks go to the XCDs in turn, so with a multiple of 8 both halves of a line are read through one L2; otherwise
    // every line crosses from memory twice.  32 columns against the wider block (us, nearest): multiple of 8: 2048 x 5984 (1496 waves)
    // 6.2 / 7.9, 4096 x 4096 (2048) 7.1 / 7.8; not: 1664 x 5728 (1253) 7.0 / 8.5, 2784 x 4128 (1419) 10.4 / 9.0, 5536 x 2560 (1760)
    // 12.0 / 9.1, 1536 x 10048 (1884) 11.7 / 7.9.
    const uint64_t waves = (uint64_t)kquads * (uint64_t)((rows + 31) / 32);
    const bool small = waves < ((kquads & 7u) == 0u ? 2048u : 1280u);
    // Wide Hadamard blocks, 64 columns: where rows or base are not whole lines, two neighbouring blocks share a line in every row.  Once
    // the matrix no longer fits the caches beside its result they have to meet in one L2: K-quads rounded up to a multiple of 8, and
    // loads that may stay there (us, blocks of 64, forward / nearest / stochastic, so and as otherwise: 13952 x 7968 54 / 46 / 53, 91 / 81 / 87;
    // 5376 x 8864, 5817 waves, 29.0 / 26.6 / 28.4, 32.7 / 29.5 / 31.2; 4608 x 7328, 4122 waves, 22 / 21 / 24, 24 / 21 / 23; aligned rows,
    // 3072 x 10944, 23 / 19 / 24, 20 / 17 / 20).
    const bool shared_lines = !small && p.nb > 1u && ((reinterpret_cast<uintptr_t>(src) | (uintptr_t)(ldx * 2)) & 127u) != 0 && waves >= 5000u;
#define QUARTET_COLUMNS(CPL, BIG, STREAM, GRID_K)                                                                                 \
    hipLaunchKernelGGL((quant_columns_kernel<MODE, MASK, BIG, CPL, STREAM>), dim3(GRID_K, (uint32_t)((rows + 32 * CPL - 1) / (32 * CPL))), \
                       dim3(256), 0, st, s, (uint32_t)rows, (uint32_t)k, ldx, codes, scales, mask, p)
    if (p.nb > 1u) {
        if (small) QUARTET_COLUMNS(1, true, false, kquads);
        else if (shared_lines) QUARTET_COLUMNS(2, true, false, (kquads + 7u) & ~7u);
        else QUARTET_COLUMNS(2, true, true, kquads);
    } else if (small) {
        QUARTET_COLUMNS(1, false, false, kquads);
    } else {
        hipLaunchKernelGGL((quant_transposed_kernel<MODE, MASK>), dim3(kquads, (uint32_t)((rows + 127) / 128)), dim3(256), 0, st, s,
                           (uint32_t)rows, (uint32_t)k, ldx, codes, scales, mask, p);
    }
#undef QUARTET_COLUMNS
}

template <int MODE>
static hipError_t launch_transposed(const void* src, int64_t rows, int64_t k, int64_t ldx, uint8_t* codes,
                                    uint8_t* scales, uint32_t* mask, const SrParams& p, hipStream_t st) {
    if (rows == 0 || k == 0) return hipSuccess;
    constexpr bool CAN_MASK = MODE == kFwd;           // the backward rules never clip
    if (CAN_MASK && mask) launch_transposed_nb<MODE, CAN_MASK>(src, rows, k, ldx, codes, scales, mask, p, st);
    else launch_transposed_nb<MODE, false>(src, rows, k, ldx, codes, scales, nullptr, p, st);
    return hipGetLastError();
}

hipError_t launch_quant(int mode, const void* x, int64_t rows, int64_t k, int64_t ldx, int transpose,
                        const SrParams& p, uint8_t* codes, uint8_t* scales, uint32_t* mask, hipStream_t st) {
    if (!transpose) {
        switch (mode) {
        case kFwd: return launch_row<kFwd>(x, rows, k, ldx, codes, scales, mask, p, st);
        case kBwdRtn: return launch_row<kBwdRtn>(x, rows, k, ldx, codes, scales, nullptr, p, st);
        default: return launch_row<kBwdSr>(x, rows, k, ldx, codes, scales, nullptr, p, st);
        }
    }
    switch (mode) {
    case kFwd: return launch_transposed<kFwd>(x, rows, k, ldx, codes, scales, mask, p, st);
    case kBwdRtn: return launch_transposed<kBwdRtn>(x, rows, k, ldx, codes, scales, nullptr, p, st);
    default: return launch_transposed<kBwdSr>(x, rows, k, ldx, codes, scales, nullptr, p, st);
    }
}

template <int MODE, bool BIG>
static void launch_requant_big(const uint8_t* src_codes, const uint8_t* src_scales, int64_t rows, int64_t k, const SrParams& p,
                               uint8_t* codes, uint8_t* scales, hipStream_t st) {
    const uint32_t nc = requant_columns((uint64_t)rows * (uint64_t)k), kquads = (uint32_t)((k + 255) / 256);
    const uint32_t columns = (uint32_t)((rows + 32 * nc - 1) / (32 * nc));
    // Where the rows of codes or their base are not whole lines, two neighbouring blocks share a line in every row: with the K-quads first
    // and a multiple of 8 of them they run on one XCD and its L2 serves both (see launch_transposed_nb).  Blocks of 128 bytes of a
    // row and 16 K-quads or more (us, stochastic / nearest, so and columns first: 6144 x 8640 30.6 / 21.6, 32.4 / 23.2; 13568 x 3968 32.6 /
    // 21.7, 33.5 / 23.1; 9 K-quads, 2112 x 8160, 17.1 / 12.0, 14.0 / 10.3; whole lines, 16384 x 11008, 75 / 46.3, 74 / 46.1).
    const bool shared_lines = nc == 8u && kquads >= 16u && columns <= 65535u && ((reinterpret_cast<uintptr_t>(src_codes) | (uintptr_t)(rows / 2)) & 127u) != 0;
#define QUARTET_REQUANT(NC, SHARED, X, Y)                                                                                         \
    hipLaunchKernelGGL((requant_transposed_kernel<MODE, BIG, NC, SHARED>), dim3(X, Y), dim3(256), 0, st, src_codes, src_scales,    \
                       (uint32_t)rows, (uint32_t)k, codes, scales, p)
    if (shared_lines) QUARTET_REQUANT(8, true, (kquads + 7u) & ~7u, columns);
    else if (nc == 8u) QUARTET_REQUANT(8, false, columns, kquads);
    else if (nc == 4u) QUARTET_REQUANT(4, false, columns, kquads);
    else QUARTET_REQUANT(2, false, columns, kquads);
#undef QUARTET_REQUANT
}

hipError_t launch_requant_transpose(int mode, const uint8_t* src_codes, const uint8_t* src_scales,
                                    int64_t rows, int64_t k, const SrParams& p, uint8_t* codes,
                                    uint8_t* scales, hipStream_t st) {
    if (rows == 0 || k == 0) return hipSuccess;
    if (mode == kBwdRtn) {
        if (p.nb > 1u) launch_requant_big<kBwdRtn, true>(src_codes, src_scales, rows, k, p, codes, scales, st);
        else launch_requant_big<kBwdRtn, false>(src_codes, src_scales, rows, k, p, codes, scales, st);
    } else {
        if (p.nb > 1u) launch_requant_big<kBwdSr, true>(src_codes, src_scales, rows, k, p, codes, scales, st);
        else launch_requant_big<kBwdSr, false>(src_codes, src_scales, rows, k, p, codes, scales, st);
    }
    return hipGetLastError();
}

hipError_t launch_fwd_operands(const void* x, int64_t tokens, const void* w, int64_t out, int64_t in, uint8_t* xq_codes,
                               uint8_t* xq_scales, uint32_t* x_mask, uint8_t* wq_codes, uint8_t* wq_scales, uint32_t* w_mask,
                               const SrParams& p, hipStream_t st) {
    if (in == 0 || (tokens == 0 && out == 0)) return hipSuccess;
    const uint32_t gk = (uint32_t)(in / 32);
    const uint32_t k_blocks = (gk + 31) / 32;
    const uint64_t na = (uint64_t)((tokens + 7) / 8) * k_blocks, nb = (uint64_t)((out + 7) / 8) * k_blocks;
    if (na + nb >= ((uint64_t)1 << 31)) return hipErrorInvalidValue;
    RowMatrix a = {(const uint16_t*)x, (uint32_t)tokens, in, (uint4*)xq_codes, xq_scales, x_mask};
    RowMatrix b = {(const uint16_t*)w, (uint32_t)out, in, (uint4*)wq_codes, wq_scales, w_mask};
    // a and b from block 0 on, or b alone (split 0)
    auto launch = [&](uint64_t blocks, uint64_t split) {
        if (p.nb > 1u)
            hipLaunchKernelGGL((quant_row_pair_kernel<kFwd, true, true>), dim3((uint32_t)blocks), dim3(256), 0, st, a, b, (uint32_t)split,
                               gk, p, k_blocks, make_fast_div(k_blocks));
        else
            hipLaunchKernelGGL((quant_row_pair_kernel<kFwd, true, false>), dim3((uint32_t)blocks), dim3(256), 0, st, a, b, (uint32_t)split,
                               gk, p, k_blocks, make_fast_div(k_blocks));
        return hipGetLastError();
    };
    // a launch holds fewer than 2^32 threads: where the two matrices together have more, each has its own
    if (na == 0 || nb == 0 || na + nb < ((uint64_t)1 << 24)) return launch(na + nb, na);
    const hipError_t e = launch(na, na);
    return e == hipSuccess ? launch(nb, 0) : e;
}

hipError_t launch_bwd_operands(int mode, const void* dy, int64_t tokens, int64_t in, int64_t out,
                               const uint8_t* xq_codes, const uint8_t* xq_scales, const uint8_t* wq_codes, const uint8_t* wq_scales,
                               const SrParams& p_dyt, const SrParams& p_x, const SrParams& p_w,
                               uint8_t* dyt_codes, uint8_t* dyt_scales, uint8_t* xt_codes, uint8_t* xt_scales,
                               uint8_t* wt_codes, uint8_t* wt_scales,
                               const SrParams& p_dy, uint8_t* dy_codes, uint8_t* dy_scales, hipStream_t st) {
    BwdOperandsMap map;
    const uint32_t kq_t = (uint32_t)((tokens + 255) / 256), kq_o = (uint32_t)((out + 255) / 256);
    const SrParams& p = p_dyt;        // the four differ in the Philox stream alone
    const bool big = p.nb > 1u;
    const uint32_t nc = requant_columns((uint64_t)tokens * (uint64_t)out + (uint64_t)in * (uint64_t)(tokens + out));
    const int64_t t_cols = nc == 8u ? (big ? 64 : 128) : 32, q_cols = 32 * nc;
    // dy^T: logical [out x tokens]; X_q^T: [in x tokens] from [tokens x in]; W_q^T: [in x out] from [out x in].
    // An empty dimension empties the conversions it belongs to, not the others.
    map.t_gx = kq_t;
    map.t_gy = (uint32_t)((out + t_cols - 1) / t_cols);
    map.quads = (uint32_t)((in + q_cols - 1) / q_cols);
    map.n_rq_w = map.quads * kq_o;
    map.n_rq = map.n_rq_w + map.quads * kq_t;
    uint64_t total = (uint64_t)map.t_gx * map.t_gy + map.n_rq;
    if (total >= ((uint64_t)1 << 31)) return hipErrorInvalidValue;
    map.n_tiles_end = (uint32_t)total;
    // optional fourth conversion: dy [tokens x out] in row mode, 8 rows x 1024 columns per block
    map.r_k_blocks = (uint32_t)((out / 32 + 31) / 32);
    if (dy_codes) total += (uint64_t)((tokens + 7) / 8) * map.r_k_blocks;
    if (total == 0) return hipSuccess;
    if (total >= ((uint64_t)1 << 31)) return hipErrorInvalidValue;
    map.div_t_gx = make_fast_div(map.t_gx ? map.t_gx : 1u);
    map.div_quads = make_fast_div(map.quads ? map.quads : 1u);
    const RequantMatrix w = {wq_codes, wq_scales, (uint32_t)in, (uint32_t)out, wt_codes, wt_scales, p_w.stream_id};
    const RequantMatrix x = {xq_codes, xq_scales, (uint32_t)in, (uint32_t)tokens, xt_codes, xt_scales, p_x.stream_id};
    map.div_r_k_blocks = make_fast_div(map.r_k_blocks ? map.r_k_blocks : 1u);
#define QUARTET_BWD_OPERANDS(MODE, BIG, CPL, NC)                                                                                  \
    hipLaunchKernelGGL((bwd_operands_kernel<MODE, BIG, CPL, NC>), dim3((uint32_t)total), dim3(256), 0, st, (const uint16_t*)dy,    \
                       (uint32_t)out, (uint32_t)tokens, out, dyt_codes, dyt_scales, p_dyt.stream_id, w, x,                         \
                       reinterpret_cast<uint4*>(dy_codes), dy_scales, p_dy.stream_id, p, map)
#define QUARTET_BWD_OPERANDS_SIZE(MODE, BIG)                                                                                      \
    do {                                                                                                                          \
        if (nc == 8u) QUARTET_BWD_OPERANDS(MODE, BIG, 2, 8);                                                                      \
        else if (nc == 4u) QUARTET_BWD_OPERANDS(MODE, BIG, 1, 4);                                                                 \
        else QUARTET_BWD_OPERANDS(MODE, BIG, 1, 2);                                                                               \
    } while (0)
    if (mode == kBwdRtn) { if (big) QUARTET_BWD_OPERANDS_SIZE(kBwdRtn, true); else QUARTET_BWD_OPERANDS_SIZE(kBwdRtn, false); }
    else { if (big) QUARTET_BWD_OPERANDS_SIZE(kBwdSr, true); else QUARTET_BWD_OPERANDS_SIZE(kBwdSr, false); }
#undef QUARTET_BWD_OPERANDS_SIZE
#undef QUARTET_BWD_OPERANDS
    return hipGetLastError();
}

hipError_t launch_dequant(const uint8_t* codes, const uint8_t* scales, int64_t rows, int64_t k, float* out,
                          hipStream_t st) {
    uint64_t n_groups = (uint64_t)rows * (uint64_t)(k / 32);
    if (n_groups == 0) return hipSuccess;
    dim3 grid((uint32_t)((n_groups + 255) / 256)), block(256);
    hipLaunchKernelGGL(dequant_kernel, grid, block, 0, st, codes, scales, (uint32_t)n_groups, (uint32_t)(k / 32),
                       make_fast_div((uint32_t)(k / 32)), out);
    return hipGetLastError();
}

}  // namespace quartet
