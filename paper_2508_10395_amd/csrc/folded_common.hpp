// Shared pieces of the folded attention kernels (folded_attn.hip, folded_per_channel.hpp): the order in which operand slots hold channels and tokens, the unpacking of packed codes to
// normal fp16 numbers, the layout of the workspace.
//
// What they compute (Sec. 3.1 of arxiv 2508.10395, with the products taken in another order).  For a query row q of KV
// head h, K = X^ Wk_h and V = X^ Wv_h enter the attention only through
//     q K^T = (q Wk_h^T) X^T = u X^T        and        p V = (p X^) Wv_h = y Wv_h,
// so a decode step needs no key and no value: u (d numbers per query row) is formed once per sequence, the scores are
// products of u with the cached rows, y is the softmax-weighted sum of the cached rows, and Wv_h is applied to that sum.
// Per cached token and query row 4 d operations, against 4 d 128 per token and KV head when K and V are
// rematerialised: with one query per sequence 128 / (query heads per KV head) times fewer, and the step is bound by
// reading the cache and the weights instead of by the matrix cores' power draw.
//
// Precision.  u, the softmax weights times the scales, and y are fp32 numbers that enter the matrix cores as sums of
// fp16 parts (hi + lo, 22 bits, against integer codes that are exact in fp16) or of bf16 parts (hi + mid + lo, all 24
// bits, against bf16 rows or weights); products are accumulated in fp32.
#pragma once
#include "remat_common.hpp"

namespace xq {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// ---- query rows.  A sequence has one per query head; they are taken in blocks of 16 RT (RT = 1 or 2 MFMA row tiles).
constexpr int FOLD_TILE = 128;           // tokens of a score workgroup: unit of the stored softmax weights
constexpr int FOLD_VTILE = 256;          // tokens a value workgroup stages at a time

// one source of cached rows (the keys' or the values' side of a latent cache, or the whole X cache for both)
struct FoldSource {
    const uint8_t* codes;
    const uint16_t* scale;
    const uint16_t* zero;
    const uint16_t* rows;                // dense source: bf16 rows
    long long row_bytes;                 // between consecutive tokens of codes / rows
    int cap;                             // tokens between consecutive sequences
    int ng_row;                          // groups per row of scale / zero
    int meta_shift;                      // group g of the walk takes scale and zero-point g >> meta_shift
    int n_slabs, ng;                     // slabs of 128 walked channels, groups of the walk
};

// the prepared weight stream that belongs to a source (the first one, 32-column fragments, remat_layout.hpp): KV head h
// has the 128 columns of its keys (or values) in the column blocks [nb0, nb0 + 4) of stream head sh
struct FoldWeights {
    const uint8_t* stream;
    const int32_t* shift;                // per stream head; null for bf16 streams
    long long head_bytes;
    int n16;                             // k-steps of 16 channels
    int group;                           // group size the stream is laid out for
    int pair;                            // a stream head is a pair of KV heads
    int nibbles;                         // odd channels carry 16 times the weight of the even ones (8-bit caches)
};

// slot (tick, quarter, i) of a slab's 128 codes, as the score kernel's token operand holds them: a lane of quarter q
// holds 32 consecutive codes (groups of 128) or 16 consecutive codes of each group (groups of 64), taken as octets of
// 8; a tick's dword v pairs code 4 (tick & 1) + v of two adjacent octets
template <int G>
__host__ __device__ constexpr int fold_channel(int tick, int q, int i)
{
    const int v = i >> 1, hb = i & 1;
    return G == 128 ? 32 * q + 8 * (2 * (tick >> 1) + hb) + 4 * (tick & 1) + v
                    : 64 * (tick >> 1) + 16 * q + 8 * hb + 4 * (tick & 1) + v;
}

// bytes of a slab of folded queries of one row block
constexpr int FOLD_U_CODED(int rt) { return rt * (4 * 2 + 1) * 1024; }      // [rt][tick][hi, lo] then [rt] zero-point fragments
constexpr int FOLD_U_DENSE(int rt) { return rt * 4 * 3 * 1024; }            // [rt][tick][hi, mid, lo]

// ---- unpacking.  A pair of octets (8 codes each: BITS bytes) becomes 8 dwords of two fp16 numbers: dword k holds code k
// of either octet as the normal number (code - zi) 2^-9: the bits are masked into the mantissa under a zero exponent (a
// subnormal, exactly code 2^(o - 24) at bit offset o) and one packed fused multiply-add brings them to the common scale
// and takes the integer zi off, exactly.  Subnormals alone would do for the matrix cores, but these align products by
// exponent fields, and every leading zero of an operand is a bit of accumulation precision given away.
//
// zi is the integer zero-point of the code's (token, group): x^ = code s + z = (code - zi) s + (z + zi s) with
// zi = rint(-z / s) clamped to the codes.  In a group whose range an outlier sets, code s and z are some ten times the
// ordinary channels' values and cancel; (code - zi) and the remainder z + zi s (at most s / 2 where the range holds 0)
// do not, so the rounding of what multiplies them is not magnified.  For any zi the identity is exact.
constexpr float FOLD_CODE_UNIT = 512.0f;          // operand = (code - zi) / FOLD_CODE_UNIT

template <int BITS, int OFF>
__device__ __forceinline__ uint32_t fold_field(uint32_t x, uint32_t minus_zi)
{
    constexpr uint32_t M1 = ((1u << BITS) - 1u) << OFF;
    static_assert(OFF + BITS <= 10, "field inside the fp16 mantissa");
    const uint32_t t = x & (M1 | (M1 << 16));
    constexpr _Float16 up = (_Float16)(float)(1 << (15 - OFF));
    const xq_f16x2 mul = {up, up};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(xq_f16x2, t), mul, __builtin_bit_cast(xq_f16x2, minus_zi)));
}

// codes 0-7 of two octets from their merged halves: BITS 2: m0 = both 16-bit octets; BITS 3: m0 = bits 0-15 and m1 = bits
// 8-23 of both 24-bit octets; BITS 4: m0 = low and m1 = high halves of both 32-bit octets.  minus_zi: -zi 2^-9 of the two.
template <int BITS, int K>
__device__ __forceinline__ uint32_t fold_code(uint32_t m0, uint32_t m1, uint32_t minus_zi)
{
    if constexpr (BITS == 2) {
        if constexpr (K < 5) return fold_field<2, 2 * K>(m0, minus_zi);
        else return fold_field<2, 2 * K - 10>(m0 >> 10, minus_zi);
    } else if constexpr (BITS == 3) {
        if constexpr (K < 3) return fold_field<3, 3 * K>(m0, minus_zi);
        else if constexpr (K < 6) return fold_field<3, 3 * K - 8>(m1, minus_zi);
        else return fold_field<3, 3 * K - 18>(m1 >> 10, minus_zi);
    } else {
        const uint32_t m = K < 4 ? m0 : m1;
        constexpr int k = K & 3;
        if constexpr (k < 2) return fold_field<4, 4 * k>(m, minus_zi);
        else return fold_field<4, 4 * k - 8>(m >> 8, minus_zi);
    }
}

// integer zero-point of a (token, group) and what is left of its zero-point; qmax = largest code
__device__ __forceinline__ float fold_integer_zero(float s, float z, float qmax, float& rest)
{
    float zi = fminf(fmaxf(rintf(-z * __builtin_amdgcn_rcpf(s)), 0.0f), qmax);      // (NaN, from 0 inf, becomes 0)
    zi = s > 0.0f ? zi : 0.0f;
    rest = __builtin_fmaf(zi, s, z);
    return zi;
}
__device__ __forceinline__ uint32_t f16_bits(float v) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v); }

__device__ __forceinline__ uint32_t perm_bytes(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// exact split of an fp32 number into three bf16 parts (8 + 8 + 8 bits, by truncation): the upper halves of the results
__device__ __forceinline__ void split_bf16x3(float v, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = __float_as_uint(v) & 0xFFFF0000u;
    const float r1 = v - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xFFFF0000u;
    l = __float_as_uint(r1 - __uint_as_float(m));
}
__device__ __forceinline__ uint32_t pack_hi16(uint32_t a, uint32_t b) { return perm_bytes(b, a, 0x07060302u); }   // upper halves, a low

// workgroup order: the workgroups of one XCD (blockIdx % 8) get a contiguous range of the work, so that what neighbours
// share (a sequence's folded queries, its softmax weights) is fetched into one L2
__device__ __forceinline__ int xcd_contiguous(int n, int wg)
{
    const int per = (n + 7) >> 3;
    return (wg & 7) * per + (wg >> 3);
}
inline int xcd_grid(int n) { return (n + 7) / 8 * 8; }

}  // namespace xq
