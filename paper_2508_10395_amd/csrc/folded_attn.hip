// Decode attention without rematerialised keys and values (see folded_common.hpp for the algebra and the precision):
//   fold_query_kernel    u = q Wk_h^T for every query row, split and laid out as operand fragments of the score kernel
//   fold_scores_kernel   S = u X^T for 128 tokens a workgroup; softmax weights against the tile's maximum
//                        (fold_scores_digits_kernel, folded_digits.hpp: 2-bit codes on the f8f6f4 products, 256 tokens)
//   fold_values_kernel   y = sum over tokens of softmax weight times cached row, for a slab range and a token range
//   fold_output_kernel   o = y Wv_h, split over the channels
//   fold_finish_kernel   sum of these splits, divided by the softmax denominator
// Against rematerialising K and V tile by tile (MI355X, us per step with the append, before / after): 8 x 4096 tokens, 3 bits,
// 32 KV heads of a d = 4096 layer 1664 / 102; 16 x up to 8191, 2 bits in groups of 64, 32 on 8 heads 1512 / 192; 4 x 32768,
// 2 bits 6330 / 195; bf16 accumulator, 4 x up to 6000 1080 / 118.  The operations no longer bound it: what is left is the
// unpacking beside the matrix instructions, and 14 us each for reading the two halves of the weight stream.
#include <algorithm>

#include "folded_common.hpp"
#include "folded_attn.hpp"

namespace xq {

// What a launch sees of the problem: nb sequences starting at sequence b0 of the call.
struct FoldShape {
    int b0, nb, Hq, Hkv, R, nrb;         // query rows per sequence R = Hq, nrb row blocks of 16 RT rows
    int tiles;                           // score tiles (128 tokens) per sequence in the arrays, even
    int splits;                          // token splits in the arrays of the value kernel
    int block;                           // per-channel caches: tokens per block (else 0)
    int mhalf;                           // softmax weights and maxima per 128 tokens (0) or 64 (1: per-channel blocks of 64)
    BatchI32 len;                        // of the call's sequences
    int dealt;                           // score and value workgroups take the launch's sequences in the order below (else as they come)
    uint8_t order[XQ_MAX_BATCH];
};
static_assert(XQ_MAX_BATCH <= 256, "a sequence's number in a byte");
__device__ __forceinline__ int fold_sequence(const FoldShape& s, int k) { return s.dealt ? __builtin_amdgcn_readfirstlane((int)s.order[k]) : k; }

// The tokens a workgroup may take and where their tiles lie.  A per-channel cache's complete blocks come first, its window
// has the tiles behind them (from an even one on) and the last split; it is the work of the first workgroups of a launch.
struct FoldSpan { int len, tile0; };
__device__ __forceinline__ FoldSpan fold_span(const FoldShape& s, int b, bool window)
{
    const int len = s.len.v[s.b0 + b];
    if (s.block == 0) return {len, 0};
    const int coded = len / s.block * s.block;
    return window ? FoldSpan{len - coded, (coded + FOLD_VTILE - 1) / FOLD_VTILE * 2} : FoldSpan{coded, 0};
}
// splits of a sequence that hold tokens: the first `used` ones, and the last one if `window`
__device__ __forceinline__ void fold_used_splits(const FoldShape& s, int b, int& used, bool& window)
{
    const int len = s.len.v[s.b0 + b], coded = s.block ? len / s.block * s.block : len, splits = s.block ? s.splits - 1 : s.splits;
    const int nt = (coded + FOLD_VTILE - 1) / FOLD_VTILE, per = max(1, (nt + splits - 1) / splits);
    used = (nt + per - 1) / per;
    window = len > coded;
}

// element positions inside a fragment block of the softmax weights: [tile32][rt][part 2][lane 64][4 fp32], token
// 4 i + q of the 32 is slot i of quarter q (rows of four adjacent tokens are read by one load of the value kernel)
template <int RT>
constexpr int FOLD_P_TILE32 = RT * 2 * 256;      // floats per 32 tokens

// =====================================================================================================================
// Folded queries.  A wave owns one slab (128 channels) of one KV head and 32 query columns (sequence, query token, query
// head of the KV head).  The prepared stream holds the weights with 32 output columns along the lanes, contraction index
// inside the lane -- right for x W, but here the contraction runs over the output columns.  The matrix cores transpose:
// a product with a selection matrix gives every fragment's 16 channels as fp32 accumulator columns (exactly: one product
// with 1 each), whose registers, cut to bf16 (exactly: the weights are bf16 numbers times a power of two), are the
// operand of the product with the query rows.  The slab of u goes through LDS in natural channel order and leaves as
// operand fragments of the score kernel.  Bound by reading the key half of the stream once.
// =====================================================================================================================
struct FoldQueryArgs {
    FoldWeights w;
    FoldShape s;
    const uint16_t* q;                   // [B][Hq][128]
    uint8_t* u;                          // [nb][nrb][n_slabs][u_slab]
    float* rowfac;                       // [nb][nrb 16 RT]
    float scale_log2e;
    int u_slab, n_slabs, rt;
    UnpackTable tab;                     // coded streams: channel of every slot of the stream
    uint8_t* u_dense;                    // per-channel caches: the same u for the window's bf16 rows, or null
};

// channel inside its slab of slot (half, i) of k-step ks of the slab, in the first prepared stream; code: tab.code_of_slot[ks & 3][i]
__device__ __forceinline__ int stream_channel(int group, int ks, int half, int code)
{
    const int ksg_n = group >> 4, gi = ks / ksg_n, ksg = ks % ksg_n;
    return gi * group + half * (group >> 1) + (ksg >> 2) * 32 + code;
}

constexpr int FQ_STRIDE = 132;           // floats per query column in LDS: 16-byte pieces of different columns on different banks

// u of a slab in base-32 digits (folded_digits.hpp)
constexpr float FOLD_WIDE_ROWS = 8.0f;
template <int G>
__device__ __forceinline__ void fold_store_digits(const FoldQueryArgs& a, const float* mine, const int* place, int lane, int slab, bool wide_rows);

template <bool DENSE, int G, bool DIGITS = false>
__global__ __launch_bounds__(128) void fold_query_kernel(const FoldQueryArgs a)
{
    __shared__ __attribute__((aligned(16))) float ul[2][32 * FQ_STRIDE];
    __shared__ float nrm[2][32];
    __shared__ __attribute__((aligned(4))) int8_t table[2][64];      // coded streams: code_of_slot, then wexp_of_code
    __shared__ int place[2][32];             // row block of the launch 16 RT + row inside it, per column (-1: none)
    __shared__ float row_tops[2][DIGITS ? 128 : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int half = lane >> 5, c32 = lane & 31;
    const int slab = blockIdx.x * 2 + wave, h = blockIdx.y, cb = blockIdx.z;
    if (slab >= a.n_slabs) return;                                  // (no workgroup barrier below: a wave's LDS is its own)
    const FoldShape& s = a.s;
    const int gq = s.Hq / s.Hkv, ncol = s.nb * gq;
    float* mine = ul[wave];
    // column -> (sequence of the launch, row of the sequence)
    auto row_of = [&](int col, int& b) -> int {
        b = col / gq;
        return h * gq + (col - b * gq);
    };

    const int rpb = 16 * a.rt;
    if (half == 0) {
        int b;
        const int row = row_of(min(cb * 32 + c32, ncol - 1), b), rb = row / rpb;
        place[wave][c32] = cb * 32 + c32 < ncol ? (b * s.nrb + rb) * rpb + (row - rb * rpb) : -1;
    }

    const int sh = a.w.pair ? h >> 1 : h, nb0 = a.w.pair ? 4 * (h & 1) : 0, shift = DENSE ? 0 : a.w.shift[sh];
    // the 32 query rows as an operand: lane = column, k-slots in the order the accumulator rows below come in
    uint4 qa[4][2];
    float l1 = 0.0f;
    {
        int b;
        const int row = row_of(min(cb * 32 + c32, ncol - 1), b);
        const uint16_t* qv = a.q + ((long long)(s.b0 + b) * s.R + row) * 128 + 4 * half;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint2 x = *reinterpret_cast<const uint2*>(qv + 32 * nb + 16 * k);
                const uint2 y = *reinterpret_cast<const uint2*>(qv + 32 * nb + 16 * k + 8);
                qa[nb][k] = make_uint4(x.x, x.y, y.x, y.y);
            }
    }
    // Every weight fragment of the wave's slab is asked for before anything is waited for (2 waves in flight on a SIMD at most,
    // 32 loads each), and no load comes behind them: 34 MB of 8 x 4096 tokens, d = 4096, 16.2 us with eight at a time, 15.8 with byte
    // loads of the tables behind them, 13.6 now (weights already in the Infinity Cache: 12.0, 13.3, 12.3).
    const uint8_t* wsrc = a.w.stream + (long long)sh * a.w.head_bytes + lane * 16;
    uint4 wf[4][4][2];
#pragma unroll
    for (int pr = 0; pr < 4; ++pr)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                // coded streams: column block nb runs 7 - nb k-steps late, cyclically
                int pos = slab * 8 + 2 * pr + k + (DENSE ? 0 : COL_BLOCK_LAG_MAX - (nb0 + nb));
                if (pos >= a.w.n16) pos -= a.w.n16;
                wf[pr][nb][k] = *reinterpret_cast<const uint4*>(wsrc + (long long)pos * 8192 + (nb0 + nb) * 1024);
            }
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t w4[4] = {qa[nb][k].x, qa[nb][k].y, qa[nb][k].z, qa[nb][k].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) l1 += fabsf(bf16_lo_to_f32(w4[i])) + fabsf(bf16_hi_to_f32(w4[i]));
        }
    l1 += __shfl_xor(l1, 32);
    // Coded streams: code index and exponent of the lane's slot, of even and odd pairs of k-steps.  The tables come by scalar loads
    // and are looked up in LDS: a vector load behind the weights would wait for all of them.
    int slot_code[2] = {}, slot_exp[2] = {};
    if constexpr (!DENSE) {
        uint32_t w[16], mine_w = 0u;
        __builtin_memcpy(w, &a.tab, 64);
#pragma unroll
        for (int k = 0; k < 16; ++k) mine_w = (lane & 15) == k ? w[k] : mine_w;
        reinterpret_cast<uint32_t*>(table[wave])[lane & 15] = mine_w;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            slot_code[k] = table[wave][(2 * k + (c32 >> 4)) * 8 + (c32 & 7)];
            slot_exp[k] = table[wave][32 + slot_code[k]];
        }
    }
    // A coded stream's weights are at most 2^12 (times the slot's factor): |u| <= 2^12 |q|_1, which a power of two brings
    // below 2^15 for the fp16 parts of u.  The score kernel takes it (and the stream's own factor) out again.
    int e = 0;
    if constexpr (!DENSE) {
        const uint32_t bits = __float_as_uint(l1);
        if (bits) e = min(129 - (int)(bits >> 23), 100);
        if (half == 0) nrm[wave][c32] = ldexpf(1.0f, e);
    }
    if (slab == 0 && half == 0 && cb * 32 + c32 < ncol) {
        int b;
        const int row = row_of(cb * 32 + c32, b);
        const float f = DENSE ? a.scale_log2e : ldexpf(a.scale_log2e * (DIGITS ? 1.0f : FOLD_CODE_UNIT), -e - shift);
        a.rowfac[(long long)b * s.nrb * 16 * a.rt + row] = f;
    }

    // selection matrices: columns 0-15 take the 16 slots of one k-step, columns 16-31 those of the next
    uint4 sel[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool lo = (c32 >> 4) == w && (c32 & 15) == 8 * half + 2 * i, hi = (c32 >> 4) == w && (c32 & 15) == 8 * half + 2 * i + 1;
            const uint32_t one = DENSE ? 0x3F80u : 0x3C00u;
            d[i] = (lo ? one : 0u) | (hi ? one << 16 : 0u);
        }
        sel[w] = make_uint4(d[0], d[1], d[2], d[3]);
    }
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) {
        f32x16 uacc = zero16;
        [[maybe_unused]] float row_top = 0.0f;                       // digits: largest weight of the lane's channel
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            f32x16 t;
            if constexpr (DENSE) {
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[pr][nb][0]), __builtin_bit_cast(bf16x8, sel[0]), zero16, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[pr][nb][1]), __builtin_bit_cast(bf16x8, sel[1]), t, 0, 0, 0);
            } else {
                t = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, wf[pr][nb][0]), __builtin_bit_cast(f16x8, sel[0]), zero16, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, wf[pr][nb][1]), __builtin_bit_cast(f16x8, sel[1]), t, 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if constexpr (DIGITS)
#pragma unroll
                    for (int i = 0; i < 8; ++i) row_top = fmaxf(row_top, fabsf(t[8 * k + i]));
                uint32_t d[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = pack_hi16(__float_as_uint(t[8 * k + 2 * i]), __float_as_uint(t[8 * k + 2 * i + 1]));
                uacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, qa[nb][k]),
                                                               __builtin_bit_cast(bf16x8, make_uint4(d[0], d[1], d[2], d[3])), uacc, 0, 0, 0);
            }
        }
        // lane = channel slot c32, registers = 16 of the 32 query columns: to LDS in natural channel order
        int ch;
        float f = 1.0f;
        {
            const int ks = 2 * pr + (c32 >> 4), hs = (c32 >> 3) & 1, i = c32 & 7;
            if constexpr (DENSE) {
                ch = ks * 16 + hs * 8 + i;
            } else {
                ch = stream_channel(G, ks, hs, slot_code[pr & 1]);
                f = ldexpf(1.0f, -slot_exp[pr & 1]);
            }
        }
        if constexpr (DIGITS) {
            row_top = fmaxf(row_top, __shfl_xor(row_top, 32)) * f;
            if (half == 0) row_tops[wave][ch] = row_top;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int col = 8 * (i >> 2) + 4 * half + (i & 3);
            mine[col * FQ_STRIDE + ch] = DENSE ? uacc[i] : uacc[i] * f * nrm[wave][col];
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();

    if constexpr (DIGITS) {
        // 32 channels that share a power of two: do their weight rows (those not zero) differ too much?
        bool wide = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float v = row_tops[wave][64 * k + lane];
            float top = v, low = v > 0.0f ? v : INFINITY;
#pragma unroll
            for (int off = 16; off > 0; off >>= 1) {
                top = fmaxf(top, __shfl_xor(top, off));
                low = fminf(low, __shfl_xor(low, off));
            }
            wide |= top > FOLD_WIDE_ROWS * low;
        }
        fold_store_digits<G>(a, mine, place[wave], lane, slab, __any(wide));
        return;
    }
    // out: 16-byte pieces (column, tick, quarter); a fragment is read lane by lane, lane = 16 quarter + row
    const int rt_log2 = a.rt - 1 + 4;
    if (!DENSE && a.u_dense) {                                       // (a code's unit is part of the row factor)
#pragma unroll 1
        for (int it = 0; it < 8; ++it) {
            const int idx = it * 64 + lane, qd = idx & 3, tick = (idx >> 2) & 3, col = idx >> 4;
            const int at = place[wave][col], rr = at & (rpb - 1);
            if (at < 0) continue;
            uint8_t* dst = a.u_dense + ((long long)(at >> rt_log2) * a.n_slabs + slab) * FOLD_U_DENSE(a.rt) + ((rr >> 4) * 4 + tick) * 3 * 1024 +
                           (qd * 16 + (rr & 15)) * 16;
            const float* src = mine + col * FQ_STRIDE + 32 * tick + 8 * qd;
            uint32_t p[3][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t h0, m0, l0, h1, m1, l1_;
                split_bf16x3(src[2 * i] * (1.0f / FOLD_CODE_UNIT), h0, m0, l0);
                split_bf16x3(src[2 * i + 1] * (1.0f / FOLD_CODE_UNIT), h1, m1, l1_);
                p[0][i] = pack_hi16(h0, h1); p[1][i] = pack_hi16(m0, m1); p[2][i] = pack_hi16(l0, l1_);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4*>(dst + k * 1024) = make_uint4(p[k][0], p[k][1], p[k][2], p[k][3]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // (read before the coded pieces write their sums back)
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll 1
    for (int it = 0; it < 8; ++it) {
        const int idx = it * 64 + lane, qd = idx & 3, tick = (idx >> 2) & 3, col = idx >> 4;
        const int at = place[wave][col], rr = at & (rpb - 1);
        if (at < 0) continue;
        uint8_t* dst = a.u + ((long long)(at >> rt_log2) * a.n_slabs + slab) * a.u_slab + (qd * 16 + (rr & 15)) * 16;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ch = DENSE ? 32 * tick + 8 * qd + i : fold_channel<G>(tick, qd, i);
            v[i] = mine[col * FQ_STRIDE + ch];
        }
        if constexpr (DENSE) {
            uint32_t p[3][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t h0, m0, l0, h1, m1, l1_;
                split_bf16x3(v[2 * i], h0, m0, l0);
                split_bf16x3(v[2 * i + 1], h1, m1, l1_);
                p[0][i] = pack_hi16(h0, h1); p[1][i] = pack_hi16(m0, m1); p[2][i] = pack_hi16(l0, l1_);
            }
            dst += ((rr >> 4) * 4 + tick) * 3 * 1024;
#pragma unroll
            for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4*>(dst + k * 1024) = make_uint4(p[k][0], p[k][1], p[k][2], p[k][3]);
        } else {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const xq_f16x2 hh = {(_Float16)v[2 * i], (_Float16)v[2 * i + 1]};
                const xq_f16x2 ll = {(_Float16)(v[2 * i] - (float)hh.x), (_Float16)(v[2 * i + 1] - (float)hh.y)};
                hi[i] = __builtin_bit_cast(uint32_t, hh);
                lo[i] = __builtin_bit_cast(uint32_t, ll);
                // (the zero-point sums below are taken over the numbers the codes will meet)
                mine[col * FQ_STRIDE + fold_channel<G>(tick, qd, 2 * i)] = (float)hh.x + (float)ll.x;
                mine[col * FQ_STRIDE + fold_channel<G>(tick, qd, 2 * i + 1)] = (float)hh.y + (float)ll.y;
            }
            dst += ((rr >> 4) * 4 + tick) * 2 * 1024;
            *reinterpret_cast<uint4*>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(dst + 1024) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
    }
    if constexpr (!DENSE) {
        // Zero-point term: every group adds (z + zi s) sum_c u[c].  The sums of the slab's groups, split into three bf16
        // parts, are one more operand fragment against the three bf16 parts of z + zi s: quarter = part of the sum (the
        // fourth is zero), slots = [group 0 three times, 0, group 1 three times, 0].
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        float se = 0.0f, so = 0.0f;                                 // even and odd channels of this lane's half slab
        const float* src = mine + c32 * FQ_STRIDE + half * 64;
#pragma unroll 4
        for (int k = 0; k < 64; k += 4) {
            const float4 v = *reinterpret_cast<const float4*>(src + k);
            se += v.x + v.z;
            so += v.y + v.w;
        }
        float sz = (a.w.nibbles ? se : se + so) * (1.0f / FOLD_CODE_UNIT);   // (8-bit caches: a code's zero-point multiplies its weight row once)
        float sz1 = __shfl_xor(sz, 32);
        if constexpr (G == 128) { sz += sz1; sz1 = 0.0f; }
        if (half == 0 && cb * 32 + c32 < ncol) {
            const int at = place[wave][c32], rr = at & (rpb - 1);
            uint8_t* dst = a.u + ((long long)(at >> rt_log2) * a.n_slabs + slab) * a.u_slab + a.rt * 8192 + (rr >> 4) * 1024 + (rr & 15) * 16;
            uint32_t z[3], z1[3];
            split_bf16x3(sz, z[0], z[1], z[2]);
            split_bf16x3(sz1, z1[0], z1[1], z1[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *reinterpret_cast<uint4*>(dst + k * 256) = make_uint4(pack_hi16(z[k], z[k]), z[k] >> 16, pack_hi16(z1[k], z1[k]), z1[k] >> 16);
            *reinterpret_cast<uint4*>(dst + 768) = make_uint4(0u, 0u, 0u, 0u);
        }
    }
}

// =====================================================================================================================
// Scores.  A wave owns 128 tokens of a sequence, one block of 16 RT query rows and every SW-th slab, so that the slab ways are
// at neighbouring pieces of a token's cache lines at the same time (with runs of adjacent slabs per way a line left L2 before
// the wave came to its next piece: 8 x 4096 tokens of 3 bits 38 us against 31, 16 x 8191 of 2 bits in groups of 64 124 against
// 102, 4 x 32768 of 2 bits 114 against 96); a workgroup's waves are the slab ways of one tile.  A wave walks half slabs (64
// channels) and keeps a half's folded queries in registers while its 128 tokens stream past, the next half's on their way,
// so that neither LDS nor L2 is asked for them once per token.  A slab's codes are loaded row by row while the slab before
// is worked on and go through the wave's own LDS image into operand order; a lane unpacks its token's codes.  A half's
// products are summed by the matrix cores, scaled by the lane's own scale and added to the scores, which stay in
// registers; the rests of the zero-points enter through one more matrix instruction per slab and row tile.  At the end
// the slab ways' partial scores meet in LDS, and the softmax weights against the tile's maximum are stored as the value
// kernel reads them.
// Bound by issue: matrix and vector instructions of a SIMD's two waves overlap little (a 16 x 16 x 32 product alone 19 cycles, with
// three vector instructions 23, with six 39), and with nothing loaded the kernel takes 0.65 of its time.  Rests cut to bf16 parts
// where they are read, four times over, cost 2 to 3 us of 100 (1024 tiles of 2 bits); codes read in operand order straight into
// registers (64 cache lines touched by every load) two thirds more time.
// =====================================================================================================================
struct FoldScoreArgs {
    FoldSource x;
    FoldShape s;
    const uint8_t* u;
    const float* rowfac;
    float* p;                            // [nb][nrb][tiles][4][FOLD_P_TILE32]
    float* mtile;                        // [nb][nrb][tiles << mhalf][16 RT]
    int u_slab, waves;                   // waves of a workgroup
    int row_split;                       // bf16 rows: a workgroup has one row tile of the row block's two
    FoldSource window;                   // per-channel caches: the window's rows, its folded queries and workgroups
    const uint8_t* u_window;
    int n_window;
};

// the tile of a score workgroup of SW waves (4 or 8) and the slabs of a wave: every SW-th one of coded rows (step = SW), a run of
// adjacent ones of bf16 rows (step = 1)
// (nw: waves that hold any slab; rt0: first row tile of a workgroup that has one of the row block's `parts`)
struct FoldScorePlace { int b, rb, tile, tile0, len, SW, slab0, slab1, step, nw, rt0; };
__device__ __forceinline__ bool fold_score_place(const FoldShape& s, bool window, bool runs, int waves, int n_slabs, int wg, int wave, FoldScorePlace& o, int parts = 1)
{
    const int tiles = window ? 1 : s.tiles, n = s.nb * s.nrb * tiles * parts;
    int item = xcd_contiguous(n, wg);
    if (item >= n) return false;
    o.rt0 = item % parts;
    item /= parts;
    o.tile = item % tiles;
    o.rb = (item / tiles) % s.nrb;
    o.b = fold_sequence(s, item / (tiles * s.nrb));
    const FoldSpan span = fold_span(s, o.b, window);
    o.len = span.len;
    o.tile0 = span.tile0;
    o.SW = waves;
    const int per = runs ? (n_slabs + waves - 1) / waves : 1;
    o.slab0 = wave * per;
    o.slab1 = max(o.slab0, runs ? min(o.slab0 + per, n_slabs) : n_slabs);
    o.step = runs ? 1 : waves;
    o.nw = min(waves, (n_slabs + per - 1) / per);
    return o.tile * FOLD_TILE < o.len;
}

// what happens to the waves' partial scores: the end of every score kernel (BRT: row tiles of the row block)
template <int RT, int BRT = RT>
__device__ __forceinline__ void fold_scores_finish(const FoldShape& s, const float* rowfac_all, float* p_all, float* mtile_all,
                                                   f32x4 (&S)[RT][8], float* lds, const FoldScorePlace& o, int lane, int wave)
{
    // partial scores [wave][rt][tile16][lane] x 4 rows, lane = (token c16, rows 4 q + [0, 4))
    float4* part = reinterpret_cast<float4*>(lds);
    __syncthreads();
    if (o.slab0 < o.slab1)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                part[((wave * RT + rt) * 8 + i) * 64 + lane] = make_float4(S[rt][i][0], S[rt][i][1], S[rt][i][2], S[rt][i][3]);
    __syncthreads();
    const int c16 = lane & 15, q = lane >> 4, share = 8 / o.SW;      // tile16s a wave sums up
    const float* rowfac = rowfac_all + ((long long)o.b * s.nrb + o.rb) * 16 * BRT + 16 * o.rt0;
    float* mx = lds + o.SW * RT * 8 * 256;                           // [tile16][16 RT], behind the partial scores
    // (the sums replace the first wave's partial scores: what a wave reads there it has itself replaced)
    for (int j = 0; j < share; ++j) {
        const int i16 = wave * share + j, tok = o.tile * FOLD_TILE + i16 * 16 + c16;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float4* first = &part[(rt * 8 + i16) * 64 + lane];
            float4 t = *first;
            for (int k = 1; k < o.nw; ++k) {
                const float4 u = first[k * RT * 8 * 64];
                t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
            }
            float v[4] = {t.x, t.y, t.z, t.w}, m[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = tok < o.len ? v[r] * rowfac[rt * 16 + 4 * q + r] : -INFINITY;
                m[r] = v[r];
                m[r] = fmaxf(m[r], dpp_f32<DPP_QUAD_XOR1>(m[r]));
                m[r] = fmaxf(m[r], dpp_f32<DPP_QUAD_XOR2>(m[r]));
                m[r] = fmaxf(m[r], dpp_f32<DPP_ROW_HALF_MIRROR>(m[r]));
                m[r] = fmaxf(m[r], dpp_f32<DPP_ROW_MIRROR>(m[r]));
            }
            *first = make_float4(v[0], v[1], v[2], v[3]);
            if (c16 == 0)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx[i16 * 16 * RT + rt * 16 + 4 * q + r] = m[r];
        }
    }
    __syncthreads();
    // maximum of the tile, or of the wave's half of it (eight slab ways then: a wave's tile16s lie in one half)
    const int i0 = wave * share, mrow0 = (o.tile0 + o.tile) << s.mhalf | (s.mhalf ? i0 >> 2 : 0);
    const bool stores = c16 == 0 && (s.mhalf ? (i0 & 3) == 0 : i0 == 0);
    float Mu[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = rt * 16 + 4 * q + r;
            float h0 = mx[row], h1 = mx[4 * 16 * RT + row];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                h0 = fmaxf(h0, mx[k * 16 * RT + row]);
                h1 = fmaxf(h1, mx[(4 + k) * 16 * RT + row]);
            }
            const float M = s.mhalf ? (i0 & 4 ? h1 : h0) : fmaxf(h0, h1);
            Mu[rt][r] = M == -INFINITY ? 0.0f : M;                  // nothing visible: all weights 0
            if (stores) mtile_all[((((long long)o.b * s.nrb + o.rb) * s.tiles << s.mhalf) + mrow0) * 16 * BRT + 16 * o.rt0 + row] = M;
        }
    for (int j = 0; j < share; ++j) {
        const int i16 = wave * share + j, t32 = (i16 & 1) * 16 + c16, slot = t32 >> 2, qd = t32 & 3;
        float* pt = p_all + ((((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0 + o.tile) * 4 + (i16 >> 1)) * FOLD_P_TILE32<BRT> + o.rt0 * 512;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const float4 t = part[(rt * 8 + i16) * 64 + lane];
            const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int r = 0; r < 4; ++r)
                pt[(rt * 2 + (slot >> 2)) * 256 + (4 * q + r + 16 * qd) * 4 + (slot & 3)] = __builtin_amdgcn_exp2f(v[r] - Mu[rt][r]);
        }
    }
}

template <int RT>
constexpr int FOLD_SCORE_RED = 8 * RT * 8 * 1024 + 8 * 8 * 16 * RT * 4;
// a wave's codes of one slab, its records (4 bytes per token and group, 8 for nibble streams), and the tokens' rests as operands
// (8 bytes per group)
template <int BITS, int G, bool NIB>
constexpr int FOLD_SCORE_WAVE = FOLD_TILE * 16 * BITS + (128 / G) * FOLD_TILE * (NIB ? 8 : 4) + (128 / G) * FOLD_TILE * 8;
template <int BITS, int G, int RT, bool NIB>
constexpr int FOLD_SCORE_LDS = 8 * FOLD_SCORE_WAVE<BITS, G, NIB> > FOLD_SCORE_RED<RT> ? 8 * FOLD_SCORE_WAVE<BITS, G, NIB> : FOLD_SCORE_RED<RT>;

template <int BITS, int G, int RT, bool NIB>
__global__ __launch_bounds__(512) void fold_scores_kernel(const FoldScoreArgs a)
{
    constexpr int GPS = 128 / G, ROWB = 16 * BITS;                  // groups and bytes of a slab's row
    constexpr int NL = 2 * BITS;                                    // 1 KiB loads of a slab's codes per wave
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FoldShape& s = a.s;
    const FoldSource& x = a.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    FoldScorePlace o;
    if (!fold_score_place(s, false, false, a.waves, x.n_slabs, blockIdx.x, wave, o)) return;
    const int b = o.b, rb = o.rb, len = o.len, tok0 = o.tile * FOLD_TILE;
    const int c16 = lane & 15, q = lane >> 4;
    const uint8_t* cbase = x.codes + (long long)(s.b0 + b) * x.cap * x.row_bytes;
    const uint16_t* sbase = x.scale + (long long)(s.b0 + b) * x.cap * x.ng_row;
    const uint16_t* zbase = x.zero + (long long)(s.b0 + b) * x.cap * x.ng_row;
    const uint8_t* ubase = a.u + ((long long)b * s.nrb + rb) * x.n_slabs * a.u_slab;
    const uint32_t uoff = lane * 16;
    const int slab0 = o.slab0, slab1 = o.slab1;
    uint8_t* image = lds + wave * FOLD_SCORE_WAVE<BITS, G, NIB>;     // [token 128][ROWB]
    uint32_t* records = reinterpret_cast<uint32_t*>(image + FOLD_TILE * ROWB);
    uint2* rests = reinterpret_cast<uint2*>(image + FOLD_TILE * ROWB + GPS * FOLD_TILE * (NIB ? 8 : 4));     // [token][group]

    // Codes go through the wave's LDS image: loaded row by row (a load then touches 64 / BITS rows once; in operand order
    // every row would be touched by four quarter waves, and L1 look-ups bound the kernel), written once the slab before has
    // been read, read back in operand order.
    uint32_t voff[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int pc = k * 64 + lane;
        voff[k] = (uint32_t)min(tok0 + pc / BITS, len - 1) * (uint32_t)x.row_bytes + (uint32_t)(pc % BITS) * 16u;
    }
    // stored zero-points and scales of the slab's groups for the tokens lane and lane + 64
    const uint32_t moff[2] = {(uint32_t)min(tok0 + lane, len - 1) * (uint32_t)x.ng_row, (uint32_t)min(tok0 + 64 + lane, len - 1) * (uint32_t)x.ng_row};
    uint32_t zs[2][2];
    auto load_meta = [&](int slab) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if constexpr (GPS == 2) {
                zs[t][0] = *reinterpret_cast<const uint32_t*>(zbase + 2 * slab + moff[t]);
                zs[t][1] = *reinterpret_cast<const uint32_t*>(sbase + 2 * slab + moff[t]);
            } else {
                zs[t][0] = (zbase + (slab >> x.meta_shift))[moff[t]];
                zs[t][1] = (sbase + (slab >> x.meta_shift))[moff[t]];
            }
        }
    };
    // -> records: -zi (fp16) | scale (bf16); nibble streams: -zi of either nibble, scale (fp32)
    float rs[2][GPS];                                                // what is left of the zero-points
    auto write_meta = [&]() XQ_INLINE_LAMBDA {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < GPS; ++g) {
                const float z = g ? bf16_hi_to_f32(zs[t][0]) : bf16_lo_to_f32(zs[t][0]);
                const float sc = g ? bf16_hi_to_f32(zs[t][1]) : bf16_lo_to_f32(zs[t][1]);
                const float zi = fold_integer_zero(sc, z, NIB ? 255.0f : (float)((1 << BITS) - 1), rs[t][g]);
                const int at = g * FOLD_TILE + t * 64 + lane;
                if constexpr (NIB) {
                    const float zh = floorf(zi * (1.0f / 16.0f));
                    reinterpret_cast<uint2*>(records)[at] =
                        make_uint2(f16_bits((zi - 16.0f * zh) * (-1.0f / FOLD_CODE_UNIT)) | (f16_bits(zh * (-1.0f / FOLD_CODE_UNIT)) << 16),
                                   __float_as_uint(sc));
                } else {
                    records[at] = f16_bits(zi * (-1.0f / FOLD_CODE_UNIT)) | (__float_as_uint(sc) & 0xFFFF0000u);
                }
            }
    };
    // -> rests: three bf16 parts each, cut here, once per token (every quarter wave of the products needs them)
    auto write_rests = [&]() XQ_INLINE_LAMBDA {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            uint2 v[GPS];
#pragma unroll
            for (int g = 0; g < GPS; ++g) {
                uint32_t h, m, l;
                split_bf16x3(rs[t][g], h, m, l);
                v[g] = make_uint2(pack_hi16(h, m), l >> 16);
            }
            if constexpr (GPS == 2) reinterpret_cast<uint4*>(rests)[t * 64 + lane] = make_uint4(v[0].x, v[0].y, v[GPS - 1].x, v[GPS - 1].y);
            else rests[t * 64 + lane] = v[0];
        }
    };

    f32x4 S[RT][8];
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 8; ++i) S[rt][i] = zero4;
    // A slab is 16 units: half slab t / 8 against token tile t % 8.  While the 4 RT matrix instructions of unit t run, the
    // vector ALU unpacks unit t + 1 and adds unit t - 1 to the scores, a little of each behind every matrix instruction
    // (scheduling fences keep it there).
    if (slab0 < slab1) {
        uint4 u[2][RT][2][2], uz[RT];                                // folded queries of the two halves: [rt][tick][hi, lo]
        uint32_t rec[4][2];                                          // records of units t - 1 .. t + 2: -zi, scale
        uint32_t cw[4][2];                                           // code dwords of units t .. t + 2
        uint32_t F[2][8];                                            // token operands of units t, t + 1
        f32x4 P[2][RT];
        auto load_u = [&](int slab, auto HF, auto I) XQ_INLINE_LAMBDA {                  // piece I of half HF
            constexpr int h = decltype(HF)::value, i = decltype(I)::value, rt = i >> 2, t = (i >> 1) & 1, k = i & 1;
            u[h][rt][t][k] = *reinterpret_cast<const uint4*>(ubase + (long long)slab * a.u_slab + rt * 8192 + h * 4096 + t * 2048 + k * 1024 + uoff);
        };
        auto read_unit = [&](auto T) XQ_INLINE_LAMBDA {               // record and codes of unit T (16, 17: the next slab's first two)
            constexpr int t = decltype(T)::value, h = (t >> 3) & 1, i = t & 7, n = t & 3;
            const int at = (GPS == 2 ? h : 0) * FOLD_TILE + i * 16 + c16;
            if constexpr (NIB) {
                const uint2 r = reinterpret_cast<const uint2*>(records)[at];
                rec[n][0] = r.x; rec[n][1] = r.y;
            } else {
                const uint32_t r = records[at];
                rec[n][0] = r; rec[n][1] = r & 0xFFFF0000u;
            }
            const uint32_t* src = reinterpret_cast<const uint32_t*>(image + (i * 16 + c16) * ROWB);
            if constexpr (G == 128) {                                // dwords of the lane's unit of 32 codes: those of half h
                const uint32_t* w = src + q * BITS;
                if constexpr (BITS == 2) { cw[n][0] = w[h]; cw[n][1] = 0u; }
                else if constexpr (BITS == 3) { cw[n][0] = w[h]; cw[n][1] = w[h + 1]; }
                else { cw[n][0] = w[2 * h]; cw[n][1] = w[2 * h + 1]; }
            } else {                                                 // 16 codes of group h
                if constexpr (BITS == 2) { cw[n][0] = src[4 * h + q]; cw[n][1] = 0u; }
                else if constexpr (BITS == 3) { const uint32_t* w = src + 6 * h + ((6 * q) >> 2); cw[n][0] = w[0]; cw[n][1] = w[1]; }
                else { cw[n][0] = src[8 * h + 2 * q]; cw[n][1] = src[8 * h + 2 * q + 1]; }
            }
        };
        uint32_t m0, m1;
        auto unpack = [&](auto T, auto K) XQ_INLINE_LAMBDA {          // operand dword K of unit T
            constexpr int t = decltype(T)::value, h = (t >> 3) & 1, n = t & 3, k = decltype(K)::value;
            if constexpr (k == 0) {                                  // merged octet pair
                m1 = 0u;
                if constexpr (BITS == 2) {
                    m0 = cw[n][0];
                } else if constexpr (BITS == 3 && G == 128) {        // 48 bits at bit 0 / 16 of the two dwords
                    m0 = perm_bytes(cw[n][1], cw[n][0], h == 0 ? 0x04030100u : 0x06050302u);
                    m1 = perm_bytes(cw[n][1], cw[n][0], h == 0 ? 0x05040201u : 0x07060403u);
                } else if constexpr (BITS == 3) {                    // ... at bit 0 (even quarters) or 16
                    const uint32_t lo = __builtin_amdgcn_alignbit(cw[n][1], cw[n][0], (q & 1) * 16), hi = cw[n][1] >> ((q & 1) * 16);
                    m0 = perm_bytes(hi, lo, 0x04030100u);
                    m1 = perm_bytes(hi, lo, 0x05040201u);
                } else {
                    m0 = perm_bytes(cw[n][1], cw[n][0], 0x05040100u);
                    m1 = perm_bytes(cw[n][1], cw[n][0], 0x07060302u);
                }
                if constexpr (!NIB) rec[n][0] = perm_bytes(rec[n][0], rec[n][0], 0x01000100u);
            }
            uint32_t add = rec[n][0];
            if constexpr (NIB) add = perm_bytes(add, add, (k & 1) ? 0x03020302u : 0x01000100u);      // -zi of the even / odd codes
            F[t & 1][k] = fold_code<BITS, k>(m0, m1, add);
        };
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 cn[NL];
        auto load_codes = [&](int slab, auto K) XQ_INLINE_LAMBDA {
            constexpr int k = decltype(K)::value;
            cn[k] = *reinterpret_cast<const u32x4*>(cbase + slab * ROWB + voff[k]);
        };
        auto write_codes = [&]() XQ_INLINE_LAMBDA {
            static_for<0, NL>([&](auto K) XQ_INLINE_LAMBDA {
                constexpr int k = decltype(K)::value;
                *reinterpret_cast<u32x4*>(image + (k * 64 + lane) * 16) = cn[k];
            });
        };
        load_meta(slab0);
        static_for<0, NL>([&](auto K) XQ_INLINE_LAMBDA { load_codes(slab0, K); });
        static_for<0, 4 * RT>([&](auto I) XQ_INLINE_LAMBDA { load_u(slab0, std::integral_constant<int, 0>{}, I); });
        write_meta();
        write_rests();
        write_codes();
        read_unit(std::integral_constant<int, 0>{});
        read_unit(std::integral_constant<int, 1>{});
        static_for<0, 8>([&](auto K) XQ_INLINE_LAMBDA { unpack(std::integral_constant<int, 0>{}, K); });
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) P[1][rt] = zero4;
        rec[3][1] = 0u;                                              // (unit -1 adds nothing)
        for (int slab = slab0; slab < slab1; slab += o.step) {
            const int snext = slab + o.step < slab1 ? slab + o.step : slab;    // (the last iteration prepares itself again)
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, 16>([&](auto T) XQ_INLINE_LAMBDA {
                constexpr int t = decltype(T)::value, h = t >> 3, i = t & 7;
                if constexpr (t == 1) load_meta(snext);
                if constexpr (t >= 2 && t < 2 + NL) load_codes(snext, std::integral_constant<int, t - 2>{});
                // (units 14 and 15 of this slab have been read: the next slab's records and codes may take their place)
                if constexpr (t == 14) { write_meta(); write_codes(); }
                read_unit(std::integral_constant<int, t + 2>{});
                uint4 mz = make_uint4(0u, 0u, 0u, 0u);
                if constexpr (h == 1 && GPS == 2) mz = reinterpret_cast<const uint4*>(rests)[i * 16 + c16];
                if constexpr (h == 1 && GPS == 1) { const uint2 r = rests[i * 16 + c16]; mz.x = r.x; mz.y = r.y; }
                // the next half's folded queries, ahead of the codes in the first half: loads return in order, and the queries
                // come out of L2, the codes from farther away
                if constexpr (i == 0)
                    static_for<0, 4 * RT>([&](auto I) XQ_INLINE_LAMBDA { load_u(h == 0 ? slab : snext, std::integral_constant<int, h ^ 1>{}, I); });
                if constexpr (t == 0)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        uz[rt] = *reinterpret_cast<const uint4*>(ubase + (long long)slab * a.u_slab + RT * 8192 + rt * 1024 + uoff);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, 4 * RT>([&](auto M) XQ_INLINE_LAMBDA {
                    constexpr int m = decltype(M)::value, rt = m % RT, k = 1 - (m / RT) % 2, tick = m / (2 * RT);
                    const uint32_t* f = &F[t & 1][4 * tick];
                    P[t & 1][rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, u[h][rt][tick][k]), as_frag(f[0], f[1], f[2], f[3]),
                                                                          m < RT ? zero4 : P[t & 1][rt], 0, 0, 0);
                    static_for<0, 2 / RT>([&](auto E) XQ_INLINE_LAMBDA {
                        unpack(std::integral_constant<int, t + 1>{}, std::integral_constant<int, m * (2 / RT) + decltype(E)::value>{});
                    });
                    // the unit before: rows r of row tile q2
                    constexpr int q2 = m / 4, r = m & 3, ip = (t + 7) & 7;
                    S[q2][ip][r] = __builtin_fmaf(P[(t + 1) & 1][q2][r], __uint_as_float(rec[(t + 3) & 3][1]), S[q2][ip][r]);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (h == 1) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        S[rt][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, uz[rt]), __builtin_bit_cast(bf16x8, mz), S[rt][i], 0, 0, 0);
                }
                if constexpr (t == 15) write_rests();                // (the next slab's: unit 15's have been read)
                __builtin_amdgcn_sched_barrier(0);
            });
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)                              // the last unit
#pragma unroll
            for (int r = 0; r < 4; ++r) S[rt][7][r] = __builtin_fmaf(P[1][rt][r], __uint_as_float(rec[3][1]), S[rt][7][r]);
    }
    fold_scores_finish<RT>(s, a.rowfac, a.p, a.mtile, S, reinterpret_cast<float*>(lds), o, lane, wave);
}

#include "folded_digits.hpp"

// the same over bf16 rows (the cross-layer accumulator, a residual window): no codes and no groups, u in three bf16 parts.
// The rows of a half slab (128 bytes each) go through the wave's LDS image as the codes do, 16 token rows at a time; their
// 16-byte pieces are swizzled by the row, so that neither the row-wise write nor the fragment read meets bank conflicts.
// A wave has a run of adjacent slabs: its pieces are whole cache lines, so there is nothing to share with the other waves, and
// side by side these read one 2 KiB stretch of 128 rows at a time.  Whole steps, slabs dealt out as above / runs: 8 x 8192 rows of
// d = 4096 259 / 238 us, 16 x 8192 of d = 2048 and 16 heads 242 / 216, 8 x 4096 of d = 4096 148 / 142; 6 x 8192, where the XCDs
// are at different places of their sequences, 225 either way.
template <int RT, int BRT = RT>
__device__ __forceinline__ void fold_scores_dense(const FoldScoreArgs& a, const FoldSource& x, const uint8_t* u_all, bool window, int waves, uint8_t* lds)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int u_slab = FOLD_U_DENSE(BRT);
    const FoldShape& s = a.s;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    FoldScorePlace o;
    if (!fold_score_place(s, window, true, waves, x.n_slabs, blockIdx.x, wave, o, BRT / RT)) return;
    const int b = o.b, rb = o.rb, len = o.len, tok0 = o.tile * FOLD_TILE;
    const int c16 = lane & 15, q = lane >> 4;
    const uint8_t* xbase = reinterpret_cast<const uint8_t*>(x.rows) + (long long)(s.b0 + b) * x.cap * x.row_bytes;
    const uint8_t* ubase = u_all + ((long long)b * s.nrb + rb) * x.n_slabs * u_slab + o.rt0 * 4 * 3072;
    const uint32_t uoff = lane * 16;
    uint8_t* image = lds + wave * 2 * 2048;                          // two images of 16 rows x 128 bytes
    f32x4 S[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 8; ++i) S[rt][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // load side: lane = (row lane / 8, piece lane % 8) of 8 rows; fragment side: row c16, pieces 4 tick + q
    const int r8 = lane >> 3, pc = lane & 7;
    uint32_t voff[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) voff[k] = (uint32_t)min(tok0 + k * 8 + r8, len - 1) * (uint32_t)x.row_bytes + pc * 16;
    const int wpos = r8 * 128 + ((pc ^ r8) * 16), rpos = c16 * 128;
    if (o.slab0 < o.slab1) {
        uint4 u[2][RT][2][3];
        u32x4 xr[16];                                                // the half slab's rows on their way: [token tile 8][8-row part 2]
        auto load_x = [&](int half_idx, auto I) XQ_INLINE_LAMBDA {
            constexpr int i = decltype(I)::value;
            const uint8_t* base = xbase + half_idx * 128;
            xr[2 * i] = *reinterpret_cast<const u32x4*>(base + voff[2 * i]);
            xr[2 * i + 1] = *reinterpret_cast<const u32x4*>(base + voff[2 * i + 1]);
        };
        auto load_u = [&](int half_idx, auto HF) XQ_INLINE_LAMBDA {
            constexpr int h = decltype(HF)::value;
            const uint8_t* us = ubase + (long long)(half_idx >> 1) * u_slab + (half_idx & 1) * 6144;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int k = 0; k < 3; ++k) u[h][rt][t][k] = *reinterpret_cast<const uint4*>(us + (rt * 4 + t) * 3072 + k * 1024 + uoff);
        };
        load_u(2 * o.slab0, std::integral_constant<int, 0>{});
        static_for<0, 8>([&](auto I) XQ_INLINE_LAMBDA { load_x(2 * o.slab0, I); });
        for (int slab = o.slab0; slab < o.slab1; slab += o.step) {
            const int snext = slab + o.step < o.slab1 ? slab + o.step : slab;
            static_for<0, 2>([&](auto HF) XQ_INLINE_LAMBDA {
                constexpr int h = decltype(HF)::value;
                const int hn = h == 0 ? 2 * slab + 1 : 2 * snext;
                load_u(hn, std::integral_constant<int, h ^ 1>{});
                static_for<0, 8>([&](auto I) XQ_INLINE_LAMBDA {
                    constexpr int i = decltype(I)::value;
                    uint8_t* img = image + (i & 1) * 2048;
                    *reinterpret_cast<u32x4*>(img + wpos) = xr[2 * i];
                    *reinterpret_cast<u32x4*>(img + 1024 + wpos) = xr[2 * i + 1];
                    load_x(hn, I);
                    const u32x4 x0 = *reinterpret_cast<const u32x4*>(img + rpos + ((q ^ (c16 & 7)) * 16));
                    const u32x4 x1 = *reinterpret_cast<const u32x4*>(img + rpos + (((4 + q) ^ (c16 & 7)) * 16));
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const bf16x8 xf = __builtin_bit_cast(bf16x8, t ? x1 : x0);
#pragma unroll
                        for (int k = 2; k >= 0; --k)
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt)
                                S[rt][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u[h][rt][t][k]), xf, S[rt][i], 0, 0, 0);
                    }
                });
            });
        }
    }
    fold_scores_finish<RT, BRT>(s, a.rowfac, a.p, a.mtile, S, reinterpret_cast<float*>(lds), o, lane, wave);
}

template <int RT, int BRT = RT>
__global__ __launch_bounds__(512) void fold_scores_dense_kernel(const FoldScoreArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    fold_scores_dense<RT, BRT>(a, a.x, a.u, false, a.waves, lds);
}

// =====================================================================================================================
// Values.  A workgroup owns two slabs (256 channels) of a sequence, one row block and a range of tokens; its four waves are
// two slab ways and two token ways, and two workgroups share a CU where there are enough of them (fold_splits), so that one's
// set-up, barriers and sums run beside the other's products.  Per 128 tokens all waves bring the stored softmax weights to the sequence's maximum and stage them in LDS
// with the tokens' scales, integer zero-points and rests; a wave then takes 32 tokens at a time.  The contraction runs over
// tokens, so an operand dword pairs the codes of two tokens: a lane takes octet n = lane % 16 of the slab (8 channels) for
// eight tokens, merges token pairs, and column tile k of the product is code k of every lane's octet -- no transposition.
// (Groups of 64 of 4 bits: lanes n and n + 8 exchange half octets, so that a column tile lies in one group.)  The rests are summed on the
// vector ALU by the threads that stage the weights.  At the end the token ways meet in LDS.
//
// 2 and 3 bits: (code - zi) times the scale has at most 3 + 8 bits, so it is exact in fp16 and goes into the codes' operand (one
// packed product per dword), and the weights are cut into fp16 hi + lo once, when they are staged.  Other codes have a bit too
// many: there weight times scale is cut per group.  Bound by issue: the vector ALU takes about 1.5 times as long as the matrix
// instructions.  Measured, us, weight times scale in workgroups of eight waves / this: 4 x 32768 tokens of 2 bits 118 / 102,
// 16 x 8191 of 2 bits in groups of 64 149 / 104, half the width 44 / 37 (of these the loads of scales and maxima before the loop eight
// at a time 10, 3, 2); 8 x 4096 of 3 bits, where the workspace leaves a CU one workgroup, 35 / 38, and 34 with two.
//
// Range of the fp16 parts.  Weights are taken against the range's own maximum of the row and scales against the range's
// largest scale of the group.  The low parts end at 2^-24, so they are off by up to 2^-25.  Weights are cut times 2^15: a token is cut by at
// most 2^-40 of the largest scale, whatever its weight.  Weights times scales have the largest scale in [2^14, 2^15): at most 2^-39 of it.
// Every row has a token of weight 1 in its tiles, so with scales within a factor 2^13 (12 exponents) that is 2^-27 (2^-26) of what the
// row sums up, and 2^12 such cuts in random directions, 0.6 times as large in the mean, reach 2^-22 (2^-21), about what
// the parts carry.  A range with a wider group, a negative scale or a non-finite one is summed in plain
// fp32 instead (fold_values_plain), and one with zero scales among others where their tokens may hold all the weight.  Measured, one
// token of 300 larger by 2^20 / 2^28 that no row attends to: error 1.1e-5 / 1.7e-3 with one factor per group and no such limit, 5e-7 now.
// =====================================================================================================================
struct FoldValueArgs {
    FoldSource x;
    FoldShape s;
    const float* p;
    const float* mtile;
    float* y;                            // [splits][nb][R][n_slabs 128]
    float* yz;                           // [splits][nb][R][ng]: sum of weight times rest of the zero-point, per group
    float* lsum;                         // [splits][nb][nrb 16 RT]
    int cblocks;                         // workgroups per row of slabs
    FoldSource window;                   // as in FoldScoreArgs
    int n_window;
};

// Workgroups of four waves over coded rows: two slab ways, two token ways of 64 tokens.
constexpr int FOLD_VALUE_WAVES = 4, FOLD_VALUE_THREADS = 64 * FOLD_VALUE_WAVES;
constexpr int FOLD_VSTEP = 32 * FOLD_VALUE_WAVES;                               // tokens staged at a time
// the scale goes into the codes' operand: (code - zi) s has at most 8 + 3 bits (see above)
constexpr bool fold_scaled_codes(int bits) { return bits <= 3; }

template <int RT, int GROUPS, bool NIB, bool SCALED>
struct FoldValueLds {
    static constexpr int P_BYTES = FOLD_VSTEP / 32 * FOLD_P_TILE32<RT> * 4;     // softmax weights of a step
    static constexpr int STRIDE = FOLD_VSTEP + 4;                               // floats: rests (and scales) of a group's tokens
    static constexpr int H_STRIDE = FOLD_VSTEP + 8;                             // halfs: -zi (of even, then of odd codes), or -zi and scales
    static constexpr int REST = SCALED ? 0 : STRIDE * 4, HALFS = REST + STRIDE * 4;
    static constexpr int GROUP_BYTES = HALFS + (NIB || SCALED ? 2 : 1) * H_STRIDE * 2;
    static constexpr int SZ_BYTES = GROUPS * GROUP_BYTES;
    static constexpr int P_OFF = 0, SZ_OFF = 2 * P_BYTES, M_OFF = SZ_OFF + 2 * SZ_BYTES;
    static constexpr int N_OFF = M_OFF + 16 * RT * 4 * 34;                      // row maxima (a column per partial reader, twice, and the results)
    static constexpr int L_OFF = N_OFF + GROUPS * 4 * 17;
    static constexpr int LOOP = L_OFF + 8 * 16 * RT * 4;
    static constexpr int RED = FOLD_VALUE_WAVES * RT * 8 * 1024;                // every wave's accumulators, at the end
    static constexpr int TOTAL = LOOP > RED ? LOOP : RED;
    // what fold_values_plain keeps there lies below the row maxima
    static_assert(8 * FOLD_P_TILE32<RT> * 4 + GROUPS * FOLD_VTILE * 8 <= M_OFF, "256 tokens' weights, scales and zero-points");
};

constexpr int FOLD_SCALE_SPREAD = 12;        // exponents between a range's scales of a group that the fp16 parts are used for

// tile and range of a value workgroup
struct FoldValuePlace { int b, rb, cblk, split, len, tile0, t0, t1; };      // [t0, t1): 256-token tiles
__device__ __forceinline__ bool fold_value_place(const FoldShape& s, bool window, int cblocks, int wg, FoldValuePlace& o)
{
    const int splits = window ? 1 : s.block ? s.splits - 1 : s.splits;
    const int n = s.nb * s.nrb * splits * cblocks;
    const int item = xcd_contiguous(n, wg);
    if (item >= n) return false;
    o.cblk = item % cblocks;                                        // (neighbours share the softmax weights)
    const int k = (item / cblocks) % splits;
    o.split = window ? s.splits - 1 : k;
    o.rb = (item / (cblocks * splits)) % s.nrb;
    o.b = fold_sequence(s, item / (cblocks * splits * s.nrb));
    const FoldSpan span = fold_span(s, o.b, window);
    o.len = span.len;
    o.tile0 = span.tile0;
    const int nt = (o.len + FOLD_VTILE - 1) / FOLD_VTILE, per = (nt + splits - 1) / splits;
    o.t0 = k * per;
    o.t1 = min(nt, o.t0 + per);
    return o.t0 < o.t1;
}

// maximum of every row over the sequence's score tiles -> mrow[16 RT] (a workgroup barrier ends it).  FOLD_RANGE_TOP:
// over the stored maxima [r0, r1) instead, and behind them the factor from that maximum to the sequence's.  FOLD_RANGE_LOW:
// behind them the lowest of the stored maxima [r0, r1)
enum { FOLD_RANGE_TOP = 1, FOLD_RANGE_LOW = 2 };
template <int RT, int RANGE = 0, int NT = 512>
__device__ __forceinline__ void fold_row_maxima(const FoldShape& s, const float* mtile, int b, int rb, float* scratch, float* mrow, int r0 = 0, int r1 = 0)
{
    constexpr int ROWS = 16 * RT, PARTS = NT / ROWS > 16 ? 16 : NT / ROWS;
    const int tid = threadIdx.x, row = tid % ROWS, pt = tid / ROWS;
    const int len = s.len.v[s.b0 + b], coded = s.block ? len / s.block * s.block : len;
    const int unit = FOLD_TILE >> s.mhalf;                          // tokens of a stored maximum
    const int window0 = (coded + FOLD_VTILE - 1) / FOLD_VTILE * (FOLD_VTILE / unit);  // maxima of the window, if it holds anything
    const int n_coded = (coded + unit - 1) / unit, nt = len > coded ? window0 + (len - coded + unit - 1) / unit : n_coded;
    if (pt < PARTS) {
        float m = -INFINITY, mr = RANGE == FOLD_RANGE_LOW ? INFINITY : -INFINITY;
        const float* src = mtile + (((long long)b * s.nrb + rb) * s.tiles << s.mhalf) * ROWS + row;
        // (eight loads at a time: one latency for them all; behind the last maximum it is read again)
        for (int t0 = pt; t0 < nt; t0 += 8 * PARTS) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = src[(long long)min(t0 + k * PARTS, nt - 1) * ROWS];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int t = min(t0 + k * PARTS, nt - 1);
                if (t < n_coded || t >= window0) {
                    m = fmaxf(m, v[k]);
                    if (RANGE && t >= r0 && t < r1) mr = RANGE == FOLD_RANGE_LOW ? fminf(mr, v[k] == -INFINITY ? INFINITY : v[k]) : fmaxf(mr, v[k]);
                }
            }
        }
        scratch[pt * ROWS + row] = m;
        if constexpr (RANGE != 0) scratch[(PARTS + pt) * ROWS + row] = mr;
    }
    __syncthreads();
    if (tid < ROWS) {
        float m = scratch[tid];
#pragma unroll
        for (int k = 1; k < PARTS; ++k) m = fmaxf(m, scratch[k * ROWS + tid]);
        mrow[tid] = m;
        if constexpr (RANGE != 0) {
            float mr = scratch[PARTS * ROWS + tid];
#pragma unroll
            for (int k = 1; k < PARTS; ++k) {
                const float v = scratch[(PARTS + k) * ROWS + tid];
                mr = RANGE == FOLD_RANGE_LOW ? fminf(mr, v) : fmaxf(mr, v);
            }
            if constexpr (RANGE == FOLD_RANGE_TOP) {
                mrow[tid] = mr;
                mrow[ROWS + tid] = mr == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mr - m);
            } else {
                mrow[ROWS + tid] = mr;
            }
        }
    }
    __syncthreads();
}

// softmax denominators of a row block and split from every thread's share of them, times f (of row tid)
template <int RT, int NW = 8>
__device__ __forceinline__ void fold_denominators(const FoldValueArgs& a, const FoldValuePlace& o, float l, float f, float* lp)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (lane < 16) lp[wave * 16 + lane] = l;
    __syncthreads();
    if (tid < 16 * RT) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if (RT == 1 || ((w >> 1) & 1) == (tid >> 4)) t += lp[w * 16 + (tid & 15)];
        a.lsum[(((long long)o.split * a.s.nb + o.b) * a.s.nrb + o.rb) * 16 * RT + tid] = t * f;
    }
}

// The token ways of a workgroup's two slabs meet in LDS: half a row tile of a slab (row tile h / 2, column tiles 4 (h % 2) +
// [0, 4)) is summed by the wave (slab way, token way h), or by the token ways in turn where there are fewer
template <int RT, int NW>
constexpr int FOLD_MEET = NW / 2 >= 2 * RT ? 1 : 2 * RT / (NW / 2);             // halves per wave
template <int RT, int NW>
__device__ __forceinline__ void fold_meet(const f32x4 (&acc)[RT][8], uint8_t* lds, int wave, int lane, f32x4 (&t)[FOLD_MEET<RT, NW>][4])
{
    constexpr int TW = NW / 2;
    float4* acc_lds = reinterpret_cast<float4*>(lds);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int k = 0; k < 8; ++k)
            acc_lds[((wave * RT + rt) * 8 + k) * 64 + lane] = make_float4(acc[rt][k][0], acc[rt][k][1], acc[rt][k][2], acc[rt][k][3]);
    __syncthreads();
    const int sw = wave & 1, tw = wave >> 1;
    if (tw >= 2 * RT) return;
#pragma unroll
    for (int i = 0; i < FOLD_MEET<RT, NW>; ++i) {
        const int h = tw + i * TW, rt = h >> 1, kg = h & 1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float4 v = acc_lds[((sw * RT + rt) * 8 + 4 * kg + k) * 64 + lane];
#pragma unroll
            for (int w = 1; w < TW; ++w) {
                const float4 u = acc_lds[(((2 * w + sw) * RT + rt) * 8 + 4 * kg + k) * 64 + lane];
                v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
            }
            t[i][k] = f32x4{v.x, v.y, v.z, v.w};
        }
    }
}

// The sums of a range whose scales lie too far apart for fp16 parts: x^ and the sums in fp32, a thread per channel of
// either slab and half of the rows.  Rare, and bound by the vector ALU and the LDS reads of the weights, the latter uncovered where
// one workgroup of four waves has a CU: with every range on it a decode call over 8 x 4096 tokens of 3 bits (32 heads, d = 4096)
// takes 330 us (95 on the fp16 parts; 374 when the codes were waited for 8 tokens at a time; 1650 when K and V are
// rematerialised), 16 x 8191 of 2 bits in groups of 64 687 us (206; 778; 1790).
template <int BITS, int G, int RT, bool NIB>
__device__ __forceinline__ void fold_values_plain(const FoldValueArgs& a, const FoldValuePlace& o, const float* mrow, uint8_t* lds, float* lp)
{
    constexpr int NT = FOLD_VALUE_THREADS, ROWS = 16 * RT * 128 / NT, GROUPS = 256 / G, PH = 512 * RT / NT;   // PH: pieces per thread of 128 tokens' weights
    const FoldShape& s = a.s;
    const FoldSource& x = a.x;
    const int tid = threadIdx.x, part = tid >> 7, ch = tid & 127;
    const bool second = o.cblk * 2 + 1 < x.n_slabs;                  // (else the first slab's codes again, and nothing stored)
    // a channel's code lies in two bytes of its row's slab
    const int byte = BITS == 3 ? min(ch * 3 >> 3, 46) : ch * BITS >> 3, shift = ch * BITS - 8 * byte;
    const long long seq = s.b0 + o.b;
    const uint8_t* code = x.codes + seq * x.cap * x.row_bytes + o.cblk * 32 * BITS + byte;
    const int step = second ? 16 * BITS : 0;                         // from the first slab to the second
    const long long meta = seq * x.cap * x.ng_row;
    const int prow = RT == 2 ? ((tid >> 7) & 1) * 16 + (tid & 15) : tid & 15;
    const float M = mrow[prow];
    const float* psrc = a.p + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 4 * FOLD_P_TILE32<RT>;
    const float* msrc = a.mtile + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 16 * RT + prow;
    float4* p = reinterpret_cast<float4*>(lds);                      // 256 tokens' weights, as stored
    float2* sz = reinterpret_cast<float2*>(lds + 8 * FOLD_P_TILE32<RT> * 4);   // and scales and zero-points: [group][token]
    float y[2][ROWS], lacc = 0.0f;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) y[0][r] = y[1][r] = 0.0f;
    for (int t = o.t0; t < o.t1; ++t) {
        __syncthreads();
#pragma unroll 1
        for (int hf = 0; hf < 2; ++hf) {                             // (past the length: the last tile again, which counts for nothing)
            const long long t128 = min(2 * t + hf, (o.len - 1) / FOLD_TILE);
            const float m = msrc[t128 * 16 * RT];
            float4 v[PH];
#pragma unroll
            for (int e = 0; e < PH; ++e) v[e] = *reinterpret_cast<const float4*>(psrc + t128 * 4 * FOLD_P_TILE32<RT> + (e * NT + tid) * 4);
            const bool live = (2 * t + hf) * FOLD_TILE < o.len;
            const float f = m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - M);
#pragma unroll
            for (int e = 0; e < PH; ++e) {
                v[e].x = live ? v[e].x * f : 0.0f; v[e].y = live ? v[e].y * f : 0.0f; v[e].z = live ? v[e].z * f : 0.0f; v[e].w = live ? v[e].w * f : 0.0f;
                lacc += (v[e].x + v[e].y) + (v[e].z + v[e].w);
                p[(hf * PH + e) * NT + tid] = v[e];
            }
        }
#pragma unroll
        for (int e = 0; e < GROUPS * 256 / NT; ++e) {
            const int idx = e * NT + tid, g = min(o.cblk * GROUPS + (idx >> 8), x.ng - 1) >> x.meta_shift;
            const long long at = meta + (long long)min(t * FOLD_VTILE + (idx & 255), o.len - 1) * x.ng_row + g;
            sz[idx] = make_float2(bf16_bits_to_f32(x.scale[at]), bf16_bits_to_f32(x.zero[at]));
        }
        __syncthreads();
        const int ntok = min(o.len - t * FOLD_VTILE, FOLD_VTILE);
        const float2* szg = sz + ch / G * 256;
        // [tokens / 32][half of the slots][pair of quarters]: 8 tokens at a time, the next ones' codes on their way
        auto token_at = [](int k, int q, int i) XQ_INLINE_LAMBDA { return (k >> 2) * 32 + 4 * (4 * ((k >> 1) & 1) + i) + (k & 1) * 2 + q; };
        uint16_t next[2][2][4];
        auto load_codes = [&](int k) XQ_INLINE_LAMBDA {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint8_t* c = code + (long long)min(t * FOLD_VTILE + token_at(k, q, i), o.len - 1) * x.row_bytes;
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        if constexpr (BITS == 3) __builtin_memcpy(&next[n][q][i], c + n * step, 2);
                        else next[n][q][i] = c[n * step];
                    }
                }
        };
        load_codes(0);
        for (int k = 0; k < (ntok + 31) / 32 * 4; ++k) {
            const int k32 = k >> 2, h = (k >> 1) & 1, q0 = (k & 1) * 2;
            float xv[2][2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int at = token_at(k, q, i);
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const float num = (float)((next[n][q][i] >> shift) & ((1u << BITS) - 1u));
                        const float2 m = szg[n * (128 / G) * 256 + at];
                        xv[n][q][i] = NIB && (ch & 1) ? num * m.x : __builtin_fmaf(num, m.x, m.y);   // (8-bit caches: the zero-point goes with the low nibble)
                    }
                }
            load_codes(k + 1);
            asm volatile("" ::: "memory");                           // (the compiler would load them where they are used)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const int row = part * ROWS + r;
                    const float4 w = p[((k32 * RT + (row >> 4)) * 2 + h) * 64 + (row & 15) + 16 * (q0 + q)];
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        y[n][r] = __builtin_fmaf(w.x, xv[n][q][0], y[n][r]);
                        y[n][r] = __builtin_fmaf(w.y, xv[n][q][1], y[n][r]);
                        y[n][r] = __builtin_fmaf(w.z, xv[n][q][2], y[n][r]);
                        y[n][r] = __builtin_fmaf(w.w, xv[n][q][3], y[n][r]);
                    }
                }
        }
    }
    if (o.cblk == 0) fold_denominators<RT, FOLD_VALUE_WAVES>(a, o, lacc, tid < 16 * RT ? mrow[16 * RT + tid] : 0.0f, lp);
    const long long yrow0 = ((long long)o.split * s.nb + o.b) * s.R;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int local = part * ROWS + r, row = o.rb * 16 * RT + local;
            if ((n == 0 || second) && row < s.R)
                a.y[(yrow0 + row) * (x.n_slabs * 128) + (o.cblk * 2 + n) * 128 + ch] = y[n][r] * mrow[16 * RT + local];
        }
    for (int idx = tid; idx < 16 * RT * GROUPS; idx += NT) {        // (the zero-points are in y)
        const int row = o.rb * 16 * RT + idx / GROUPS, g = o.cblk * GROUPS + idx % GROUPS;
        if (row < s.R && g < x.ng) a.yz[(yrow0 + row) * x.ng + g] = 0.0f;
    }
}

// Scales of zero (constant rows: padding, a row not yet written) add nothing to the products, so only the others' spread counts,
// and how far below its row's maximum the weights of their tokens lie.  Tiles without such a scale show that: true if in
// every row they reach to within what the spread leaves of the 12 exponents.  ginv < 0 marks the groups in question.
// Read once more, and only by ranges that hold one: a decode call whose last rows are zero takes 99 us instead of 95 (8 x 4096, 3
// bits), 219 instead of 206 (16 x 8191, 2 bits in groups of 64); in plain fp32 it would be 330 and 700.
template <int NG, int RT>
__device__ __forceinline__ bool fold_zero_scales_harmless(const FoldValueArgs& a, const FoldValuePlace& o, const float* mrow, const float* ginv, int g0, uint8_t* lds)
{
    constexpr int NT = FOLD_VALUE_THREADS, NW = FOLD_VALUE_WAVES, ROWS = 16 * RT, MOST_TILES = 8192;
    const FoldShape& s = a.s;
    const FoldSource& x = a.x;
    const int tid = threadIdx.x, n_tiles = 2 * (o.t1 - o.t0);
    if (n_tiles > MOST_TILES) return false;
    uint8_t* zero_in = lds;                                          // per tile; behind it the row maxima of the other tiles
    float* clean = reinterpret_cast<float*>(lds + MOST_TILES);       // [NT / ROWS][ROWS]
    const uint16_t* sbase = x.scale + (long long)(s.b0 + o.b) * x.cap * x.ng_row;
    for (int i = tid; i < n_tiles; i += NT) zero_in[i] = 0;
    __syncthreads();
    int spread = 0;
#pragma unroll 1
    for (int g = 0; g < NG; ++g) {
        if (!(ginv[g] < 0.0f)) continue;
        int top = 0, low = 255;
        for (int t = o.t0 * FOLD_VTILE + tid; t < min(o.len, o.t1 * FOLD_VTILE); t += NT) {
            const int v = sbase[(long long)t * x.ng_row + ((g0 + g) >> x.meta_shift)];
            if (v == 0) zero_in[t / FOLD_TILE - 2 * o.t0] = 1;       // (several threads, one value)
            else { top = max(top, v >> 7); low = min(low, v >> 7); }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            top = max(top, __shfl_xor(top, off));
            low = min(low, __shfl_xor(low, off));
        }
        int* red = reinterpret_cast<int*>(clean);
        if ((tid & 63) == 0) { red[tid >> 6] = top; red[NW + (tid >> 6)] = low; }
        __syncthreads();
        for (int w = 0; w < NW; ++w) { top = max(top, red[w]); low = min(low, red[NW + w]); }
        spread = max(spread, top - low);
        __syncthreads();
    }
    const int row = tid % ROWS, pt = tid / ROWS;
    const int live_tiles = min(n_tiles, (o.len - o.t0 * FOLD_VTILE + FOLD_TILE - 1) / FOLD_TILE);
    const float* src = a.mtile + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0 + 2 * o.t0) * ROWS + row;
    float m = -INFINITY;
    for (int i = pt; i < live_tiles; i += NT / ROWS)
        if (!zero_in[i]) m = fmaxf(m, src[(long long)i * ROWS]);
    clean[pt * ROWS + row] = m;
    __syncthreads();
    bool ok = true;
    if (tid < ROWS && o.rb * ROWS + tid < s.R) {
        for (int k = 1; k < NT / ROWS; ++k) m = fmaxf(m, clean[k * ROWS + tid]);
        ok = m - mrow[tid] >= (float)(spread - FOLD_SCALE_SPREAD);
    }
    return __syncthreads_and(ok);
}

template <int BITS, int G, int RT, bool NIB>
__global__ __launch_bounds__(FOLD_VALUE_THREADS, 2) void fold_values_kernel(const FoldValueArgs a)
{
    constexpr int GPS = 128 / G, NG = 2 * GPS;                      // groups of a workgroup's two slabs
    constexpr int NT = FOLD_VALUE_THREADS, NW = FOLD_VALUE_WAVES, VT = FOLD_VSTEP;
    constexpr bool SCALED = fold_scaled_codes(BITS);
    constexpr int PPT = SCALED ? 1 : GPS;                           // phases per 32 tokens: where the weights hold the scale, one per group
    constexpr int P_EXP = SCALED ? 15 : 0;                          // softmax weights are cut to fp16 parts times 2^15
    typedef FoldValueLds<RT, NG, NIB, SCALED> L;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FoldShape& s = a.s;
    FoldValuePlace o;
    if (!fold_value_place(s, false, a.cblocks, blockIdx.x, o)) return;
    const FoldSource& x = a.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, q = lane >> 4;
    const int sw = wave & 1, tw = wave >> 1;                        // two slab ways, two token ways
    const int slab = o.cblk * 2 + sw;
    const bool live = slab < x.n_slabs;
    const int g0 = o.cblk * NG;                                     // first group of the workgroup
    const long long seq = s.b0 + o.b;
    const uint16_t* sbase = x.scale + seq * x.cap * x.ng_row;
    const uint16_t* zbase = x.zero + seq * x.cap * x.ng_row;

    // ---- codes: octet n = c16 of the wave's slab for tokens 4 i + q of its 32
    const uint8_t* cbase = x.codes + seq * x.cap * x.row_bytes + (live ? slab : 0) * (16 * BITS);     // (a way without a slab repeats the first)
    const uint32_t oct = BITS == 2 ? 4 * (c16 >> 1) : BITS == 3 ? 3 * c16 - (c16 > 0) : 4 * c16;
    uint32_t voff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) voff[i] = (uint32_t)(4 * i + q) * (uint32_t)x.row_bytes + oct;
    auto load_codes = [&](int k32, uint32_t (&r)[8]) XQ_INLINE_LAMBDA {
        const uint8_t* base = cbase + (long long)k32 * 32 * x.row_bytes;
        uint32_t off[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) off[i] = voff[i];
        if (k32 * 32 + 32 > o.len) {                                // past the length: the last row again (32-bit offsets from the sequence's start)
            base = cbase;
#pragma unroll
            for (int i = 0; i < 8; ++i) off[i] = (uint32_t)min(k32 * 32 + 4 * i + q, o.len - 1) * (uint32_t)x.row_bytes + oct;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (BITS == 3) __builtin_memcpy(&r[i], base + off[i], 4);     // three of these four bytes (lane 0: the first three)
            else r[i] = *reinterpret_cast<const uint32_t*>(base + off[i]);          // (2 bits: shared by two lanes)
        }
    };
    const int v0 = o.t0 * (FOLD_VTILE / VT), v1 = min(o.t1 * (FOLD_VTILE / VT), (o.len + VT - 1) / VT);     // steps of VT tokens
    uint32_t raw[2][8];                                             // codes of the next two times 32 tokens
    load_codes(v0 * (VT / 32) + tw * 2, raw[0]);
    load_codes(v0 * (VT / 32) + tw * 2 + 1, raw[1]);

    float* mrow = reinterpret_cast<float*>(lds + L::M_OFF) + 32 * 16 * RT;
    float* ginv = reinterpret_cast<float*>(lds + L::N_OFF) + 16 * NG;
    // power of two per group that brings the range's largest scale below 2^15 (the fp16 parts of weight times scale)
    {
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        auto max2 = [](uint32_t u, uint32_t v) XQ_INLINE_LAMBDA {
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, u), __builtin_bit_cast(u16x2, v)));
        };
        auto min2 = [](uint32_t u, uint32_t v) XQ_INLINE_LAMBDA {
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, u), __builtin_bit_cast(u16x2, v)));
        };
        uint32_t mx[GPS], mn[GPS];                                  // largest and smallest scales, of pairs of groups
#pragma unroll
        for (int j = 0; j < GPS; ++j) { mx[j] = 0u; mn[j] = 0xFFFFFFFFu; }
        const int tend = min(o.len, o.t1 * FOLD_VTILE);
        // A token's scales lie in a cache line of their own, so what counts is the lines a load touches: all groups in one load
        // where the alignment allows.
        if (x.meta_shift == 0 && g0 + NG <= x.ng && ((reinterpret_cast<uintptr_t>(sbase) | (uint32_t)x.ng_row * 2u) & (2 * NG - 1)) == 0) {
            for (int t = o.t0 * FOLD_VTILE + tid; t < tend; t += 8 * NT) {          // (eight loads at a time, the last token's again)
                uint32_t v[8][GPS];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    __builtin_memcpy(v[k], __builtin_assume_aligned(sbase + (long long)min(t + k * NT, tend - 1) * x.ng_row + g0, 2 * NG), 2 * NG);
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int j = 0; j < GPS; ++j) { mx[j] = max2(mx[j], v[k][j]); mn[j] = min2(mn[j], v[k][j]); }
            }
        } else {
            for (int t = o.t0 * FOLD_VTILE + tid; t < tend; t += NT)
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    if (g0 + g < x.ng) {
                        const uint32_t v = (uint32_t)sbase[(long long)t * x.ng_row + ((g0 + g) >> x.meta_shift)] << (16 * (g & 1));
                        mx[g >> 1] = max2(mx[g >> 1], v);
                        mn[g >> 1] = min2(mn[g >> 1], v | (0xFFFFu << (16 * (~g & 1))));
                    }
        }
#pragma unroll
        for (int j = 0; j < GPS; ++j) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                mx[j] = max2(mx[j], (uint32_t)__shfl_xor((int)mx[j], off));
                mn[j] = min2(mn[j], (uint32_t)__shfl_xor((int)mn[j], off));
            }
            if (lane == 0) {
                reinterpret_cast<uint32_t*>(lds + L::N_OFF)[wave * NG + 2 * j] = mx[j];
                reinterpret_cast<uint32_t*>(lds + L::N_OFF)[wave * NG + 2 * j + 1] = mn[j];
            }
        }
        fold_row_maxima<RT, FOLD_RANGE_TOP, NT>(s, a.mtile, o.b, o.rb, reinterpret_cast<float*>(lds + L::M_OFF), mrow, 2 * o.t0, 2 * o.t1);
        if (tid < NG) {
            const uint32_t* src = reinterpret_cast<const uint32_t*>(lds + L::N_OFF) + (tid & ~1);
            uint32_t m = 0u, n = 0xFFFFFFFFu;
#pragma unroll
            for (int w = 0; w < NW; ++w) { m = max2(m, src[w * NG]); n = min2(n, src[w * NG + 1]); }
            const int hs = 16 * (tid & 1), top = (int)(m >> hs & 0xFFFFu) >> 7, low = (int)(n >> hs & 0xFFFFu) >> 7;
            // largest scale < 2^(top - 126): times 2^(141 - top) it is below 2^15.  (0: for fold_values_plain; negative: scales too
            // far apart, if zeros count.)
            const float f = ldexpf(1.0f, min(141 - top, 120));
            ginv[tid] = top >= 255 ? 0.0f : top - low > FOLD_SCALE_SPREAD ? -f : f;
        }
    }
    __syncthreads();
    bool wide = false, never = false;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        wide |= ginv[g] <= 0.0f;
        never |= ginv[g] == 0.0f;
    }
    if (wide && !never) {
        wide = !fold_zero_scales_harmless<NG, RT>(a, o, mrow, ginv, g0, lds);
        if (!wide && tid < NG) ginv[tid] = fabsf(ginv[tid]);
        __syncthreads();
    }
    if (wide) {
        fold_values_plain<BITS, G, RT, NIB>(a, o, mrow, lds, reinterpret_cast<float*>(lds + L::L_OFF));
        return;
    }

    // ---- staging: thread -> softmax weights (always of the same row) and (token, group) pairs
    static_assert(VT == FOLD_TILE, "a step has one stored maximum per row");
    constexpr int NP = 512 * RT / NT;                               // 16-byte pieces per thread and step
    const int prow = RT == 2 ? ((wave >> 1) & 1) * 16 + c16 : c16;
    const float M = mrow[prow];
    const float* psrc = a.p + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 4 * FOLD_P_TILE32<RT>;
    const float* msrc = a.mtile + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 16 * RT + prow;
    float4 pv[NP];
    float fm;
    constexpr int NE = VT * NG / NT;                       // (token, group) pairs per thread: 1 or 2
    const int eg = tid % NG, et = tid / NG;                         // group and first token of this thread's pairs
    uint32_t sv[NE], zv[NE];
    const uint16_t* sgrp = sbase + (min(g0 + eg, x.ng - 1) >> x.meta_shift);
    const uint16_t* zgrp = zbase + (min(g0 + eg, x.ng - 1) >> x.meta_shift);
    const float my_ginv = ginv[eg];
    auto load_stage = [&](int t) XQ_INLINE_LAMBDA {
        fm = msrc[(long long)t * 16 * RT];
#pragma unroll
        for (int e = 0; e < NP; ++e) pv[e] = *reinterpret_cast<const float4*>(psrc + (long long)t * (VT / 32) * FOLD_P_TILE32<RT> + (e * NT + tid) * 4);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const uint32_t at = (uint32_t)min(t * VT + et + e * (NT / NG), o.len - 1) * (uint32_t)x.ng_row;
            sv[e] = sgrp[at];
            zv[e] = zgrp[at];
        }
    };
    // what a thread's pieces are: four adjacent slots of row prow and token quarter q of 32 tokens
    auto piece = [&](int e, int& t32, int& rt, int& part) XQ_INLINE_LAMBDA {
        const int k = e * NW + wave;
        part = k & 1; rt = (k >> 1) & (RT - 1); t32 = k / (2 * RT);
    };
    float lacc = 0.0f, az[NG];                                      // of row prow: sums of the weights, and of weight times rest per group
#pragma unroll
    for (int g = 0; g < NG; ++g) az[g] = 0.0f;
    auto write_stage = [&](int buf) XQ_INLINE_LAMBDA {
        const float f = fm == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(fm - M) * (float)(1 << P_EXP);
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            float4& v = pv[e];
            v.x *= f; v.y *= f; v.z *= f; v.w *= f;
            if (o.cblk == 0) lacc += (v.x + v.y) + (v.z + v.w);
            if constexpr (SCALED) {
                int t32, rt, part;
                piece(e, t32, rt, part);
                const xq_f32x2 a2 = {v.x, v.y}, b2 = {v.z, v.w};
                const xq_f16x2 ah = __builtin_convertvector(a2, xq_f16x2), bh = __builtin_convertvector(b2, xq_f16x2);
                const xq_f32x2 ar = {v.x - (float)ah.x, v.y - (float)ah.y}, br = {v.z - (float)bh.x, v.w - (float)bh.y};
                const xq_f16x2 al = __builtin_convertvector(ar, xq_f16x2), bl = __builtin_convertvector(br, xq_f16x2);
                uint8_t* dst = lds + L::P_OFF + buf * L::P_BYTES + (t32 * RT + rt) * 2048 + lane * 16 + part * 8;
                *reinterpret_cast<uint2*>(dst) = make_uint2(__builtin_bit_cast(uint32_t, ah), __builtin_bit_cast(uint32_t, bh));
                *reinterpret_cast<uint2*>(dst + 1024) = make_uint2(__builtin_bit_cast(uint32_t, al), __builtin_bit_cast(uint32_t, bl));
            } else {
                *reinterpret_cast<float4*>(lds + L::P_OFF + buf * L::P_BYTES + (e * NT + tid) * 16) = v;
            }
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int tok = et + e * (NT / NG), t32 = tok & 31, at = (tok & ~31) + (t32 & 3) * 8 + (t32 >> 2);
            uint8_t* grp = lds + L::SZ_OFF + buf * L::SZ_BYTES + eg * L::GROUP_BYTES;
            const float sf = bf16_bits_to_f32(sv[e]);
            float rest;
            const float zi = fold_integer_zero(sf, bf16_bits_to_f32(zv[e]), NIB ? 255.0f : (float)((1 << BITS) - 1), rest);
            reinterpret_cast<float*>(grp + L::REST)[at] = rest;
            uint16_t* zo = reinterpret_cast<uint16_t*>(grp + L::HALFS);
            if constexpr (SCALED) zo[L::H_STRIDE + at] = (uint16_t)f16_bits(sf * my_ginv);
            else reinterpret_cast<float*>(grp)[at] = sf * my_ginv;
            if constexpr (NIB) {
                const float zh = floorf(zi * (1.0f / 16.0f));
                zo[at] = (uint16_t)f16_bits((zi - 16.0f * zh) * (-1.0f / FOLD_CODE_UNIT));
                zo[L::H_STRIDE + at] = (uint16_t)f16_bits(zh * (-1.0f / FOLD_CODE_UNIT));
            } else {
                zo[at] = (uint16_t)f16_bits(zi * (-1.0f / FOLD_CODE_UNIT));
            }
        }
    };
    // weight times rest, from the weights that the thread still holds of the step staged last
    auto add_rests = [&](int buf) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            int t32, rt, part;
            piece(e, t32, rt, part);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const float4 r = *reinterpret_cast<const float4*>(lds + L::SZ_OFF + buf * L::SZ_BYTES + g * L::GROUP_BYTES + L::REST +
                                                                  (t32 * 32 + q * 8 + part * 4) * 4);
                az[g] = __builtin_fmaf(pv[e].x, r.x, az[g]);
                az[g] = __builtin_fmaf(pv[e].y, r.y, az[g]);
                az[g] = __builtin_fmaf(pv[e].z, r.z, az[g]);
                az[g] = __builtin_fmaf(pv[e].w, r.w, az[g]);
            }
        }
    };

    const uint32_t sel0 = BITS == 2 ? (c16 & 1 ? 0x07060302u : 0x05040100u) : c16 ? 0x06050201u : 0x05040100u, sel1 = c16 ? 0x07060302u : 0x06050201u;
    const bool lower = c16 < 8;

    f32x4 acc[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[rt][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // A wave has 32 tokens twice per step, in phases of 8 / PPT column tiles times 2 RT matrix instructions.  While a phase's
    // matrix instructions run, the vector ALU unpacks the next column tile and, with 4-bit codes, forms the next phase's weights,
    // a little behind every matrix instruction (fences keep it there).
    constexpr int KPP = 8 / PPT, NSLOT = KPP * 2 * RT, NSUB = SCALED ? 0 : RT * 8, START = NSLOT / 4;
    uint32_t m0[4], m1[4], F[2][4];
    // weights (of the running and the next 32 tokens if SCALED, else of the running and the next phase); -zi, scales or -zi of odd codes
    uint4 wh[2][RT], wl[2][RT], zi[2][NIB || SCALED ? 2 : 1];
    float pr[RT][8], sc[8];                                         // of the next phase
    const int lane_group = sw * GPS + (GPS == 2 ? c16 >> 3 : 0);
    auto merge_pairs = [&](uint32_t (&r)[8]) XQ_INLINE_LAMBDA {
        // (here and not earlier: merged where they are loaded, the codes would be waited for there)
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(r[i]));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (BITS == 2) { m0[j] = perm_bytes(r[2 * j + 1], r[2 * j], sel0); m1[j] = 0u; }
            else if constexpr (BITS == 3) { m0[j] = perm_bytes(r[2 * j + 1], r[2 * j], sel0); m1[j] = perm_bytes(r[2 * j + 1], r[2 * j], sel1); }
            else { m0[j] = perm_bytes(r[2 * j + 1], r[2 * j], 0x05040100u); m1[j] = perm_bytes(r[2 * j + 1], r[2 * j], 0x07060302u); }
            if constexpr (PPT == 2) {
                // (4 bits) lanes n and n + 8 exchange half octets: codes 0-3 then belong to the first group, 4-7 to the second
                const uint32_t keep = lower ? m0[j] : m1[j], got = dpp_u32<0x128 /* row_ror:8 */>(lower ? m1[j] : m0[j]);
                m0[j] = lower ? keep : got;
                m1[j] = lower ? got : keep;
            }
        }
    };
    // the next phase's data out of LDS: PH = step PPT + group (SCALED: a lane's octet lies in one group, whose numbers it takes)
    auto read_phase = [&](auto PH, int buf) XQ_INLINE_LAMBDA {
        constexpr int st = decltype(PH)::value / PPT, g = decltype(PH)::value % PPT, n = decltype(PH)::value & 1;
        const int k32 = tw * 2 + st;
        if constexpr (g == 0)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const uint8_t* src = lds + L::P_OFF + buf * L::P_BYTES + (k32 * RT + rt) * 2048 + lane * 16;
                if constexpr (SCALED) {
                    wh[st][rt] = *reinterpret_cast<const uint4*>(src);
                    wl[st][rt] = *reinterpret_cast<const uint4*>(src + 1024);
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float4 v = *reinterpret_cast<const float4*>(src + h * 1024);
                        pr[rt][4 * h] = v.x; pr[rt][4 * h + 1] = v.y; pr[rt][4 * h + 2] = v.z; pr[rt][4 * h + 3] = v.w;
                    }
                }
            }
        const uint8_t* grp = lds + L::SZ_OFF + buf * L::SZ_BYTES + (SCALED ? lane_group : sw * GPS + g) * L::GROUP_BYTES;
        if constexpr (!SCALED)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 a4 = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(grp) + k32 * 32 + q * 8 + 4 * h);
                sc[4 * h] = a4.x; sc[4 * h + 1] = a4.y; sc[4 * h + 2] = a4.z; sc[4 * h + 3] = a4.w;
            }
#pragma unroll
        for (int k = 0; k < (NIB || SCALED ? 2 : 1); ++k)
            zi[n][k] = *reinterpret_cast<const uint4*>(grp + L::HALFS + (k * L::H_STRIDE + k32 * 32 + q * 8) * 2);
    };
    // weights of the next phase, piece SUB: (row tile, token pair) products and top parts, then low parts
    auto set_dword = [](uint4& v, auto J, uint32_t x) XQ_INLINE_LAMBDA {
        constexpr int j = decltype(J)::value;
        if constexpr (j == 0) v.x = x; else if constexpr (j == 1) v.y = x; else if constexpr (j == 2) v.z = x; else v.w = x;
    };
    auto weight_piece = [&](auto PH, auto SUB) XQ_INLINE_LAMBDA {
        constexpr int n = decltype(PH)::value & 1;
        constexpr int sub = decltype(SUB)::value, rt = sub / 8, j = (sub / 2) & 3;
        const float p0 = pr[rt][2 * j], p1 = pr[rt][2 * j + 1], s0 = sc[2 * j], s1 = sc[2 * j + 1];
        if constexpr ((sub & 1) == 0) {
            const xq_f32x2 w = {p0 * s0, p1 * s1};
            set_dword(wh[n][rt], std::integral_constant<int, j>{}, __builtin_bit_cast(uint32_t, __builtin_convertvector(w, xq_f16x2)));
        } else {
            const uint32_t hb = j == 0 ? wh[n][rt].x : j == 1 ? wh[n][rt].y : j == 2 ? wh[n][rt].z : wh[n][rt].w;
            const xq_f16x2 top = __builtin_bit_cast(xq_f16x2, hb);
            const xq_f16x2 low = {(_Float16)__builtin_fmaf(p0, s0, -(float)top.x), (_Float16)__builtin_fmaf(p1, s1, -(float)top.y)};
            set_dword(wl[n][rt], std::integral_constant<int, j>{}, __builtin_bit_cast(uint32_t, low));
        }
    };
    auto component = [](const uint4& v, auto J) XQ_INLINE_LAMBDA {
        constexpr int j = decltype(J)::value;
        return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
    };
    // operand dword J of column tile K (its codes in m0, m1), with the integer zero-points of phase parity N, and then the scales
    auto unpack = [&](auto K, auto J, auto N) XQ_INLINE_LAMBDA {
        constexpr int k = decltype(K)::value, j = decltype(J)::value, n = decltype(N)::value;
        F[k & 1][j] = fold_code<BITS, k>(m0[j], m1[j], component(zi[n][NIB ? k & 1 : 0], J));
    };
    auto scale = [&](auto K, auto J, auto N) XQ_INLINE_LAMBDA {
        constexpr int k = decltype(K)::value, j = decltype(J)::value, n = decltype(N)::value;
        if constexpr (SCALED)
            F[k & 1][j] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(xq_f16x2, F[k & 1][j]) * __builtin_bit_cast(xq_f16x2, component(zi[n][1], J)));
    };
    // a column tile's four dwords over the slots of the one before; what a dword's scaling reads was not written right before it
    auto unpack_slot = [&](auto K, auto IN, auto N) XQ_INLINE_LAMBDA {
        constexpr int in = decltype(IN)::value;
        constexpr std::integral_constant<int, 0> j0{};
        constexpr std::integral_constant<int, 1> j1{};
        constexpr std::integral_constant<int, 2> j2{};
        constexpr std::integral_constant<int, 3> j3{};
        if constexpr (RT == 2) {
            if constexpr (in == 0) { unpack(K, j0, N); unpack(K, j1, N); }
            else if constexpr (in == 1) { scale(K, j0, N); unpack(K, j2, N); }
            else if constexpr (in == 2) { scale(K, j1, N); unpack(K, j3, N); }
            else { scale(K, j2, N); scale(K, j3, N); }
        } else {
            if constexpr (in == 0) { unpack(K, j0, N); unpack(K, j1, N); unpack(K, j2, N); scale(K, j0, N); }
            else { unpack(K, j3, N); scale(K, j1, N); scale(K, j2, N); scale(K, j3, N); }
        }
    };
    auto phase = [&](auto PH, int nbuf) XQ_INLINE_LAMBDA {
        constexpr int ph = decltype(PH)::value, st = ph / PPT, g = ph % PPT, n = ph & 1, nw = SCALED ? st : n, nph = (ph + 1) % (2 * PPT);
        read_phase(std::integral_constant<int, nph>{}, nbuf);
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NSLOT>([&](auto M) XQ_INLINE_LAMBDA {
            constexpr int m = decltype(M)::value, kk = m / (2 * RT), k = g * KPP + kk, in = m % (2 * RT), rt = in % RT;
            const uint32_t* f = F[k & 1];
            acc[rt][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, in < RT ? wl[nw][rt] : wh[nw][rt]), as_frag(f[0], f[1], f[2], f[3]),
                                                                acc[rt][k], 0, 0, 0);
            // the next column tile; the first one of the next step waits for its codes here
            if constexpr (k == 7 && in == 0) merge_pairs(raw[st ^ 1]);
            unpack_slot(std::integral_constant<int, (k + 1) & 7>{}, std::integral_constant<int, in>{}, std::integral_constant<int, kk == KPP - 1 ? n ^ 1 : n>{});
            constexpr int b0 = m < START ? 0 : (m - START) * NSUB / (NSLOT - START), b1 = m < START ? 0 : (m + 1 - START) * NSUB / (NSLOT - START);
            static_for<b0, b1>([&](auto SUB) XQ_INLINE_LAMBDA { weight_piece(std::integral_constant<int, nph>{}, SUB); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    load_stage(v0);
    write_stage(0);
    __syncthreads();
    add_rests(0);
    load_stage(min(v0 + 1, v1 - 1));
    read_phase(std::integral_constant<int, 0>{}, 0);
    static_for<0, NSUB>([&](auto SUB) XQ_INLINE_LAMBDA { weight_piece(std::integral_constant<int, 0>{}, SUB); });
    merge_pairs(raw[0]);
    static_for<0, 2 * RT>([&](auto IN) XQ_INLINE_LAMBDA { unpack_slot(std::integral_constant<int, 0>{}, IN, std::integral_constant<int, 0>{}); });
    // One barrier per step, before its last phase: by then every wave has read all of the step out of LDS (a phase reads
    // the next one's data), so the step after the next may overwrite it, and the next step, written since the barrier
    // before, may be read by the last phase.
    // No load stands under a condition: where paths with and without one meet, the compiler waits for all that are in flight
    // (a whole latency per step: 4 x 32768 tokens of 2 bits 118 us, 115 without).  The last loads are repeated instead.
    for (int t = v0; t < v1 - 1; ++t) {
        const int buf = (t - v0) & 1;
        // (codes are merged before their phases start: their registers take those of the step after the next)
        load_codes((t + 1) * (VT / 32) + tw * 2, raw[0]);
        static_for<0, PPT>([&](auto PH) XQ_INLINE_LAMBDA { phase(PH, buf); });
        load_codes((t + 1) * (VT / 32) + tw * 2 + 1, raw[1]);
        static_for<PPT, 2 * PPT - 1>([&](auto PH) XQ_INLINE_LAMBDA { phase(PH, buf); });
        write_stage(buf ^ 1);
        __syncthreads();
        add_rests(buf ^ 1);
        load_stage(min(t + 2, v1 - 1));
        phase(std::integral_constant<int, 2 * PPT - 1>{}, buf ^ 1);
    }
    static_for<0, 2 * PPT>([&](auto PH) XQ_INLINE_LAMBDA { phase(PH, (v1 - 1 - v0) & 1); });     // (the last one prepares nothing that is used)
    __syncthreads();

    // softmax denominators: once per row block and split
    constexpr float P_UNIT = 1.0f / (1 << P_EXP);
    if (o.cblk == 0)
        fold_denominators<RT, NW>(a, o, lacc, tid < 16 * RT ? mrow[16 * RT + tid] * P_UNIT : 0.0f, reinterpret_cast<float*>(lds + L::L_OFF));
    // row factors of what this thread stores below (the sums overwrite them)
    static_assert(16 * RT * NG <= NT, "one rest sum per thread");
    constexpr int MEET = FOLD_MEET<RT, NW>;
    const float zfac = mrow[16 * RT + (tid / (16 * NG)) % RT * 16 + (tid & 15)] * P_UNIT;
    float yfac[MEET][4];
#pragma unroll
    for (int i = 0; i < MEET; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) yfac[i][r] = mrow[16 * RT + (((tw + i * (NW / 2)) >> 1) % RT) * 16 + 4 * q + r] * P_UNIT;
    // the rests' sums meet in LDS, then the accumulators
    const float inv_g[2] = {ginv[SCALED ? lane_group : sw * GPS], ginv[SCALED ? lane_group : sw * GPS + GPS - 1]};
    __syncthreads();
    float* red = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        float z = az[g];
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        if (q == 0) red[(wave * NG + g) * 16 + c16] = z;
    }
    __syncthreads();
    const long long yrow0 = ((long long)o.split * s.nb + o.b) * s.R;
    if (tid < 16 * RT * NG) {
        const int r16 = tid & 15, g = (tid >> 4) % NG, rt = tid / (16 * NG);
        const int row = o.rb * 16 * RT + rt * 16 + r16;
        float z = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if (RT == 1 || ((w >> 1) & 1) == rt) z += red[(w * NG + g) * 16 + r16];
        if (row < s.R && g0 + g < x.ng) a.yz[(yrow0 + row) * x.ng + g0 + g] = z * zfac;
    }
    __syncthreads();
    f32x4 t[MEET][4];
    fold_meet<RT, NW>(acc, lds, wave, lane, t);
    if (live && tw < 2 * RT) {
#pragma unroll
        for (int i = 0; i < MEET; ++i) {
            const int h = tw + i * (NW / 2), rt = h >> 1, kg = h & 1;
            const int ch = PPT == 1 ? 8 * c16 + 4 * kg : 64 * kg + 8 * (c16 & 7) + 4 * (c16 >> 3);
            const float f = FOLD_CODE_UNIT / (PPT == 2 && kg ? inv_g[1] : inv_g[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = o.rb * 16 * RT + rt * 16 + 4 * q + r;
                const float fr = f * yfac[i][r];
                if (row < s.R)
                    *reinterpret_cast<float4*>(a.y + (yrow0 + row) * (x.n_slabs * 128) + slab * 128 + ch) =
                        make_float4(t[i][0][r] * fr, t[i][1][r] * fr, t[i][2][r] * fr, t[i][3][r] * fr);
            }
        }
    }
}

// the same over bf16 rows: no scales and no offsets, the softmax weights in three bf16 parts (made once per workgroup)
template <int RT>
struct FoldValueDenseLds {
    static constexpr int W_BYTES = 8 * RT * 3 * 1024;                           // [tile32][rt][part][lane 64][16 B]
    static constexpr int M_OFF = 2 * W_BYTES;
    static constexpr int L_OFF = M_OFF + 16 * RT * 4 * 17;
    static constexpr int LOOP = L_OFF + 8 * 16 * RT * 4;
    static constexpr int RED = 8 * RT * 8 * 1024;
    static constexpr int TOTAL = LOOP > RED ? LOOP : RED;
};
template <int RT>
__device__ __forceinline__ void fold_values_dense(const FoldValueArgs& a, const FoldSource& x, bool window, uint8_t* lds)
{
    typedef FoldValueDenseLds<RT> L;
    const FoldShape& s = a.s;
    FoldValuePlace o;
    if (!fold_value_place(s, window, a.cblocks, blockIdx.x, o)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, q = lane >> 4;
    const int sw = wave & 1, tw = wave >> 1;
    const int slab = o.cblk * 2 + sw;
    const bool live = slab < x.n_slabs;
    float* mrow = reinterpret_cast<float*>(lds + L::M_OFF) + 16 * 16 * RT;
    fold_row_maxima<RT>(s, a.mtile, o.b, o.rb, reinterpret_cast<float*>(lds + L::M_OFF), mrow);

    constexpr int NP = 2 * RT;
    const int prow = RT == 2 ? ((wave >> 1) & 1) * 16 + c16 : c16;
    const float M = mrow[prow];
    const float* psrc = a.p + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 4 * FOLD_P_TILE32<RT>;
    // (maxima per 64 tokens: the window of blocks of 64 holds fewer, all in the first half of its first tile)
    const float* msrc = a.mtile + ((((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) << s.mhalf) * 16 * RT + prow;
    float4 pv[NP];
    float fm[2];
    auto load_stage = [&](int t) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int t128 = 2 * t + hf;
            const bool ok = t128 * FOLD_TILE < o.len;
            fm[hf] = ok ? msrc[(long long)(t128 << s.mhalf) * 16 * RT] : -INFINITY;
#pragma unroll
            for (int k = 0; k < RT; ++k) {
                const int e = hf * RT + k;
                pv[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (ok) pv[e] = *reinterpret_cast<const float4*>(psrc + (long long)t * 8 * FOLD_P_TILE32<RT> + (e * 512 + tid) * 4);
            }
        }
    };
    float lacc = 0.0f;
    auto write_stage = [&](int buf) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const float f = fm[hf] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(fm[hf] - M);
#pragma unroll
            for (int k = 0; k < RT; ++k) {
                const int e = hf * RT + k;
                const float v[4] = {pv[e].x * f, pv[e].y * f, pv[e].z * f, pv[e].w * f};
                lacc += (v[0] + v[1]) + (v[2] + v[3]);
                uint32_t h[4], m[4], l[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) split_bf16x3(v[i], h[i], m[i], l[i]);
                // piece e 512 + tid of [tile32][rt][half of the slots][lane]
                const int idx = e * 512 + tid, hs = (idx >> 6) & 1, blk = idx >> 7;
                uint8_t* dst = lds + buf * L::W_BYTES + blk * 3072 + lane * 16 + hs * 8;
                *reinterpret_cast<uint2*>(dst) = make_uint2(pack_hi16(h[0], h[1]), pack_hi16(h[2], h[3]));
                *reinterpret_cast<uint2*>(dst + 1024) = make_uint2(pack_hi16(m[0], m[1]), pack_hi16(m[2], m[3]));
                *reinterpret_cast<uint2*>(dst + 2048) = make_uint2(pack_hi16(l[0], l[1]), pack_hi16(l[2], l[3]));
            }
        }
    };
    const uint8_t* xbase = reinterpret_cast<const uint8_t*>(x.rows) + (long long)(s.b0 + o.b) * x.cap * x.row_bytes + (live ? slab : 0) * 256;
    uint4 raw[2][8];
    uint32_t voff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) voff[i] = (uint32_t)(4 * i + q) * (uint32_t)x.row_bytes + c16 * 16;
    auto load_rows = [&](int k32, uint4 (&r)[8]) XQ_INLINE_LAMBDA {
        const uint8_t* base = xbase + (long long)k32 * 32 * x.row_bytes;
        uint32_t off[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) off[i] = voff[i];
        if (k32 * 32 + 32 > o.len) {                                // past the length: the last row again
            base = xbase;
#pragma unroll
            for (int i = 0; i < 8; ++i) off[i] = (uint32_t)min(k32 * 32 + 4 * i + q, o.len - 1) * (uint32_t)x.row_bytes + c16 * 16;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = *reinterpret_cast<const uint4*>(base + off[i]);
    };
    f32x4 acc[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[rt][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto step = [&](const uint8_t* wb, int k32, const uint4 (&r)[8]) XQ_INLINE_LAMBDA {
        uint4 w[RT][3];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int k = 0; k < 3; ++k) w[rt][k] = *reinterpret_cast<const uint4*>(wb + ((k32 * RT + rt) * 3 + k) * 1024 + lane * 16);
        static_for<0, 8>([&](auto K) XQ_INLINE_LAMBDA {
            constexpr int k = decltype(K)::value;
            uint32_t d[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t x0[4] = {r[2 * j].x, r[2 * j].y, r[2 * j].z, r[2 * j].w};
                const uint32_t x1[4] = {r[2 * j + 1].x, r[2 * j + 1].y, r[2 * j + 1].z, r[2 * j + 1].w};
                d[j] = perm_bytes(x1[k >> 1], x0[k >> 1], (k & 1) ? 0x07060302u : 0x05040100u);
            }
            const bf16x8 xf = __builtin_bit_cast(bf16x8, make_uint4(d[0], d[1], d[2], d[3]));
#pragma unroll
            for (int p = 2; p >= 0; --p)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[rt][p]), xf, acc[rt][k], 0, 0, 0);
        });
    };
    load_stage(o.t0);
    load_rows(o.t0 * 8 + tw * 2, raw[0]);
    load_rows(o.t0 * 8 + tw * 2 + 1, raw[1]);
    write_stage(0);
    __syncthreads();
    for (int t = o.t0; t < o.t1; ++t) {
        const int buf = (t - o.t0) & 1;
        const bool more = t + 1 < o.t1;
        if (more) load_stage(t + 1);
        const uint8_t* wb = lds + buf * L::W_BYTES;
        if (live) step(wb, tw * 2, raw[0]);
        if (more) load_rows((t + 1) * 8 + tw * 2, raw[0]);
        if (live) step(wb, tw * 2 + 1, raw[1]);
        if (more) load_rows((t + 1) * 8 + tw * 2 + 1, raw[1]);
        if (more) write_stage(buf ^ 1);
        __syncthreads();
    }
    if (o.cblk == 0) {
        fold_denominators<RT>(a, o, lacc, 1.0f, reinterpret_cast<float*>(lds + L::L_OFF));
        __syncthreads();
    }
    f32x4 t[1][4];
    fold_meet<RT, 8>(acc, lds, wave, lane, t);
    if (live && tw < 2 * RT) {
        const int rt = tw >> 1, kg = tw & 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = o.rb * 16 * RT + rt * 16 + 4 * q + r;
            if (row < s.R)
                *reinterpret_cast<float4*>(a.y + (((long long)o.split * s.nb + o.b) * s.R + row) * (x.n_slabs * 128) + slab * 128 + 8 * c16 + 4 * kg) =
                    make_float4(t[0][0][r], t[0][1][r], t[0][2][r], t[0][3][r]);
        }
    }
}

template <int RT>
__global__ __launch_bounds__(512) void fold_values_dense_kernel(const FoldValueArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    fold_values_dense<RT>(a, a.x, false, lds);
}

#include "folded_per_channel.hpp"

// =====================================================================================================================
// Output projection.  A workgroup takes one KV head, 32 query columns and a few slabs: it sums y over the token splits,
// adds the offsets of the groups, and multiplies by the slabs' share of Wv_h, the prepared stream's fragments as they
// are (fp16 ones are cut to bf16, exactly) against y in three bf16 parts.  Bound by the latency of three rounds of loads (the
// splits in use, y, the third slab's weights) and by reading the value half of the stream once.  No load of the sums stands
// under a condition, which would make it a wait of its own: 32 splits of 3 x 13012 tokens, d = 1024, 18.3 / 12.0 us so (and
// fold_finish_kernel 9.0 / 5.2), 4 splits of 4 x 4096 tokens, d = 4096, 16.1 / 13.8.
// =====================================================================================================================
struct FoldOutArgs {
    FoldWeights w;
    FoldShape s;
    const float* y;
    const float* yz;
    float* part;                         // [chunks][nb][R][128]
    int n_slabs, ng, group, chunk_slabs;
    UnpackTable tab;
};

constexpr int FO_MAX_SLABS = 4;
constexpr int FO_STRIDE = FO_MAX_SLABS * 128 + 4;
constexpr int FO_LDS = 32 * FO_STRIDE * 4;               // 66 KiB, reused for the waves' partial sums (64 KiB)
constexpr int FO_MAX_GROUPS = FO_MAX_SLABS * 2;

template <bool DENSE>
__global__ __launch_bounds__(512, 4) void fold_output_kernel(const FoldOutArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float* yl = reinterpret_cast<float*>(lds);
    const FoldShape& s = a.s;
    const int chunk = blockIdx.x, h = blockIdx.y, cb = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, c32 = lane & 31;
    const int gq = s.Hq / s.Hkv, ncol = s.nb * gq;
    const int slab0 = chunk * a.chunk_slabs, ns = min(a.chunk_slabs, a.n_slabs - slab0);
    const int d = a.n_slabs * 128;
    const long long split_stride = (long long)s.nb * s.R;
    // the weights first: they come out of HBM while the sums below wait for what the value kernel left (a wave's k-step: the
    // same place in every slab)
    const int sh = a.w.pair ? h >> 1 : h, nb0 = a.w.pair ? 4 * (h & 1) : 4;
    const uint8_t* wsrc = a.w.stream + (long long)sh * a.w.head_bytes + lane * 16;
    const int shift = DENSE ? 0 : a.w.shift[sh];
    uint4 wf[2][4];                                                  // (two slabs ahead: with all four two workgroups do not fit a CU)
    auto load_weights = [&](int sl, uint4 (&f)[4]) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            int pos = (slab0 + min(sl, ns - 1)) * 8 + wave + (DENSE ? 0 : COL_BLOCK_LAG_MAX - (nb0 + nb));
            if (pos >= a.w.n16) pos -= a.w.n16;
            f[nb] = *reinterpret_cast<const uint4*>(wsrc + (long long)pos * 8192 + (nb0 + nb) * 1024);
        }
    };
    load_weights(0, wf[0]);
    load_weights(1, wf[1]);
    auto row_of = [&](int col, int& b) -> int {
        b = col / gq;
        return h * gq + (col - b * gq);
    };
    __shared__ float zl[32 * FO_MAX_GROUPS];
    __shared__ int crow[32], cused[32];                              // per column: row of y, splits (and 256: the window's)
    __shared__ __attribute__((aligned(16))) float unit[32];          // coded streams: what a code's weight row is divided by
    if (tid < 32) {
        if constexpr (!DENSE) unit[tid] = __uint_as_float((uint32_t)(127 - a.tab.wexp_of_code[tid]) << 23);
        int b = 0, used = 0, row = 0;
        bool window = false;
        if (cb * 32 + tid < ncol) {
            row = row_of(cb * 32 + tid, b);
            fold_used_splits(s, b, used, window);
        }
        crow[tid] = b * s.R + row;
        cused[tid] = used + (window ? 256 : 0);
    }
    __syncthreads();
    // the groups' offsets: [column][group of the workgroup]
    const bool offsets = !DENSE && a.ng;
    const int cg = offsets ? ns * 128 / a.group : 1;
    if (offsets && tid < 32 * cg) {
        const int col = tid / cg, g = slab0 * 128 / a.group + tid - col * cg, used = cused[col] & 255, n = used + (cused[col] >> 8);
        float z[4] = {};                                             // (short chains of roundings, here and below)
        for (int k = 0; k < n; k += 8) {
            float t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j] = a.yz[((k + j < used ? k + j : n > used ? s.splits - 1 : used - 1) * split_stride + crow[col]) * a.ng + g];
#pragma unroll
            for (int j = 0; j < 8; ++j) z[j & 3] += k + j < n ? t[j] : 0.0f;
        }
        zl[col * FO_MAX_GROUPS + tid - col * cg] = (z[0] + z[1]) + (z[2] + z[3]);
    }
    __syncthreads();
    // 16-byte pieces [column][channel / 4], eight loads of a thread at a time: two pieces and four splits, or one piece and eight
    // splits where every thread has one at most.  (Columns that hold no query stay as they are: nothing of theirs is stored.)
    const int pieces = min(32, ncol - cb * 32) * ns * 32;
    auto sum_pieces = [&](auto PIECES) XQ_INLINE_LAMBDA {
        constexpr int P = decltype(PIECES)::value, K = 8 / P;
        for (int p0 = tid; p0 < pieces; p0 += P * 512) {
            const float* src[P];
            int col[P], c4[P], n[P], last[P], most = 0;
            float4 v[4][P] = {};
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int idx = min(p0 + i * 512, pieces - 1);
                col[i] = idx / (ns * 32);
                c4[i] = idx - col[i] * (ns * 32);
                const int used = cused[col[i]] & 255;
                n[i] = used + (cused[col[i]] >> 8);
                most = max(most, n[i]);
                last[i] = n[i] > used ? s.splits - 1 : used - 1;     // where the last of them lies
                src[i] = a.y + (long long)crow[col[i]] * d + slab0 * 128 + 4 * c4[i];
            }
            for (int k = 0; k < most; k += K) {
                float4 t[K][P];
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int i = 0; i < P; ++i)
                        t[j][i] = *reinterpret_cast<const float4*>(src[i] + (k + j < n[i] - 1 ? k + j : last[i]) * split_stride * d);
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int i = 0; i < P; ++i)
                    {
                        const bool ok = k + j < n[i];
                        float4& w = v[j & 3][i];
                        w.x += ok ? t[j][i].x : 0.0f; w.y += ok ? t[j][i].y : 0.0f; w.z += ok ? t[j][i].z : 0.0f; w.w += ok ? t[j][i].w : 0.0f;
                    }
            }
#pragma unroll
            for (int i = 0; i < P; ++i) {
                float4 w = make_float4((v[0][i].x + v[1][i].x) + (v[2][i].x + v[3][i].x), (v[0][i].y + v[1][i].y) + (v[2][i].y + v[3][i].y),
                                       (v[0][i].z + v[1][i].z) + (v[2][i].z + v[3][i].z), (v[0][i].w + v[1][i].w) + (v[2][i].w + v[3][i].w));
                if (offsets) {
                    // (8-bit caches: a code's zero-point multiplies its weight row once, that of the low nibble)
                    const float z = zl[col[i] * FO_MAX_GROUPS + 4 * c4[i] / a.group], zo = a.w.nibbles ? 0.0f : z;
                    w.x += z; w.y += zo; w.z += z; w.w += zo;
                }
                if constexpr (!DENSE) {
                    const float4 f = *reinterpret_cast<const float4*>(unit + (4 * c4[i] & 31));
                    w.x *= f.x; w.y *= f.y; w.z *= f.z; w.w *= f.w;
                }
                *reinterpret_cast<float4*>(yl + col[i] * FO_STRIDE + 4 * c4[i]) = w;     // (behind the last piece it is written again)
            }
        }
    };
    if (pieces > 512) sum_pieces(std::integral_constant<int, 2>{});
    else sum_pieces(std::integral_constant<int, 1>{});
    __syncthreads();
    f32x16 acc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nb][i] = 0.0f;
#pragma unroll
    for (int sl = 0; sl < FO_MAX_SLABS; ++sl) {
        if (sl >= ns) break;
        const int ks = wave;
        uint32_t yp[3][4];
        {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int ch = DENSE ? ks * 16 + half * 8 + i : stream_channel(a.w.group, ks, half, a.tab.code_of_slot[ks & 3][i]);
                v[i] = yl[c32 * FO_STRIDE + sl * 128 + ch];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t h0, m0, l0, h1, m1, l1;
                split_bf16x3(v[2 * i], h0, m0, l0);
                split_bf16x3(v[2 * i + 1], h1, m1, l1);
                yp[0][i] = pack_hi16(h0, h1); yp[1][i] = pack_hi16(m0, m1); yp[2][i] = pack_hi16(l0, l1);
            }
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            uint4 wb = wf[sl & 1][nb];
            if constexpr (!DENSE) {                                  // fp16 -> bf16: at most 8 significant bits, exact
                const uint32_t w4[4] = {wb.x, wb.y, wb.z, wb.w};
                uint32_t d4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const xq_f16x2 hv = __builtin_bit_cast(xq_f16x2, w4[i]);
                    d4[i] = pack_hi16(__float_as_uint((float)hv.x), __float_as_uint((float)hv.y));
                }
                wb = make_uint4(d4[0], d4[1], d4[2], d4[3]);
            }
#pragma unroll
            for (int p = 2; p >= 0; --p)
                acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wb),
                                                                  __builtin_bit_cast(bf16x8, make_uint4(yp[p][0], yp[p][1], yp[p][2], yp[p][3])),
                                                                  acc[nb], 0, 0, 0);
        }
        if (sl + 2 < FO_MAX_SLABS) {
            load_weights(sl + 2, wf[sl & 1]);
            asm volatile("" ::: "memory");                           // (the compiler would move them behind the next slab's products)
        }
    }
    // the waves' sums, two column blocks at a time: [wave][block][register quad][lane] x 4
    const float f = DENSE ? 1.0f : ldexpf(1.0f, -shift);
    float4* red = reinterpret_cast<float4*>(lds);
    int b = 0, row = 0;
    const bool ok = cb * 32 + c32 < ncol;
    if (ok) row = row_of(cb * 32 + c32, b);
    float* dst = a.part + (((long long)chunk * s.nb + b) * s.R + row) * 128 + 4 * half;
#pragma unroll
    for (int rd = 0; rd < 2; ++rd) {
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x16& v = acc[2 * rd + n];
                red[((wave * 2 + n) * 4 + i4) * 64 + lane] = make_float4(v[4 * i4], v[4 * i4 + 1], v[4 * i4 + 2], v[4 * i4 + 3]);
            }
        __syncthreads();
        // wave w sums (block w / 4, register quad w % 4): columns 32 nb + 8 i4 + 4 half + [0, 4)
        float4 t = red[wave * 64 + lane];
#pragma unroll
        for (int w = 1; w < 8; ++w) {
            const float4 u = red[(w * 8 + wave) * 64 + lane];
            t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
        }
        if (ok) *reinterpret_cast<float4*>(dst + 32 * (2 * rd + (wave >> 2)) + 8 * (wave & 3)) = make_float4(t.x * f, t.y * f, t.z * f, t.w * f);
    }
}

// out = (sum over the channel splits) / (softmax denominator, summed over the token splits)
__global__ __launch_bounds__(256) void fold_finish_kernel(const float* __restrict__ part, const float* __restrict__ lsum, float* __restrict__ out,
                                                          FoldShape s, int chunks, int rt)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;                  // (sequence, row, four columns)
    if (idx >= s.nb * s.R * 32) return;
    const int c4 = idx & 31, row = (idx >> 5) % s.R, b = (idx >> 5) / s.R;
    int used;
    bool window;
    fold_used_splits(s, b, used, window);
    float L4[4] = {};
    for (int k = 0; k < used; k += 8) {                              // (eight loads at a time, the last split's again)
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = lsum[((long long)min(k + j, used - 1) * s.nb + b) * s.nrb * 16 * rt + row];
#pragma unroll
        for (int j = 0; j < 8; ++j) L4[j & 3] += k + j < used ? t[j] : 0.0f;
    }
    float L = (L4[0] + L4[1]) + (L4[2] + L4[3]);
    if (window) L += lsum[((long long)(s.splits - 1) * s.nb + b) * s.nrb * 16 * rt + row];
    float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 4
    for (int k = 0; k < chunks; ++k) {
        const float4 u = *reinterpret_cast<const float4*>(part + (((long long)k * s.nb + b) * s.R + row) * 128 + 4 * c4);
        t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    *reinterpret_cast<float4*>(out + ((long long)(s.b0 + b) * s.R + row) * 128 + 4 * c4) = make_float4(t.x / L, t.y / L, t.z / L, t.w / L);
}

// =====================================================================================================================
// Host side
// =====================================================================================================================
template <typename Args>
static hipError_t launch(void (*kernel)(const Args), int grid, int lds_bytes, const Args& a, hipStream_t s, int waves = 8)
{
    if (lds_bytes > 65536) {
        hipError_t e = allow_large_lds(reinterpret_cast<const void*>(kernel), lds_bytes);
        if (e != hipSuccess) return e;
    }
    kernel<<<dim3(grid), dim3(64 * waves), lds_bytes, s>>>(a);
    return hipGetLastError();
}

static size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// Workspace of one launch group of nb of the call's B sequences.  What shapes the sums (token splits, slabs per output
// workgroup, slab ways) follows from B, so that a sequence's result does not depend on the group it is launched in.
struct FoldPlan {
    int rt, nrb, tiles, splits, chunks, chunk_slabs, u_slab;
    int digits;                                            // queries in base-32 digits
    size_t p, mtile, rowfac, lsum, uy, yz, ud, total;      // bytes; u and y share a region (u is dead when y is written),
                                                           // the output splits lie over p (dead by then)
};

// Token splits of the value kernel: enough workgroups for the 256 CUs, two on each over coded rows (groups along the channels),
// but no more than leave a tile each.
int fold_splits(int nb, int nrb, int n_slabs_v, int max_len, int per_cu)
{
    const int per = nb * nrb * ((n_slabs_v + 1) / 2), nt = (max_len + FOLD_VTILE - 1) / FOLD_VTILE;
    return std::max(1, std::min({nt, (256 * per_cu + per - 1) / per, 16 * per_cu}));
}

static FoldPlan fold_plan(const FoldProblem& f, int B, int nb, int max_len, int splits)
{
    FoldPlan L{};
    const int R = f.Hq;
    L.rt = R <= 16 ? 1 : 2;
    const int rpb = 16 * L.rt;
    L.nrb = (R + rpb - 1) / rpb;
    L.tiles = (max_len + FOLD_VTILE - 1) / FOLD_VTILE * 2 + (f.block ? 2 : 0);
    L.digits = f.digits;
    L.splits = splits = splits + (f.block ? 1 : 0);
    L.u_slab = f.dense ? FOLD_U_DENSE(L.rt) : f.digits ? FOLD_UD_SLAB : FOLD_U_CODED(L.rt);
    const int colblocks = (B * (f.Hq / f.Hkv) + 31) / 32;
    L.chunk_slabs = std::max(1, std::min(FO_MAX_SLABS, f.n_slabs_v * f.Hkv * colblocks / 256));
    L.chunks = (f.n_slabs_v + L.chunk_slabs - 1) / L.chunk_slabs;
    L.p = align256(std::max((size_t)nb * L.nrb * L.tiles * 4 * (L.rt * 512) * 4, (size_t)L.chunks * nb * R * 512));
    L.mtile = align256(((size_t)nb * L.nrb * L.tiles * rpb * 4) << (f.block == 64));
    L.rowfac = align256((size_t)nb * L.nrb * rpb * 4);
    L.lsum = align256((size_t)splits * nb * L.nrb * rpb * 4);
    const size_t u_block = f.digits ? (size_t)fold_ud_block(f.n_slabs_k, f.n_slabs_k * (128 / f.group)) : (size_t)f.n_slabs_k * L.u_slab;
    L.uy = align256(std::max((size_t)nb * L.nrb * u_block, (size_t)splits * nb * R * f.n_slabs_v * 512));
    L.yz = f.dense || f.block ? 0 : align256((size_t)splits * nb * R * f.ng_v * 4);
    L.ud = f.block ? align256((size_t)nb * L.nrb * f.n_slabs_k * FOLD_U_DENSE(L.rt)) : 0;
    L.total = L.p + L.mtile + L.rowfac + L.lsum + L.uy + L.yz + L.ud;
    return L;
}

// Two workgroups a CU where their sums fit the partials of the rematerialising kernels, which a caller brings at the least, so that
// the query stays what it is and such a step never goes in groups.  (8 x 4096 tokens of 32 heads would ask for a tenth more than
// these: two splits there, a workgroup of four waves on every CU, 38 us where four splits take 34; with three the step is the same.
// Counts between the two took it to 0.89 to 1.11 times its time on 44 other shapes.)
static int fold_splits(const FoldProblem& f, int B, int nrb, int max_len)
{
    const int one = fold_splits(B, nrb, f.n_slabs_v, max_len, 1);
    if (f.dense || f.block) return one;
    const int two = fold_splits(B, nrb, f.n_slabs_v, max_len, 2);
    const size_t partials = (size_t)B * f.Hq * ((max_len + TILE_TOKENS - 1) / TILE_TOKENS) * (TILE_TOKENS / CHUNK_TOKENS) * (128 + 2) * sizeof(float);
    return fold_plan(f, B, B, max_len, two).total <= std::max(partials, fold_plan(f, B, B, max_len, one).total) ? two : one;
}

size_t fold_workspace_bytes(const FoldProblem& f, int B, int max_len)
{
    const int R = f.Hq, nrb = (R + (R <= 16 ? 15 : 31)) / (R <= 16 ? 16 : 32);
    return fold_plan(f, B, B, max_len, fold_splits(f, B, nrb, max_len)).total;
}

// Queries in base-32 digits for 2-bit codes with the scales along the channels and more than 16 query rows, where the tiles of 128 tokens fill
// rounds of 512 workgroups of 256 tokens no less than rounds of 512 of 128: a round takes 76 us over 32 slabs of groups of 128, one of the
// fp16 kernel 48 (1024 tiles 76 / 97, 1536 would be 152 / 144) - and where their buffers, larger by half, are no more than
// what a caller brings.
static int fold_digits(FoldProblem f, int B, int max_len)
{
    if (f.dense || f.nibbles || f.block || f.bits != 2 || f.Hq <= 16) return 0;
    const int nrb = (f.Hq + 31) / 32, n = B * nrb * ((max_len + FOLD_VTILE - 1) / FOLD_VTILE * 2);
    if (n < 1024 || 2 * ((n + 1023) / 1024) > (n + 511) / 512) return 0;
    f.digits = 1;
    return fold_workspace_bytes(f, B, max_len) <= f.query_bytes;
}

// The largest launch group that fits the workspace, for B sequences; where not even one does, one with fewer splits; false if
// that does not either.  `bytes` is cut to what the query asks for, so that results do not depend on how much more a caller
// brings; they depend on less only where splits are given up.
static bool fold_fit_plan(const FoldProblem& f, int B, int max_len, size_t bytes, bool fewer_splits, int* nb, FoldPlan* plan)
{
    const int R = f.Hq, nrb = (R + (R <= 16 ? 15 : 31)) / (R <= 16 ? 16 : 32);
    bytes = std::min(bytes, std::max(f.query_bytes, fold_workspace_bytes(f, B, max_len)));
    const int splits = fold_splits(f, B, nrb, max_len);
    for (int groups = 1;; ++groups) {
        const int n = (B + groups - 1) / groups;
        const FoldPlan p = fold_plan(f, B, n, max_len, splits);
        if (p.total <= bytes) { *nb = n; *plan = p; return true; }
        if (n == 1) break;
    }
    for (int sp = splits - 1; fewer_splits && sp >= 1; --sp) {
        const FoldPlan p = fold_plan(f, B, 1, max_len, sp);
        if (p.total <= bytes) { *nb = 1; *plan = p; return true; }
    }
    return false;
}
// (digits, whose buffers are larger, only where they fit)
static bool fold_fit(FoldProblem f, int B, int max_len, size_t bytes, int* nb, FoldPlan* plan)
{
    f.digits = fold_digits(f, B, max_len);
    if (f.digits && fold_fit_plan(f, B, max_len, bytes, false, nb, plan)) return true;
    f.digits = 0;
    return fold_fit_plan(f, B, max_len, bytes, true, nb, plan);
}

bool fold_fits(const FoldProblem& f, int B, int max_len, size_t bytes)
{
    int nb;
    FoldPlan p;
    return fold_fit(f, B, max_len, bytes, &nb, &p);
}

// Order of a launch's sequences.  Every XCD gets a contiguous eighth of the work items (xcd_contiguous), so with sequences of
// different lengths the XCD with the longest ones is the last to finish.  From two sequences per XCD on they are dealt out,
// longest first, each to the XCD with the fewest tokens that still has a place.  16 sequences of 4177 to 8191 tokens, us: value
// kernel 113 -> 103, scores 110.5 -> 109, whole step 237 -> 225.
static void fold_order(FoldShape& s)
{
    int by_len[XQ_MAX_BATCH], place[XQ_MAX_BATCH], n_of[8] = {}, first[9] = {};
    int shortest = s.len.v[s.b0], longest = shortest;
    for (int i = 1; i < s.nb; ++i) {
        shortest = std::min(shortest, s.len.v[s.b0 + i]);
        longest = std::max(longest, s.len.v[s.b0 + i]);
    }
    s.dealt = s.nb >= 16 && shortest < longest;
    if (!s.dealt) return;
    for (int i = 0; i < s.nb; ++i) by_len[i] = i;
    std::stable_sort(by_len, by_len + s.nb, [&](int a, int b) { return s.len.v[s.b0 + a] > s.len.v[s.b0 + b]; });
    for (int x = 0; x <= 8; ++x) first[x] = (x * s.nb + 7) / 8;           // (a sequence that two XCDs share counts for the first)
    long long load[8] = {};
    for (int i = 0; i < s.nb; ++i) {
        int best = -1;
        for (int x = 0; x < 8; ++x)
            if (n_of[x] < first[x + 1] - first[x] && (best < 0 || load[x] < load[best])) best = x;
        place[first[best] + n_of[best]++] = by_len[i];
        load[best] += s.len.v[s.b0 + by_len[i]];
    }
    for (int i = 0; i < s.nb; ++i) s.order[i] = (uint8_t)place[i];
}

template <int BITS, int G, int RT>
static hipError_t run_scores(const FoldScoreArgs& a, bool nibbles, int grid, hipStream_t s)
{
    if constexpr (BITS == 4 && G == 128) {
        if (nibbles) return launch(fold_scores_kernel<4, 128, RT, true>, grid, FOLD_SCORE_LDS<4, 128, RT, true> / 8 * a.waves, a, s, a.waves);
    }
    return launch(fold_scores_kernel<BITS, G, RT, false>, grid, FOLD_SCORE_LDS<BITS, G, RT, false> / 8 * a.waves, a, s, a.waves);
}
template <int BITS, int G, int RT>
static hipError_t run_values(const FoldValueArgs& a, bool nibbles, int grid, hipStream_t s)
{
    if constexpr (BITS == 4 && G == 128) {
        if (nibbles) return launch(fold_values_kernel<4, 128, RT, true>, grid, FoldValueLds<RT, 2, true, false>::TOTAL, a, s, FOLD_VALUE_WAVES);
    }
    return launch(fold_values_kernel<BITS, G, RT, false>, grid, FoldValueLds<RT, 2 * (128 / G), false, fold_scaled_codes(BITS)>::TOTAL, a, s, FOLD_VALUE_WAVES);
}
template <int RT>
static hipError_t scores_for(int bits, int G, bool nibbles, const FoldScoreArgs& a, int grid, hipStream_t s)
{
    switch (bits * 1000 + G) {
        case 2064: return run_scores<2, 64, RT>(a, nibbles, grid, s);
        case 2128: return run_scores<2, 128, RT>(a, nibbles, grid, s);
        case 3064: return run_scores<3, 64, RT>(a, nibbles, grid, s);
        case 3128: return run_scores<3, 128, RT>(a, nibbles, grid, s);
        case 4064: return run_scores<4, 64, RT>(a, nibbles, grid, s);
        case 4128: return run_scores<4, 128, RT>(a, nibbles, grid, s);
    }
    if constexpr (RT == 2)
        if (a.row_split) return launch(fold_scores_dense_kernel<1, 2>, grid, FOLD_SCORE_RED<1> / 8 * a.waves, a, s, a.waves);
    return launch(fold_scores_dense_kernel<RT>, grid, FOLD_SCORE_RED<RT> / 8 * a.waves, a, s, a.waves);
}
template <int RT>
static hipError_t values_for(int bits, int G, bool nibbles, const FoldValueArgs& a, int grid, hipStream_t s)
{
    switch (bits * 1000 + G) {
        case 2064: return run_values<2, 64, RT>(a, nibbles, grid, s);
        case 2128: return run_values<2, 128, RT>(a, nibbles, grid, s);
        case 3064: return run_values<3, 64, RT>(a, nibbles, grid, s);
        case 3128: return run_values<3, 128, RT>(a, nibbles, grid, s);
        case 4064: return run_values<4, 64, RT>(a, nibbles, grid, s);
        case 4128: return run_values<4, 128, RT>(a, nibbles, grid, s);
    }
    return launch(fold_values_dense_kernel<RT>, grid, FoldValueDenseLds<RT>::TOTAL, a, s);
}

template <int BITS, int RT>
static hipError_t scores_pc(const FoldScoreArgs& a, int grid, hipStream_t s)
{
    return a.s.block == 64 ? launch(fold_scores_pc_kernel<BITS, 2, RT>, grid, FOLD_SCORE_PC_LDS<BITS, RT>, a, s)
                           : launch(fold_scores_pc_kernel<BITS, 1, RT>, grid, FOLD_SCORE_PC_LDS<BITS, RT>, a, s);
}
template <int RT>
static hipError_t scores_pc_for(int bits, const FoldScoreArgs& a, int grid, hipStream_t s)
{
    return bits == 2 ? scores_pc<2, RT>(a, grid, s) : bits == 3 ? scores_pc<3, RT>(a, grid, s) : scores_pc<4, RT>(a, grid, s);
}
template <int RT>
static hipError_t values_pc_for(int bits, const FoldValueArgs& a, int grid, hipStream_t s)
{
    typedef FoldValuePcLds<RT> L;
    return bits == 2 ? launch(fold_values_pc_kernel<2, RT>, grid, L::TOTAL, a, s)
         : bits == 3 ? launch(fold_values_pc_kernel<3, RT>, grid, L::TOTAL, a, s) : launch(fold_values_pc_kernel<4, RT>, grid, L::TOTAL, a, s);
}

hipError_t run_folded_attn(const FoldProblem& f, const uint16_t* q, const FoldSource& kx, const FoldSource& vx, const FoldWeights& kw,
                           const FoldWeights& vw, int B, const BatchI32& len, int max_len, float softmax_scale, float* out, void* ws,
                           size_t ws_bytes, hipStream_t s, const FoldSource* window)
{
    int nb;
    FoldPlan L;
    if (!fold_fit(f, B, max_len, ws_bytes, &nb, &L)) return hipErrorInvalidValue;
    const int bits = f.dense ? 16 : f.bits;
    UnpackTable tab{};
    if (!f.dense && !unpack_table_for(bits, &tab)) return hipErrorInvalidValue;
    uint8_t* w = static_cast<uint8_t*>(ws);
    float* p = reinterpret_cast<float*>(w); w += L.p;
    float* mtile = reinterpret_cast<float*>(w); w += L.mtile;
    float* rowfac = reinterpret_cast<float*>(w); w += L.rowfac;
    float* lsum = reinterpret_cast<float*>(w); w += L.lsum;
    uint8_t* u = w;
    float* y = reinterpret_cast<float*>(w); w += L.uy;
    float* yz = reinterpret_cast<float*>(w); w += L.yz;
    uint8_t* u_dense = f.block ? w : nullptr;
    float* part = p;
    bool any_window = false;
    for (int b = 0; b < B; ++b) any_window |= f.block && len.v[b] % f.block;
    const int gq = f.Hq / f.Hkv;
    for (int b0 = 0; b0 < B; b0 += nb) {
        FoldShape sh{};
        sh.b0 = b0; sh.nb = std::min(nb, B - b0); sh.Hq = f.Hq; sh.Hkv = f.Hkv; sh.R = f.Hq; sh.nrb = L.nrb;
        sh.tiles = L.tiles; sh.splits = L.splits; sh.len = len;
        sh.block = f.block; sh.mhalf = f.block == 64;
        fold_order(sh);
        const int coded_splits = L.splits - (f.block ? 1 : 0);
        const int colblocks = (sh.nb * gq + 31) / 32;
        {
            FoldQueryArgs a{kw, sh, q, u, rowfac, softmax_scale * 1.44269504088896340736f, L.u_slab, f.n_slabs_k, L.rt, tab, u_dense};
            const dim3 grid((f.n_slabs_k + 1) / 2, f.Hkv, colblocks);
            if (f.dense) fold_query_kernel<true, 128><<<grid, dim3(128), 0, s>>>(a);
            else if (L.digits && f.group == 64) fold_query_kernel<false, 64, true><<<grid, dim3(128), 0, s>>>(a);
            else if (L.digits) fold_query_kernel<false, 128, true><<<grid, dim3(128), 0, s>>>(a);
            else if (f.group == 64) fold_query_kernel<false, 64><<<grid, dim3(128), 0, s>>>(a);
            else fold_query_kernel<false, 128><<<grid, dim3(128), 0, s>>>(a);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        {
            // A workgroup is one token tile with eight slab ways, or with four where that still gives most CUs two workgroups
            // (registers allow two waves per SIMD, so two of four waves fit): one's set-up, last loads and meeting of the slab
            // ways then run beside the other's products, and fewer ways meet.  Whole steps, eight waves / four: 1024 tiles of 2
            // bits 233 / 215 us (group 128), 273 / 263 (group 64), latent 136 / 127, 16 heads of 4 bits 124 / 111; 512 tiles of
            // 3 bits 143 / 138; 384 tiles 166 / 161; 256 tiles 94.4 / 94.1.
            // Over bf16 rows of 17 query heads and more four waves only where their rounds of 512 workgroups are no emptier than those
            // of 256 of eight waves: eight / four, d = 4096: 512 tiles 245 / 238, 1024 tiles 443 / 426, but 768 tiles 372 / 390; with 16
            // heads 768 tiles of d = 2048 202 / 202, 520 tiles 148 / 140, and with 2 slabs, on which eight waves idle, 640 tiles 63 / 59.
            const int n = B * sh.nrb * sh.tiles;
            const bool four = !f.block && n >= 3 * 128 && (!f.dense || L.rt == 1 || f.n_slabs_k <= 4 || 2 * ((n + 511) / 512) <= (n + 255) / 256);
            const int waves = four ? 4 : 8;
            // Over bf16 rows a tile's two row tiles go to workgroups of their own where half of the CUs or more would be left without one: half
            // of the products and queries each, and the rows come out of L2 for the second (neighbours on one XCD).  The sums are the same.
            // This kernel, both row tiles / one: 128 tiles of d = 4096 36.1 / 29.2 us, 126 35.9 / 28.2, 63 (half of a round) 32.8 / 24.0,
            // 16 31.4 / 21.7, 64 of d = 1024 23.4 / 19.2.  From 129 tiles on the second ones would wait for a second round.
            const int row_split = f.dense && !f.block && L.rt == 2 && n <= 128;
            FoldScoreArgs a{kx, sh, u, rowfac, p, mtile, L.u_slab, waves, row_split, FoldSource{}, u_dense, 0};
            if (any_window) { a.window = *window; a.n_window = xcd_grid(sh.nb * sh.nrb); }
            const int grid = a.n_window + xcd_grid(sh.nb * sh.nrb * sh.tiles * (row_split ? 2 : 1) / (L.digits ? 2 : 1));
            e = L.digits ? (f.group == 64 ? launch(fold_scores_digits_kernel<64>, grid, FoldDigitLds::TOTAL, a, s, 4)
                                          : launch(fold_scores_digits_kernel<128>, grid, FoldDigitLds::TOTAL, a, s, 4))
              : f.block ? (L.rt == 1 ? scores_pc_for<1>(bits, a, grid, s) : scores_pc_for<2>(bits, a, grid, s))
                        : (L.rt == 1 ? scores_for<1>(bits, f.group, f.nibbles, a, grid, s) : scores_for<2>(bits, f.group, f.nibbles, a, grid, s));
            if (e != hipSuccess) return e;
        }
        {
            FoldValueArgs a{vx, sh, p, mtile, y, yz, lsum, (f.n_slabs_v + 1) / 2, FoldSource{}, 0};
            if (any_window) { a.window = *window; a.n_window = xcd_grid(sh.nb * sh.nrb * a.cblocks); }
            const int grid = a.n_window + xcd_grid(sh.nb * sh.nrb * coded_splits * a.cblocks);
            e = f.block ? (L.rt == 1 ? values_pc_for<1>(bits, a, grid, s) : values_pc_for<2>(bits, a, grid, s))
                        : (L.rt == 1 ? values_for<1>(bits, f.group, f.nibbles, a, grid, s) : values_for<2>(bits, f.group, f.nibbles, a, grid, s));
            if (e != hipSuccess) return e;
        }
        {
            FoldOutArgs a{vw, sh, y, yz, part, f.n_slabs_v, f.block ? 0 : f.ng_v, f.group, L.chunk_slabs, tab};
            const dim3 grid(L.chunks, f.Hkv, colblocks);
            if (f.dense) {
                e = allow_large_lds(reinterpret_cast<const void*>(fold_output_kernel<true>), FO_LDS);
                if (e != hipSuccess) return e;
                fold_output_kernel<true><<<grid, dim3(512), FO_LDS, s>>>(a);
            } else {
                e = allow_large_lds(reinterpret_cast<const void*>(fold_output_kernel<false>), FO_LDS);
                if (e != hipSuccess) return e;
                fold_output_kernel<false><<<grid, dim3(512), FO_LDS, s>>>(a);
            }
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        fold_finish_kernel<<<dim3((sh.nb * sh.R * 32 + 255) / 256), dim3(256), 0, s>>>(part, lsum, out, sh, L.chunks, L.rt);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace xq
