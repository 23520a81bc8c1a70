// Folded queries and scores over caches of 2 bits with the queries in base-32 digits; part of folded_attn.hip, inside its namespace.
//
// The f8f6f4 products of the matrix cores take 64 channels in the time that the fp16 form takes 16, and a 2-bit code under two zeros is
// already an operand of theirs, the fp4 number code / 2.  So unpacking is masks (6 instructions for 32 codes, where the fp16 form takes
// some 50), and the precision is a matter of u: 32 channels of a query row share a power of two (the operand's block scale) and every u is
// five digits of -16 .. 16, each an fp6 (e2m3) number, digit p worth 32^-p: a multiple of 2^-24 of the power of two above the block's
// largest.  All products and their sums within an instruction are exact; instructions accumulate in fp32, largest digits first.
//
// Integer zero-points (see folded_common.hpp): the sum over 64 channels of digit sums times -zi is what the accumulator starts
// from, by one fp16 product.  That start is exact: the channel sum is cut to a multiple of 2^-16 of that power of two (some 23 bits, in two fp16
// parts; zi has two), so what the first digits leave of it is exact too and only the small rest is ever rounded.  What was cut off goes through
// the rests' product, times zi s.
//
// What five digits cut from a channel's u counts as much as from the block's largest, which is no loss where the channels' u are of
// one size, some of them small by chance.  Where they are not - weight rows that differ by more than FOLD_WIDE_ROWS, or a u below
// 2^-FOLD_WIDE_U of the largest (32 normal numbers have one in 20000 blocks) - the block has eight digits, 2^-39, of which the last
// three are added by a loop of their own.
#pragma once

constexpr int FOLD_DIGITS = 5, FOLD_DIGITS_MORE = 3, FOLD_WIDE_U = 20;
// bytes of folded queries: of a slab, [half slab 2][digits as 16-byte pieces, as 8-byte pieces, (start, block scale)][lane 64], then
// the same of the further digits; behind all slabs of a row block the groups' channel sums, [16 groups][part 5][lane 64][16 B]
constexpr int FOLD_UD_HALF = 64 * 128, FOLD_UD_MORE = 64 * 24 * FOLD_DIGITS_MORE, FOLD_UD_SLAB = 2 * (FOLD_UD_HALF + FOLD_UD_MORE);
constexpr int FOLD_UD_SUMS = 5 * 1024;
__host__ __device__ constexpr long long fold_ud_block(int n_slabs, int ng) { return (long long)n_slabs * FOLD_UD_SLAB + (ng + 15) / 16 * FOLD_UD_SUMS; }

// code (of the 32 that a lane holds in two dwords) in operand slot i: a dword's even codes, then its odd ones
__host__ __device__ constexpr int fold_slot_code(int i) { return (i >> 4) * 16 + 2 * (i & 7) + ((i >> 3) & 1); }
// first channel of the 32 that lane half `q` holds in half slab h: in groups of 128 a lane takes 16 adjacent bytes of a row
template <int G>
__host__ __device__ constexpr int fold_block_channel(int h, int q) { return G == 128 ? 64 * q + 32 * h : 64 * h + 32 * q; }

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x6 __attribute__((ext_vector_type(6)));

// The folded queries of a wave's slab, from LDS (FQ_STRIDE floats per query column, natural channel order): a lane takes 32
// channels of a column at a time.
template <int G>
__device__ __forceinline__ void fold_store_digits(const FoldQueryArgs& a, const float* mine, const int* place, int lane, int slab, bool wide_rows)
{
    constexpr int GPS = 128 / G;
    const int ng = a.n_slabs * GPS;
#pragma unroll 1
    for (int it = 0; it < 2; ++it) {
        const int idx = it * 64 + lane, q = idx & 1, h = (idx >> 1) & 1, col = idx >> 2;
        const int at = place[col], rr = at & 31;
        if (__all(at < 0)) continue;
        float r[32];
        const float* src = mine + col * FQ_STRIDE + fold_block_channel<G>(h, q);
        uint32_t top = 0u, low_u = 0xFFFFFFFFu;                      // largest, smallest nonzero number less 1
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float4 v = *reinterpret_cast<const float4*>(src + 4 * k);
            r[4 * k] = v.x; r[4 * k + 1] = v.y; r[4 * k + 2] = v.z; r[4 * k + 3] = v.w;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t m = __float_as_uint(r[4 * k + i]) & 0x7FFFFFFFu;
                top = max(top, m);
                low_u = min(low_u, m - 1u);
            }
        }
        const bool wide = wide_rows || low_u + (FOLD_WIDE_U << 23) < top;
        // block below 2^(be - 126); digits of u 2^(4 - (be - 126))
        const int be = max((int)(top >> 23), 3);
        const float up = __uint_as_float((uint32_t)(257 - be) << 23);
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < 32; ++i) { sum += (double)r[i]; r[i] *= up; }
        uint8_t* blk = a.u + (long long)(at >> 5) * fold_ud_block(a.n_slabs, ng);
        uint8_t* dst = blk + (long long)slab * FOLD_UD_SLAB + h * FOLD_UD_HALF;
        const int pl = q * 32 + rr;                                   // the lane of the products
        auto digits = [&](uint8_t* to, int p, int n) XQ_INLINE_LAMBDA {
            f32x16 e, o;
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const float d = rintf(r[i]);
                r[i] = (r[i] - d) * 32.0f;
#pragma unroll
                for (int k = 0; k < 16; ++k) {                         // (the conversion takes even and odd slots from two registers)
                    if (fold_slot_code(2 * k) == i) e[k] = d;
                    if (fold_slot_code(2 * k + 1) == i) o[k] = d;
                }
            }
            const u32x6 v = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(e, o, 8.0f);
            if (at >= 0) {
                *reinterpret_cast<uint4*>(to + (p * 64 + pl) * 16) = make_uint4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<uint2*>(to + n * 1024 + (p * 64 + pl) * 8) = make_uint2(v[4], v[5]);
            }
        };
#pragma unroll 1
        for (int p = 0; p < FOLD_DIGITS; ++p) digits(dst, p, FOLD_DIGITS);
        int low = be - 126 - 4 - 5 * FOLD_DIGITS;                     // exponent of what is left of a digit
        if (wide) {
            uint8_t* more = blk + (long long)slab * FOLD_UD_SLAB + 2 * FOLD_UD_HALF + h * FOLD_UD_MORE;
#pragma unroll 1
            for (int p = 0; p < FOLD_DIGITS_MORE; ++p) digits(more, p, FOLD_DIGITS_MORE);
            low -= 5 * FOLD_DIGITS_MORE;
        }
        // channel sums of the numbers that the codes will meet
        double left = 0.0;
#pragma unroll
        for (int i = 0; i < 32; ++i) left += (double)r[i];
        sum -= ldexp(left, low);
        sum += __shfl_xor(sum, 1);                                    // of the half slab
        const int grid = max(max(be, __shfl_xor(be, 1)) - 126 - 16, -16);
        const double first = ldexp(rint(ldexp(sum, -grid)), grid);
        const float f8 = (float)(first * (1.0 / 256.0));
        const _Float16 s0 = (_Float16)f8, s1 = (_Float16)(f8 - (float)s0);
        double rest = sum - first;
        if (at >= 0) {
            const xq_f16x2 st = {s0, s1};
            const uint32_t scale = (top >> 23) == 255u ? 255u : (uint32_t)(be + 1);
            *reinterpret_cast<uint2*>(dst + FOLD_DIGITS * 1536 + pl * 8) =
                make_uint2(q == 0 ? __builtin_bit_cast(uint32_t, st) : 0u, scale | (wide ? 256u : 0u));
        }
        if constexpr (GPS == 1) {
            sum += __shfl_xor(sum, 2);
            rest += __shfl_xor(rest, 2);
        }
        auto sums = [&](int g, float s, float t) XQ_INLINE_LAMBDA {
            uint16_t* to = reinterpret_cast<uint16_t*>(blk + (long long)a.n_slabs * FOLD_UD_SLAB + (g >> 4) * FOLD_UD_SUMS + ((g >> 3 & 1) * 32 + rr) * 16) + (g & 7);
            uint32_t p[3], t3[3];
            split_bf16x3(s, p[0], p[1], p[2]);
            split_bf16x3(-t, t3[0], t3[1], t3[2]);
            to[0] = p[0] >> 16; to[512] = p[1] >> 16; to[1024] = p[2] >> 16; to[1536] = t3[0] >> 16; to[2048] = t3[1] >> 16;
        };
        if (at >= 0 && q == 0 && (GPS == 2 || h == 0)) sums(slab * GPS + (GPS == 2 ? h : 0), (float)sum, (float)rest);
        if (at >= 0 && (idx & 3) == 0 && slab == a.n_slabs - 1)
            for (int g = ng; g & 15; ++g) sums(g, 0.0f, 0.0f);
    }
}

// =====================================================================================================================
// Scores.  A workgroup owns 256 tokens of a sequence and one block of 32 query rows; each of its four waves has 64 tokens and walks all
// slabs.  The digits of a slab come through LDS, once for the workgroup, in two buffers; a lane has its token's codes in
// registers, as they come from memory, and the tokens' records (scale, -zi) of a run of groups are in LDS.  Half a slab against 32
// tokens is a chain of six products, the start and five digits, and a slab is four chains.  Behind each product stand the vector instructions that unpack
// the next chain's codes and add the chain before to the scores, and, where a digit has been used, the LDS read that replaces it
// by the next half slab's.
// A chain takes 204 cycles of a SIMD alone, 222 with what stands behind its products, and 290 with the loads; a third of a workgroup's time are its
// first loads, the records and the end.  Measured (us, one layer after the other, the fp16 form / this): 4 x 32768 tokens, d = 4096, 32 heads
// 97 / 76; 16 x up to 8191 in groups of 64 103 / 76, 40 heads 193 / 146; 16 x 8192 of d = 1024 43 / 32; 2 x 65536 of d = 1024, 20 heads 40 / 30.
// Tiles of 128 tokens with four slab ways, on which a half slab's digits serve two waves, took as long as the fp16 form (256 tiles
// of 3 bits 35 / 33, 1024 of 2 bits 96 / 102), and longer at 4 bits, whose operands (fp6) take 20 instructions for 32 codes (512 tiles 71 / 85).
// =====================================================================================================================
struct FoldDigitLds {
    static constexpr int SLAB = 2 * FOLD_UD_HALF, TOKENS = 256, GROUPS = 48;       // records of so many groups at a time (two workgroups a CU)
    static constexpr int RECORDS = 2 * SLAB, TOTAL = RECORDS + GROUPS * TOKENS * 4;
};

template <int G>
__global__ __launch_bounds__(256, 2) void fold_scores_digits_kernel(const FoldScoreArgs a)
{
    typedef FoldDigitLds L;
    constexpr int GPS = 128 / G, ROWB = 32, NT = 2;
    constexpr int DIG8 = FOLD_DIGITS * 1024, START = FOLD_DIGITS * 1536;         // in a half slab: 8-byte pieces; starts and scales
    constexpr int TOP = 127;                                         // digit p counts 2^(E - 4 - 5 p) 8 times its operand, a code twice its own
    constexpr int SCALE03 = TOP | (TOP - 5) << 8 | (TOP - 10) << 16 | (TOP - 15) << 24, SCALE4 = TOP - 20;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FoldShape& s = a.s;
    const FoldSource& x = a.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wtiles = s.tiles / 2, item = xcd_contiguous(s.nb * s.nrb * wtiles, blockIdx.x);
    if (item >= s.nb * s.nrb * wtiles) return;
    const int wt = item % wtiles, rb = (item / wtiles) % s.nrb, b = fold_sequence(s, item / (wtiles * s.nrb)), len = s.len.v[s.b0 + b];
    if (wt * L::TOKENS >= len) return;
    const int c32 = lane & 31, half = lane >> 5, n_slabs = x.n_slabs;
    const uint8_t* cbase = x.codes + (long long)(s.b0 + b) * x.cap * x.row_bytes;
    const uint16_t* sbase = x.scale + (long long)(s.b0 + b) * x.cap * x.ng_row;
    const uint16_t* zbase = x.zero + (long long)(s.b0 + b) * x.cap * x.ng_row;
    const uint8_t* ubase = a.u + ((long long)b * s.nrb + rb) * fold_ud_block(n_slabs, x.ng);
    const int tok0 = wt * L::TOKENS + wave * 64 + c32;                // the lane's first token; the other is 32 on
    int row[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) row[tt] = min(tok0 + 32 * tt, len - 1);
    const uint32_t flag = rb * 32 + c32 < s.R ? 256u : 0u;           // (what lies in the places of rows that are not there is not looked at)
    uint32_t* records = reinterpret_cast<uint32_t*>(lds + L::RECORDS) + wave * 64 + c32;             // [group][token]: -256 zi (fp16) | scale (bf16)

    // ---- loads: digits of a slab (16-byte piece tid of 256, four times), codes
    int slab0 = 0, last_slab = 0;                                    // of the run of groups whose records are in LDS
    u32x4 st[4];                                                     // digits on their way to LDS
    auto load_digits = [&](int slab) XQ_INLINE_LAMBDA {
        const uint8_t* src = ubase + (long long)min(slab, last_slab) * FOLD_UD_SLAB + tid * 16;
#pragma unroll
        for (int k = 0; k < 4; ++k) st[k] = *reinterpret_cast<const u32x4*>(src + k * 4096);
    };
    auto write_digits = [&](int buf) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<u32x4*>(lds + buf + tid * 16 + k * 4096) = st[k];
    };
    uint32_t voff[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) voff[tt] = (uint32_t)row[tt] * (uint32_t)x.row_bytes + half * 16u;
    u32x4 cw[2][NT];                                                 // codes of this slab and the next
    auto load_codes = [&](int slab, auto N) XQ_INLINE_LAMBDA {
        const uint8_t* src = cbase + (long long)min(slab, last_slab) * ROWB;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) cw[decltype(N)::value][tt] = *reinterpret_cast<const u32x4*>(src + voff[tt]);
    };

    // Scores, and (T) what has been added to them since the last FLUSH slabs: rounded at their full size once per half slab the result was off
    // by 9.5e-7 (16 sequences of up to 8191 tokens, groups of 64), 5.9e-7 so, against 6.0e-7 on the fp16 form; 5.4e-7 against 5.4e-7 over eight
    // slabs, where 8 instead of 4 gave 6.3e-7
    constexpr int FLUSH = 4;
    float S[NT][16], T[NT][16];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int i = 0; i < 16; ++i) S[tt][i] = 0.0f;
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;

    // ---- records, and what the rests of the zero-points add, 16 groups of 32 tokens at a time: lane = (token, 8 groups).  The next scales and
    // zero-points are asked for while the ones before are worked on.
    const bool wide_meta = ((reinterpret_cast<uintptr_t>(sbase) | reinterpret_cast<uintptr_t>(zbase) | (uint32_t)x.ng_row * 2u) & 15u) == 0;
    uint4 sv, zv;
    auto load_item = [&](int gbeg, int c, bool second) XQ_INLINE_LAMBDA {
        const int g8 = gbeg + c * 16 + 8 * half, r0 = row[0], r1 = row[1];
        const long long at = (long long)(second ? r1 : r0) * x.ng_row + g8;
        if (wide_meta && g8 + 8 <= x.ng) {
            sv = *reinterpret_cast<const uint4*>(sbase + at);
            zv = *reinterpret_cast<const uint4*>(zbase + at);
        } else {
            uint32_t se[8], ze[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                se[k] = g8 + k < x.ng ? sbase[at + k] : 0u;
                ze[k] = g8 + k < x.ng ? zbase[at + k] : 0u;
            }
            sv = make_uint4(se[0] | se[1] << 16, se[2] | se[3] << 16, se[4] | se[5] << 16, se[6] | se[7] << 16);
            zv = make_uint4(ze[0] | ze[1] << 16, ze[2] | ze[3] << 16, ze[4] | ze[5] << 16, ze[6] | ze[7] << 16);
        }
    };
    auto make_records = [&](int gbeg) XQ_INLINE_LAMBDA {
        const int nc = (min(L::GROUPS, x.ng - gbeg) + 15) / 16;
        static_for<0, NT>([&](auto TT) XQ_INLINE_LAMBDA {
        constexpr int tt = decltype(TT)::value;
        f32x16 t = zero16, v = zero16;                               // small products apart from the large ones
#pragma unroll 1
        for (int c = 0; c < nc; ++c) {
            const uint32_t s4[4] = {sv.x, sv.y, sv.z, sv.w}, z4[4] = {zv.x, zv.y, zv.z, zv.w};
            const uint4* us = reinterpret_cast<const uint4*>(ubase + (long long)n_slabs * FOLD_UD_SLAB + ((gbeg >> 4) + c) * FOLD_UD_SUMS + lane * 16);
            const bf16x8 A0 = __builtin_bit_cast(bf16x8, us[0]), A1 = __builtin_bit_cast(bf16x8, us[64]), A2 = __builtin_bit_cast(bf16x8, us[128]),
                         A3 = __builtin_bit_cast(bf16x8, us[192]), A4 = __builtin_bit_cast(bf16x8, us[256]);
            if (c + 1 < nc) load_item(gbeg, c + 1, tt == 1);
            else if (tt == 0) load_item(gbeg, 0, true);
            uint32_t R[4][4];                                        // parts of the rests, and zi s
            uint32_t* rec = records + (c * 16 + 8 * half) * L::TOKENS + 32 * tt;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t p[2][3];
                float e[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float sc = j ? bf16_hi_to_f32(s4[k]) : bf16_lo_to_f32(s4[k]);
                    float rest;
                    const float zi = fold_integer_zero(sc, j ? bf16_hi_to_f32(z4[k]) : bf16_lo_to_f32(z4[k]), 3.0f, rest);
                    split_bf16x3(rest, p[j][0], p[j][1], p[j][2]);
                    e[j] = zi * sc;
                    rec[(2 * k + j) * L::TOKENS] = f16_bits(-256.0f * zi) | (__float_as_uint(sc) & 0xFFFF0000u);
                }
#pragma unroll
                for (int n = 0; n < 3; ++n) R[n][k] = pack_hi16(p[0][n], p[1][n]);
                R[3][k] = pack_bf16x2_rne(e[0], e[1]);
            }
            auto B = [&](int n) XQ_INLINE_LAMBDA { return __builtin_bit_cast(bf16x8, make_uint4(R[n][0], R[n][1], R[n][2], R[n][3])); };
            v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A0, B(0), v, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A4, B(3), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A2, B(1), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, B(2), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A3, B(3), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A0, B(2), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A2, B(0), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, B(1), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A0, B(1), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, B(0), t, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) S[tt][k] += t[k] + v[k];
        });
    };

    // ---- operands of chain X of a slab: half slab X / 2, tokens X % 2
    uint32_t rec[2][NT][GPS];                                        // records of this slab and the next
    uint32_t F[2][4];                                                // codes of this chain and the next as operands
    f32x16 P[2];
    u32x4 ua[FOLD_DIGITS];
    u32x2 ub[FOLD_DIGITS], us[2];                                    // digits; starts and scales of this half slab and the next
    auto read_records = [&](int slab, auto N) XQ_INLINE_LAMBDA {
        constexpr int n = decltype(N)::value;
        const int g = (min(slab, last_slab) - slab0) * GPS;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int i = 0; i < GPS; ++i) rec[n][tt][i] = records[(g + i) * L::TOKENS + 32 * tt];
    };
    auto exchange = [&](auto N) XQ_INLINE_LAMBDA {                    // groups of 64: lane halves swap, for each group's first and second 32 channels
        constexpr int n = decltype(N)::value;
        if constexpr (G == 64)
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                u32x4& w = cw[n][tt];
                const auto e = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false), f = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                w = u32x4{e[0], f[0], e[1], f[1]};
            }
    };
    auto unpack = [&](auto N, auto X) XQ_INLINE_LAMBDA {
        constexpr int n = decltype(N)::value, h = decltype(X)::value / 2, tt = decltype(X)::value % 2;
        const uint32_t w0 = cw[n][tt][2 * h], w1 = cw[n][tt][2 * h + 1];
        uint32_t (&f)[4] = F[decltype(X)::value & 1];
        f[0] = w0 & 0x33333333u; f[1] = (w0 >> 2) & 0x33333333u;
        f[2] = w1 & 0x33333333u; f[3] = (w1 >> 2) & 0x33333333u;
    };
    auto digit = [&](int p) XQ_INLINE_LAMBDA {
        return i32x8{(int)ua[p][0], (int)ua[p][1], (int)ua[p][2], (int)ua[p][3], (int)ub[p][0], (int)ub[p][1], 0, 0};
    };
    auto codes = [&](const uint32_t (&f)[4]) XQ_INLINE_LAMBDA { return i32x8{(int)f[0], (int)f[1], (int)f[2], (int)f[3], 0, 0, 0, 0}; };
    auto read_digit = [&](int buf, int h, int p) XQ_INLINE_LAMBDA {
        const uint8_t* src = lds + buf + h * FOLD_UD_HALF;
        ua[p] = *reinterpret_cast<const u32x4*>(src + p * 1024 + lane * 16);
        ub[p] = *reinterpret_cast<const u32x2*>(src + DIG8 + p * 512 + lane * 8);
    };
    auto read_start = [&](int buf, int h) XQ_INLINE_LAMBDA { us[h] = *reinterpret_cast<const u32x2*>(lds + buf + h * FOLD_UD_HALF + START + lane * 8); };
    // a quarter of the multiply-adds of chain X (its slab's records have index N; slabs behind the last one add nothing)
    auto add_piece = [&](auto X, auto N, auto K, bool live) XQ_INLINE_LAMBDA {
        constexpr int c = decltype(X)::value, n = decltype(N)::value, k = decltype(K)::value, h = c / 2, tt = c % 2;
        const float sc = __uint_as_float(live ? rec[n][tt][GPS == 2 ? h : 0] & 0xFFFF0000u : 0u);
#pragma unroll
        for (int i = 4 * k; i < 4 * (k + 1); ++i) T[tt][i] = __builtin_fmaf(P[c & 1][i], sc, T[tt][i]);
    };

    auto flush = [&]() XQ_INLINE_LAMBDA {
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                S[tt][i] += T[tt][i];
                T[tt][i] = 0.0f;
            }
    };

    for (; slab0 < n_slabs; slab0 += L::GROUPS / GPS) {
        last_slab = min(n_slabs, slab0 + L::GROUPS / GPS) - 1;
        load_item(slab0 * GPS, 0, false);
        load_digits(slab0);
        load_codes(slab0, std::integral_constant<int, 0>{});
        load_codes(slab0 + 1, std::integral_constant<int, 1>{});
        if (slab0) __syncthreads();                                  // (buffers and records are read to the end)
        make_records(slab0 * GPS);
        write_digits(0);
        load_digits(slab0 + 1);
        write_digits(L::SLAB);
        load_digits(slab0 + 2);
        __syncthreads();
        read_start(0, 0);
#pragma unroll
        for (int p = 0; p < FOLD_DIGITS; ++p) read_digit(0, 0, p);
        read_records(slab0, std::integral_constant<int, 0>{});
        exchange(std::integral_constant<int, 0>{});
        unpack(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                for (int i = 0; i < 16; ++i) T[tt][i] = 0.0f;
        P[1] = zero16;                                               // (the chain before the first adds nothing)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int i = 0; i < GPS; ++i) rec[1][tt][i] = 0u;
        unsigned long long more = 0;                                 // slabs with further digits
        for (int j0 = slab0; j0 <= last_slab; j0 += 2) {             // (a slab behind the last one adds nothing)
            static_for<0, 2>([&](auto J) XQ_INLINE_LAMBDA {
                constexpr int jj = decltype(J)::value;
                constexpr std::integral_constant<int, jj> N{};
                constexpr std::integral_constant<int, jj ^ 1> NN{};
                const int j = j0 + jj, rd = jj * L::SLAB, nx = (jj ^ 1) * L::SLAB;
                static_for<0, 4>([&](auto X) XQ_INLINE_LAMBDA {
                    constexpr int c = decltype(X)::value, h = c / 2, tt = c % 2;
                    constexpr std::integral_constant<int, (c + 3) & 3> BEFORE{};
                    constexpr std::integral_constant<int, (c + 1) & 3> NEXT{};
                    constexpr std::integral_constant<int, c == 0 ? jj ^ 1 : jj> NB{};
                    const uint32_t zr = rec[jj][tt][GPS == 2 ? h : 0];
                    if constexpr (c == 3) {
                        // By here every wave has all of this slab out of LDS, and its own part of the next in: the buffer takes the
                        // one after the next
                        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    }
                    P[c & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_frag(us[h][0], 0u, 0u, 0u), as_frag(perm_bytes(zr, zr, 0x01000100u), 0u, 0u, 0u), zero16, 0, 0, 0);
                    if constexpr (c == 1) read_start(rd, 1);
                    if constexpr (c == 3) { read_start(nx, 0); exchange(NN); }
                    if constexpr (tt == 0) more |= __any((int)(us[h][1] & flag)) ? 1ull << (j - slab0) : 0ull;
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<0, FOLD_DIGITS>([&](auto D) XQ_INLINE_LAMBDA {
                        constexpr int p = decltype(D)::value;
                        P[c & 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(digit(p), codes(F[c & 1]), P[c & 1], 2, 4, 0, (int)us[h][1],
                                                                                  p < 4 ? p : 0, p < 4 ? SCALE03 : SCALE4);
                        if constexpr (c == 1) read_digit(rd, 1, p);
                        if constexpr (c == 3) read_digit(nx, 0, p);
                        if constexpr (p == 0) unpack(std::integral_constant<int, c == 3 ? jj ^ 1 : jj>{}, NEXT);
                        else add_piece(BEFORE, NB, std::integral_constant<int, p - 1>{}, c == 0 || j <= last_slab);
                        if constexpr (c == 2 && p == 4) read_records(j + 1, NN);
                        if constexpr (c == 3 && p == 2) {
                            write_digits(rd);
                            load_digits(j + 3);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    if constexpr (c == 2) load_codes(j + 2, N);      // (all of this slab's codes are unpacked)
                });
            });
            if ((j0 + 2) % FLUSH == 0) flush();
        }
        static_for<0, 4>([&](auto K) XQ_INLINE_LAMBDA { add_piece(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{}, K, (last_slab - slab0) & 1); });     // the last chain

        // ---- further digits, where there are any
        for (int j = 0; more != 0ull; ++j, more >>= 1) {
            const int slab = slab0 + j;
            if (!(more & 1ull) || slab > last_slab) continue;
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                const uint32_t w = *reinterpret_cast<const uint32_t*>(ubase + (long long)slab * FOLD_UD_SLAB + h * FOLD_UD_HALF + START + lane * 8 + 4);
                const uint8_t* src = ubase + (long long)slab * FOLD_UD_SLAB + 2 * FOLD_UD_HALF + h * FOLD_UD_MORE;
                i32x8 dig[FOLD_DIGITS_MORE];
#pragma unroll
                for (int p = 0; p < FOLD_DIGITS_MORE; ++p) {
                    u32x4 d4 = *reinterpret_cast<const u32x4*>(src + p * 1024 + lane * 16);
                    u32x2 d2 = *reinterpret_cast<const u32x2*>(src + FOLD_DIGITS_MORE * 1024 + p * 512 + lane * 8);
                    if (!(w & flag)) { d4 = u32x4{0u, 0u, 0u, 0u}; d2 = u32x2{0u, 0u}; }                      // (a block without them)
                    dig[p] = i32x8{(int)d4[0], (int)d4[1], (int)d4[2], (int)d4[3], (int)d2[0], (int)d2[1], 0, 0};
                }
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    const uint32_t* cs = reinterpret_cast<const uint32_t*>(cbase + (long long)row[tt] * x.row_bytes + slab * ROWB + fold_block_channel<G>(h, half) / 4);
                    const uint32_t w0 = cs[0], w1 = cs[1], f[4] = {w0 & 0x33333333u, (w0 >> 2) & 0x33333333u, w1 & 0x33333333u, (w1 >> 2) & 0x33333333u};
                    const float sc = __uint_as_float(records[((slab - slab0) * GPS + (GPS == 2 ? h : 0)) * L::TOKENS + 32 * tt] & 0xFFFF0000u);
                    constexpr int LOW = TOP - 5 * FOLD_DIGITS, SCALES = LOW | (LOW - 5) << 8 | (LOW - 10) << 16;
                    f32x16 t = zero16;
                    t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(dig[2], codes(f), t, 2, 4, 0, (int)w, 2, SCALES);
                    t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(dig[1], codes(f), t, 2, 4, 0, (int)w, 1, SCALES);
                    t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(dig[0], codes(f), t, 2, 4, 0, (int)w, 0, SCALES);
#pragma unroll
                    for (int i = 0; i < 16; ++i) T[tt][i] = __builtin_fmaf(t[i], sc, T[tt][i]);
                }
            }
        }
        flush();
    }

    // ---- maxima of the tiles, weights.  Registers 4 i + [0, 4) are rows 8 i + 4 half + [0, 4)
    const float* rowfac = a.rowfac + ((long long)b * s.nrb + rb) * 32 + 4 * half;
    float4 f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const float4*>(rowfac + 8 * i);
    float* mx = reinterpret_cast<float*>(lds);                       // [32 tokens][row 32]
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float f4[4] = {f[i].x, f[i].y, f[i].z, f[i].w};
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
            float m[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float& v = S[tt][4 * i + r];
                v = tok0 + 32 * tt < len ? v * f4[r] : -INFINITY;
                m[r] = wave32_max(v);
            }
            if (c32 == 0) *reinterpret_cast<float4*>(mx + (wave * 2 + tt) * 32 + 8 * i + 4 * half) = make_float4(m[0], m[1], m[2], m[3]);
        }
    }
    __syncthreads();
    const long long out = ((long long)b * s.nrb + rb) * s.tiles + wt * 2 + wave / 2;                 // tile of 128 tokens
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r0 = 8 * i + 4 * half;
        const float* src = mx + (wave / 2) * 4 * 32 + r0;
        float4 M = *reinterpret_cast<const float4*>(src);
#pragma unroll
        for (int n = 1; n < 4; ++n) {
            const float4 u = *reinterpret_cast<const float4*>(src + n * 32);
            M.x = fmaxf(M.x, u.x); M.y = fmaxf(M.y, u.y); M.z = fmaxf(M.z, u.z); M.w = fmaxf(M.w, u.w);
        }
        if (wave % 2 == 0 && c32 == 0) *reinterpret_cast<float4*>(a.mtile + out * 32 + r0) = M;
        const float m[4] = {M.x, M.y, M.z, M.w};
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
            float* to = a.p + (out * 4 + (wave % 2) * 2 + tt) * FOLD_P_TILE32<2> + (r0 >> 4) * 512 + (r0 & 15) * 4 + (c32 >> 4) * 256 + 64 * (c32 & 3) + ((c32 >> 2) & 3);
#pragma unroll
            for (int r = 0; r < 4; ++r) to[4 * r] = __builtin_amdgcn_exp2f(S[tt][4 * i + r] - (m[r] == -INFINITY ? 0.0f : m[r]));    // (nothing visible: all weights 0)
        }
    }
}
