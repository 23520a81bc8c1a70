// Down-projection of layer inputs into the latent spaces of the K and V projections
// (Sec. 3.3.1 of arxiv 2508.10395: for GQA models the cache holds X Uk and X Uv, where
// Wk = Uk Sk Bk^T and Wv = Uv Sv Bv^T are SVDs computed offline).
//
// out[m][n] = bf16( sum_c x[m][c] * Ut[n][c] ),  fp32 accumulation, one RNE rounding.
// Ut is U transposed (one row per latent channel), so both MFMA operands read 8 consecutive
// contraction indices with one 16-byte load.  A workgroup computes a 32 x 32 output tile; its 8
// waves each take one eighth of the contraction, 16 channels after the other, and the partial tiles
// are summed through LDS in fixed order.  Few rows (decode: M = batch) leave that kernel with fewer
// workgroups than CUs; they take latent_project_rows16_kernel, which adds up in the same order: a
// row's latents have the same bits however many rows come with it.
//
// Cross-layer variant (Sec. 3.3.2): the projected rows are deltas x - a against the accumulator
// rows X^_{i-1}.  The fp32 difference of two bf16 values does not fit one bf16, so it enters the
// MFMA as a bf16 hi part plus a bf16 lo part (two MFMAs per k-step; what is left is below 2^-16 of
// the delta).
#include <type_traits>

#include "common.hpp"

namespace xq {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// 8 bf16 (one 16-byte load) -> fp32
__device__ __forceinline__ void widen8(const uint4& v, float (&f)[8])
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = bf16_lo_to_f32(w[i]);
        f[2 * i + 1] = bf16_hi_to_f32(w[i]);
    }
}

// x - s of 8 channels as bf16 hi + lo operands
__device__ __forceinline__ void delta_parts(const uint4& x, const uint4& s, uint4& vh, uint4& vl)
{
    float xf[8], sf[8];
    widen8(x, xf);
    widen8(s, sf);
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float d0 = xf[2 * i] - sf[2 * i], d1 = xf[2 * i + 1] - sf[2 * i + 1];
        hi[i] = pack_bf16x2_rne(d0, d1);
        lo[i] = pack_bf16x2_rne(d0 - bf16_lo_to_f32(hi[i]), d1 - bf16_hi_to_f32(hi[i]));
    }
    vh = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    vl = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// Between a wave's writes to LDS and its own lanes' reads of them, and the other way round: the LDS unit keeps a wave's order, the
// compiler has to.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One round of a wave: STEPS times 16 channels from channel k on, all of them asked for before the first product (the fence keeps
// the loads in front of it).  Four steps (two of deltas) leave three or four workgroups to a CU, which hide more than longer rounds
// do.  One step at a time / these / 16: 512 rows of d = 4096 to 512 latent channels 19.9 / 16.3 / 16.5 us, 2048 rows of d = 256
// to 2048 18.3 / 17.2 / 27.9, of d = 5120 333 / 282 / 303; deltas 29.5 / 24.9 / 27.3, 25.8 / 26.5 / 40.9, 502 / 433 / 490.
template <int STEPS, bool DELTA>
__device__ __forceinline__ void project_round(const uint16_t* ap, const uint16_t* bp, const uint16_t* sp, int k, f32x16& acc)
{
    uint4 x[STEPS], b[STEPS], s[DELTA ? STEPS : 1];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        b[i] = *reinterpret_cast<const uint4*>(bp + k + 16 * i);
        x[i] = *reinterpret_cast<const uint4*>(ap + k + 16 * i);
        if constexpr (DELTA) s[i] = *reinterpret_cast<const uint4*>(sp + k + 16 * i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        if constexpr (DELTA) {
            uint4 vh, vl;
            delta_parts(x[i], s[i], vh, vl);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vl), __builtin_bit_cast(bf16x8, b[i]),
                                                          acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vh), __builtin_bit_cast(bf16x8, b[i]),
                                                          acc, 0, 0, 0);
        } else {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[i]), __builtin_bit_cast(bf16x8, b[i]),
                                                          acc, 0, 0, 0);
        }
    }
}

// DELTA: row m = b * T + t of x is paired with accumulator row start[b] + t of sequence b
template <bool DELTA>
__global__ __launch_bounds__(512) void latent_project_kernel(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ ut,
                                                             uint16_t* __restrict__ out, int M, int d, int n_lat,
                                                             const uint16_t* __restrict__ a, int T, int cap,
                                                             const BatchI32 start)
{
    __shared__ float red[8][32][33];
    const int nb = blockIdx.x, mb = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int r = lane & 31, kb = lane >> 5;
    const int row = min(mb * 32 + r, M - 1);            // rows past M repeat the last one, never stored
    const int col = nb * 32 + r;
    const int steps = d >> 7;                            // contraction share of one wave, in steps of 16 channels
    const uint16_t* ap = x + (long long)row * d + wave * steps * 16 + kb * 8;
    const uint16_t* bp = ut + (long long)col * d + wave * steps * 16 + kb * 8;
    const uint16_t* sp = nullptr;
    if constexpr (DELTA) {
        const int b = row / T, t = row - b * T;
        sp = a + ((long long)b * cap + start.v[b] + t) * d + wave * steps * 16 + kb * 8;
    }
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    constexpr int MOST = DELTA ? 2 : 4;
    int i = 0;
    for (; i + MOST <= steps; i += MOST) project_round<MOST, DELTA>(ap, bp, sp, i * 16, acc);
    if (MOST > 2 && steps - i >= 2) { project_round<2, DELTA>(ap, bp, sp, i * 16, acc); i += 2; }
    if (steps - i >= 1) project_round<1, DELTA>(ap, bp, sp, i * 16, acc);
    // accumulator element i of lane (r, kb) is D[m][n] with n = r, m = 8 (i/4) + 4 kb + i%4
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][8 * (e >> 2) + 4 * kb + (e & 3)][r] = acc[e];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 1024; idx += 512) {
        const int m = idx >> 5, n = idx & 31;
        float s = red[0][m][n];
#pragma unroll
        for (int w = 1; w < 8; ++w) s += red[w][m][n];
        if (mb * 32 + m < M) out[(long long)(mb * 32 + m) * n_lat + nb * 32 + n] = (uint16_t)f32_to_bf16_rne(s);
    }
}

// The same for few rows, to the bit: 16 x 16 output tiles, in a corner of the same products, whose other rows and columns repeat
// them.  An operand load of the kernel above touches 32 cache lines for 32 bytes each, which bounds it once its loads are in
// flight (16 rows of d = 4096 to 2048 latent channels 13 us); here rows are read by whole lines, eight of them a load, and go
// through LDS into operand order, 512 channels (256 of deltas) asked for before the first is used.  Pieces of 16 bytes are
// swizzled by the row against bank conflicts.  16 rows to 2048 latent channels 8.6 us (19.2 in 32 x 32 tiles with one step's
// loads at a time), of deltas 12.7 (24.8); the 16.8 MB of Ut take 3.
constexpr int LP_ROW_BYTES = 128;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool DELTA>
__global__ __launch_bounds__(512) void latent_project_rows16_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ ut,
                                                                    uint16_t* __restrict__ out, int M, int d, int n_lat,
                                                                    const uint16_t* __restrict__ a, int T, int cap, const BatchI32 start)
{
    constexpr int IMAGE = 16 * LP_ROW_BYTES, PARTS = DELTA ? 3 : 2;      // of a wave: rows (hi, lo of deltas), columns
    __shared__ __attribute__((aligned(16))) uint8_t lds[8][PARTS][IMAGE];
    __shared__ float red[8][16][17];
    const int nb = blockIdx.x, mb = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int share = d >> 3, steps = d >> 7;            // a wave's channels, and its steps of 16
    // as loaded: rows 0-7 and 8-15 of the tile, 8 lanes a row
    const int row8 = lane >> 3, piece = lane & 7;
    const uint16_t *xr[2], *ur[2], *ar[2] = {};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = min(mb * 16 + row8 + 8 * i, M - 1);             // rows past M repeat the last one, never stored
        xr[i] = x + (long long)row * d + wave * share;
        ur[i] = ut + (long long)(nb * 16 + row8 + 8 * i) * d + wave * share;
        if constexpr (DELTA) {
            const int b = row / T, t = row - b * T;
            ar[i] = a + ((long long)b * cap + start.v[b] + t) * d + wave * share;
        }
    }
    uint8_t* put = &lds[wave][0][0] + row8 * LP_ROW_BYTES + ((piece ^ row8) << 4);
    // as operands: lane (r, kb) has channels 8 kb + [0, 8) of a step
    const int r = lane & 15, kb = lane >> 5;
    const uint8_t* get = &lds[wave][0][0] + r * LP_ROW_BYTES;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    // N pieces of 64 channels from the wave's channel k on; a single one may hold fewer steps
    auto round = [&](auto CHUNKS, int k, int n_steps) __attribute__((always_inline)) {
        constexpr int N = decltype(CHUNKS)::value;
        u32x4 xv[2 * N], uv[2 * N], av[DELTA ? 2 * N : 1];
        const int p8 = 8 * (N == 1 ? min(piece, 2 * n_steps - 1) : piece);
#pragma unroll
        for (int e = 0; e < 2 * N; ++e) {
            const int at = k + 64 * (e >> 1) + p8;
            uv[e] = *reinterpret_cast<const u32x4*>(ur[e & 1] + at);
            xv[e] = *reinterpret_cast<const u32x4*>(xr[e & 1] + at);
            if constexpr (DELTA) av[e] = *reinterpret_cast<const u32x4*>(ar[e & 1] + at);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 2 * N; ++e) {
            uint8_t* dst = put + (e & 1) * 8 * LP_ROW_BYTES;
            *reinterpret_cast<u32x4*>(dst) = uv[e];
            if constexpr (DELTA) {
                uint4 hi, lo;
                delta_parts(__builtin_bit_cast(uint4, xv[e]), __builtin_bit_cast(uint4, av[e]), hi, lo);
                *reinterpret_cast<uint4*>(dst + IMAGE) = hi;
                *reinterpret_cast<uint4*>(dst + 2 * IMAGE) = lo;
            } else {
                *reinterpret_cast<u32x4*>(dst + IMAGE) = xv[e];
            }
            if ((e & 1) == 0) continue;
            wave_lds_order();
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (N == 1 && s >= n_steps) break;
                const uint8_t* src = get + (((2 * s + kb) ^ (r & 7)) << 4);
                const bf16x8 u = *reinterpret_cast<const bf16x8*>(src);
                if constexpr (DELTA) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(src + 2 * IMAGE), u, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(src + IMAGE), u, acc, 0, 0, 0);
            }
            wave_lds_order();
        }
    };
    constexpr int MOST = DELTA ? 4 : 8;
    int s = 0;
    for (; s + 4 * MOST <= steps; s += 4 * MOST) round(std::integral_constant<int, MOST>{}, s * 16, 4);
    if (MOST > 4 && s + 16 <= steps) { round(std::integral_constant<int, 4>{}, s * 16, 4); s += 16; }
    if (s + 8 <= steps) { round(std::integral_constant<int, 2>{}, s * 16, 4); s += 8; }
    for (; s < steps; s += 4) round(std::integral_constant<int, 1>{}, s * 16, min(4, steps - s));
    // accumulator element i of lane (r, kb) is D[m][n] with n = r, m = 8 (i/4) + 4 kb + i%4
    if ((lane & 31) < 16)
#pragma unroll
        for (int i = 0; i < 8; ++i) red[wave][8 * (i >> 2) + 4 * kb + (i & 3)][r] = acc[i];
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = threadIdx.x >> 4, n = threadIdx.x & 15;
        float t = red[0][m][n];
#pragma unroll
        for (int w = 1; w < 8; ++w) t += red[w][m][n];
        if (mb * 16 + m < M) out[(long long)(mb * 16 + m) * n_lat + nb * 16 + n] = (uint16_t)f32_to_bf16_rne(t);
    }
}

template <bool DELTA>
static hipError_t launch_project(const uint16_t* x, const uint16_t* ut, uint16_t* out, int M, int d, int n_lat, const uint16_t* a, int T, int cap,
                                 const BatchI32& start, hipStream_t s)
{
    // As long as two workgroups a CU hold all 16 x 16 tiles.  us a call in 32 x 32 / 16 x 16 tiles, d = 4096, 2048 latent channels:
    // 16 rows 13.4 / 10.3, 64 rows 16.0 / 11.4, 128 rows 16.0 / 20.7; 512 latent channels: 256 rows 15.8 / 11.1, 512 rows 16.3 / 20.7.
    if ((long long)(n_lat / 16) * ((M + 15) / 16) <= 512)
        latent_project_rows16_kernel<DELTA><<<dim3(n_lat / 16, (M + 15) / 16), dim3(512), 0, s>>>(x, ut, out, M, d, n_lat, a, T, cap, start);
    else
        latent_project_kernel<DELTA><<<dim3(n_lat / 32, (M + 31) / 32), dim3(512), 0, s>>>(x, ut, out, M, d, n_lat, a, T, cap, start);
    return hipGetLastError();
}

hipError_t run_latent_project(const uint16_t* x, const uint16_t* ut, int M, int d, int n_lat, uint16_t* out,
                              hipStream_t s)
{
    return launch_project<false>(x, ut, out, M, d, n_lat, nullptr, 1, 0, BatchI32{}, s);
}

// x [B][T][d] against accumulator rows start[b] + t of acc [B][cap][d]
hipError_t run_latent_delta_project(const uint16_t* x, const uint16_t* acc, const uint16_t* ut, int B, int T, int cap,
                                    const BatchI32& start, int d, int n_lat, uint16_t* out, hipStream_t s)
{
    return launch_project<true>(x, ut, out, B * T, d, n_lat, acc, T, cap, start, s);
}

}  // namespace xq
