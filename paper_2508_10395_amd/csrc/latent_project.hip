// Down-projection of layer inputs into the latent spaces of the K and V projections
// (Sec. 3.3.1 of arxiv 2508.10395: for GQA models the cache holds X Uk and X Uv, where
// Wk = Uk Sk Bk^T and Wv = Uv Sv Bv^T are SVDs computed offline).
//
// out[m][n] = bf16( sum_c x[m][c] * Ut[n][c] ),  fp32 accumulation, one RNE rounding.
// Ut is U transposed (one row per latent channel), so both MFMA operands read 8 consecutive
// contraction indices with one 16-byte load.  A workgroup computes a 32 x 32 output tile; its 8
// waves each take one eighth of the contraction and the partial tiles are summed through LDS in
// fixed order.  Few rows (decode: M = batch) leave that kernel with fewer workgroups than CUs and eight waits for memory in a
// row; they take latent_project_rows16_kernel.
//
// Cross-layer variant (Sec. 3.3.2): the projected rows are deltas x - a against the accumulator
// rows X^_{i-1}.  The fp32 difference of two bf16 values does not fit one bf16, so it enters the
// MFMA as a bf16 hi part plus a bf16 lo part (two MFMAs per k-step; what is left is below 2^-16 of
// the delta).
#include "common.hpp"

namespace xq {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

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
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 31, kb = lane >> 5;
    const int row = min(mb * 32 + r, M - 1);            // rows past M repeat the last one, never stored
    const int col = nb * 32 + r;
    const int kchunk = d >> 3;                           // contraction share of one wave (multiple of 16)
    const uint16_t* ap = x + (long long)row * d + wave * kchunk + kb * 8;
    const uint16_t* bp = ut + (long long)col * d + wave * kchunk + kb * 8;
    const uint16_t* sp = nullptr;
    if constexpr (DELTA) {
        const int b = row / T, t = row - b * T;
        sp = a + ((long long)b * cap + start.v[b] + t) * d + wave * kchunk + kb * 8;
    }
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll 4
    for (int k = 0; k < kchunk; k += 16) {
        const uint4 xa = *reinterpret_cast<const uint4*>(ap + k);
        const uint4 b = *reinterpret_cast<const uint4*>(bp + k);
        if constexpr (DELTA) {
            const uint4 sa = *reinterpret_cast<const uint4*>(sp + k);
            uint4 vh, vl;
            delta_parts(xa, sa, vh, vl);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vl), __builtin_bit_cast(bf16x8, b),
                                                          acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vh), __builtin_bit_cast(bf16x8, b),
                                                          acc, 0, 0, 0);
        } else {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa), __builtin_bit_cast(bf16x8, b),
                                                          acc, 0, 0, 0);
        }
    }
    // accumulator element i of lane (r, kb) is D[m][n] with n = r, m = 8 (i/4) + 4 kb + i%4
#pragma unroll
    for (int i = 0; i < 16; ++i) red[wave][8 * (i >> 2) + 4 * kb + (i & 3)][r] = acc[i];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 1024; idx += 512) {
        const int m = idx >> 5, n = idx & 31;
        float s = red[0][m][n];
#pragma unroll
        for (int w = 1; w < 8; ++w) s += red[w][m][n];
        if (mb * 32 + m < M) out[(long long)(mb * 32 + m) * n_lat + nb * 32 + n] = (uint16_t)f32_to_bf16_rne(s);
    }
}

// The same for few rows: 16 x 16 output tiles, so that twice as many CUs read Ut, and sixteen waves that deal the steps of 32
// channels among themselves and ask for eight of them before the first is used.  Bound by the latency of that one round of
// loads: 16 rows of d = 4096 to 2048 latent channels 9.4 us (19 us in 32 x 32 tiles),
// its 16.8 MB take 3.
constexpr int LP_STEPS = 8;
template <bool DELTA>
__global__ __launch_bounds__(1024) void latent_project_rows16_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ ut,
                                                                     uint16_t* __restrict__ out, int M, int d, int n_lat,
                                                                     const uint16_t* __restrict__ a, int T, int cap, const BatchI32 start)
{
    __shared__ float red[16][16][17];
    const int nb = blockIdx.x, mb = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int row = min(mb * 16 + r, M - 1);             // rows past M repeat the last one, never stored
    const uint16_t* ap = x + (long long)row * d + q * 8;
    const uint16_t* bp = ut + (long long)(nb * 16 + r) * d + q * 8;
    const uint16_t* sp = nullptr;
    if constexpr (DELTA) {
        const int b = row / T, t = row - b * T;
        sp = a + ((long long)b * cap + start.v[b] + t) * d + q * 8;
    }
    const int steps = d >> 5;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = wave; s0 < steps; s0 += 16 * LP_STEPS) {
        uint4 xa[LP_STEPS], b[LP_STEPS], sa[DELTA ? LP_STEPS : 1];
#pragma unroll
        for (int i = 0; i < LP_STEPS; ++i) {
            const int k = min(s0 + 16 * i, steps - 1) * 32;
            b[i] = *reinterpret_cast<const uint4*>(bp + k);
            xa[i] = *reinterpret_cast<const uint4*>(ap + k);
            if constexpr (DELTA) sa[i] = *reinterpret_cast<const uint4*>(sp + k);
        }
#pragma unroll
        for (int i = 0; i < LP_STEPS; ++i) {
            if (s0 + 16 * i >= steps) break;
            if constexpr (DELTA) {
                uint4 vh, vl;
                delta_parts(xa[i], sa[i], vh, vl);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vl), __builtin_bit_cast(bf16x8, b[i]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vh), __builtin_bit_cast(bf16x8, b[i]), acc, 0, 0, 0);
            } else {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[i]), __builtin_bit_cast(bf16x8, b[i]), acc, 0, 0, 0);
            }
        }
    }
    // accumulator element i of lane (r, q) is D[m][n] with n = r, m = 4 q + i
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][4 * q + i][r] = acc[i];
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = threadIdx.x >> 4, n = threadIdx.x & 15;
        float s[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) s[w] = (red[w][m][n] + red[w + 4][m][n]) + (red[w + 8][m][n] + red[w + 12][m][n]);
        if (mb * 16 + m < M) out[(long long)(mb * 16 + m) * n_lat + nb * 16 + n] = (uint16_t)f32_to_bf16_rne((s[0] + s[1]) + (s[2] + s[3]));
    }
}

template <bool DELTA>
static hipError_t launch_project(const uint16_t* x, const uint16_t* ut, uint16_t* out, int M, int d, int n_lat, const uint16_t* a, int T, int cap,
                                 const BatchI32& start, hipStream_t s)
{
    // As long as two workgroups a CU hold all 16 x 16 tiles.  us with 32 x 32 / 16 x 16 tiles, d = 4096, 2048 latent channels: 16
    // rows 19.1 / 10.7, 64 rows 22.5 / 17.4, 128 rows 23 / 31; 512 latent channels: 256 rows 17.7 / 16.5, 512 rows 21 / 30.
    if ((long long)(n_lat / 16) * ((M + 15) / 16) <= 512)
        latent_project_rows16_kernel<DELTA><<<dim3(n_lat / 16, (M + 15) / 16), dim3(1024), 0, s>>>(x, ut, out, M, d, n_lat, a, T, cap, start);
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
