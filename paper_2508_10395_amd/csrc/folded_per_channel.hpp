// The folded score and value kernels over a per-channel cache (one scale and zero-point per channel and block of 64 or 128
// tokens); part of folded_attn.hip, inside its namespace.
//
// x^ = (code - c0) s + (z + c0 s) with c0 = 2^(BITS - 1).  Scores: the scale is a factor of the token operand, one packed fp16
// multiplication ((code - c0) has at most 3 significant bits, s has 8: exact, but that the operand is a multiple of 2^-24 and
// carries 2^-9, so that with scales more than 2^22 below the block's largest it is rounded, by at most 2^-31 of a code step of the
// largest), so every product of a tile goes straight into its scores; sum_c u[c] z[c] and sum_c u[c] s[c] are one more token tile, whose first columns hold z and s.
// Values: the codes are summed with the softmax weights alone, and every 64 tokens the sums are taken times the block's scales
// into y, z + c0 s times the sum of the weights (one more column tile, of ones) along with them.  The weights are cut to fp16
// hi + lo, with parts down to 2^-40, against the sequence's maximum of their row.  A block whose own maximum lies more than 2^16
// below that would keep too few digits there, and it may yet count, being far larger than the others: a range that holds such
// a block cuts the weights as they are stored, against the maximum of their own block (128 or 64 tokens, FoldShape::mhalf),
// and multiplies the rest of the factor in with the scales, in fp32.  So a block's largest weight is cut to 2^-25 of itself or
// better (a block 2^30 larger at weights of 2^-30 was off by 2e-4 without).  Both loops take as
// long (measured on a step of 8 x 4077 tokens); one loop that always does the latter, unrolled alone, ran 3 us slower.
// Bound by issue and by the latency of the loads, as the per-token kernels.  8 sequences of up to 4077 tokens, 3 bits, 32 KV
// heads, d = 4096, six layers in turn: scores 47 us, values 43 us with the windows (one layer again and again 36 and 42); the step
// 1432 us when K and V were rematerialised, 116 now.
#pragma once

template <int BITS>
constexpr int FOLD_PC_CENTRE = 1 << (BITS - 1);
// -c0 in the unit of fold_code, twice
template <int BITS>
__device__ __forceinline__ uint32_t fold_pc_add()
{
    constexpr _Float16 c = (_Float16)(-FOLD_PC_CENTRE<BITS> / FOLD_CODE_UNIT);
    const xq_f16x2 v = {c, c};
    return __builtin_bit_cast(uint32_t, v);
}

template <int BITS, int RT>
constexpr int FOLD_SCORE_PC_IMAGES = 8 * FOLD_TILE * 16 * BITS > FOLD_SCORE_RED<RT> ? 8 * FOLD_TILE * 16 * BITS : FOLD_SCORE_RED<RT>;
template <int BITS, int RT>
constexpr int FOLD_SCORE_PC_LDS = FOLD_SCORE_PC_IMAGES<BITS, RT> + 256;         // behind them: the blocks' largest numbers

// Workgroup and waves as in fold_scores_kernel (one tile, eight slab ways); NB blocks per tile of 128 tokens.  The first
// n_window workgroups (a multiple of 8) take the windows: few, and each slow at its one tile, they run beside the coded
// tiles' workgroups.
template <int BITS, int NB, int RT>
__global__ __launch_bounds__(512) void fold_scores_pc_kernel(const FoldScoreArgs a)
{
    constexpr int ROWB = 16 * BITS, NL = 2 * BITS;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FoldShape& s = a.s;
    const FoldSource& x = a.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if ((int)blockIdx.x < a.n_window) {
        fold_scores_dense<RT>(a, a.window, a.u_window, true, 8, lds);
        return;
    }
    FoldScorePlace o;
    if (!fold_score_place(s, false, false, 8, x.n_slabs, (int)blockIdx.x - a.n_window, wave, o)) return;
    const int b = o.b, rb = o.rb, len = o.len, tok0 = o.tile * FOLD_TILE;
    const int c16 = lane & 15, q = lane >> 4, d = x.n_slabs * 128;
    const int nblk = len / s.block, blk0 = tok0 / s.block;
    const uint8_t* cbase = x.codes + (long long)(s.b0 + b) * x.cap * x.row_bytes;
    const long long meta0 = (long long)(s.b0 + b) * (x.cap / s.block) * d;
    const uint8_t* ubase = a.u + ((long long)b * s.nrb + rb) * x.n_slabs * a.u_slab;
    const uint32_t uoff = lane * 16;
    const int slab0 = o.slab0, slab1 = o.slab1;
    uint8_t* image = lds + wave * (FOLD_TILE * ROWB);
    const uint16_t* srow[NB];
    const uint16_t* zrow[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const long long r = meta0 + (long long)min(blk0 + n, nblk - 1) * d;
        srow[n] = x.scale + r;
        zrow[n] = x.zero + r;
    }

    // powers of two that bring the largest scale and zero-point of a block below 2^15
    float fs[NB], fz[NB], ifs[NB], ifz[NB];
    {
        uint32_t* red = reinterpret_cast<uint32_t*>(lds + FOLD_SCORE_PC_IMAGES<BITS, RT>);
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            uint32_t ms = 0u, mz = 0u;
            for (int c = threadIdx.x * 8; c < d; c += 512 * 8) {
                const uint4 sv = *reinterpret_cast<const uint4*>(srow[n] + c), zv = *reinterpret_cast<const uint4*>(zrow[n] + c);
                const uint32_t s4[4] = {sv.x, sv.y, sv.z, sv.w}, z4[4] = {zv.x, zv.y, zv.z, zv.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ms = max(ms, max(s4[i] & 0x7FFFu, (s4[i] >> 16) & 0x7FFFu));
                    mz = max(mz, max(z4[i] & 0x7FFFu, (z4[i] >> 16) & 0x7FFFu));
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                ms = max(ms, (uint32_t)__shfl_xor((int)ms, off));
                mz = max(mz, (uint32_t)__shfl_xor((int)mz, off));
            }
            if (lane == 0) {
                red[(n * 2) * 8 + wave] = ms;
                red[(n * 2 + 1) * 8 + wave] = mz;
            }
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            uint32_t ms = 0u, mz = 0u;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                ms = max(ms, red[(n * 2) * 8 + w]);
                mz = max(mz, red[(n * 2 + 1) * 8 + w]);
            }
            const int es = ms ? min(141 - (int)(ms >> 7), 120) : 0, ez = mz ? min(141 - (int)(mz >> 7), 120) : 0;
            fs[n] = ldexpf(1.0f, es); ifs[n] = ldexpf(1.0f, -es);
            fz[n] = ldexpf(1.0f, ez); ifz[n] = ldexpf(1.0f, -ez);
        }
    }

    // codes: row by row through the wave's LDS image, as in fold_scores_kernel
    uint32_t voff[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int pc = k * 64 + lane;
        voff[k] = (uint32_t)min(tok0 + pc / BITS, len - 1) * (uint32_t)x.row_bytes + (uint32_t)(pc % BITS) * 16u;
    }
    f32x4 S[RT][8], Z[RT];
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        Z[rt] = zero4;
#pragma unroll
        for (int i = 0; i < 8; ++i) S[rt][i] = zero4;
    }
    // the extra token tile: column 2 n is block n's zero-points, column 2 n + 1 its scales (further columns are not used)
    const bool second = NB == 2 && (c16 & 2);
    const uint16_t* zsrc = (c16 & 1) ? (second ? srow[NB - 1] : srow[0]) : second ? zrow[NB - 1] : zrow[0];
    const float zfac = (c16 & 1) ? (second ? fs[NB - 1] : fs[0]) : second ? fz[NB - 1] : fz[0];
    if (slab0 < slab1) {
        uint4 u[2][RT][2][2];
        uint32_t cw[4][2], F[2][8], fac[2][NB][8], zf[8];
        uint4 rs[NB][2], rz[2];
        u32x4 cn[NL];
        auto load_u = [&](int slab, auto HF, auto I) XQ_INLINE_LAMBDA {
            constexpr int h = decltype(HF)::value, i = decltype(I)::value, rt = i >> 2, t = (i >> 1) & 1, k = i & 1;
            u[h][rt][t][k] = *reinterpret_cast<const uint4*>(ubase + (long long)slab * a.u_slab + rt * 8192 + h * 4096 + t * 2048 + k * 1024 + uoff);
        };
        // the lane's 16 channels of half slab h: 32 q + 16 h + [0, 16)
        auto load_fac = [&](int slab, int h) XQ_INLINE_LAMBDA {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int k = 0; k < 2; ++k) rs[n][k] = *reinterpret_cast<const uint4*>(srow[n] + slab * 128 + 32 * q + 16 * h + 8 * k);
        };
        auto load_z = [&](int slab, int h) XQ_INLINE_LAMBDA {
#pragma unroll
            for (int k = 0; k < 2; ++k) rz[k] = *reinterpret_cast<const uint4*>(zsrc + slab * 128 + 32 * q + 16 * h + 8 * k);
        };
        // operand dword k: channel k of either octet, times f
        auto to_fp16 = [&](const uint4 (&r)[2], float f, uint32_t (&out)[8]) XQ_INLINE_LAMBDA {
            const uint32_t r0[4] = {r[0].x, r[0].y, r[0].z, r[0].w}, r1[4] = {r[1].x, r[1].y, r[1].z, r[1].w};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float v0 = (k & 1) ? bf16_hi_to_f32(r0[k >> 1]) : bf16_lo_to_f32(r0[k >> 1]);
                const float v1 = (k & 1) ? bf16_hi_to_f32(r1[k >> 1]) : bf16_lo_to_f32(r1[k >> 1]);
                const xq_f32x2 w = {v0 * f, v1 * f};
                out[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(w, xq_f16x2));
            }
        };
        auto read_unit = [&](auto T) XQ_INLINE_LAMBDA {
            constexpr int t = decltype(T)::value, h = (t >> 3) & 1, i = t & 7, n = t & 3;
            const uint32_t* w = reinterpret_cast<const uint32_t*>(image + (i * 16 + c16) * ROWB) + q * BITS;
            if constexpr (BITS == 2) { cw[n][0] = w[h]; cw[n][1] = 0u; }
            else if constexpr (BITS == 3) { cw[n][0] = w[h]; cw[n][1] = w[h + 1]; }
            else { cw[n][0] = w[2 * h]; cw[n][1] = w[2 * h + 1]; }
        };
        uint32_t m0, m1;
        auto unpack = [&](auto T, auto K) XQ_INLINE_LAMBDA {
            constexpr int t = decltype(T)::value, h = (t >> 3) & 1, n = t & 3, k = decltype(K)::value, nb = NB == 2 ? (t >> 2) & 1 : 0;
            if constexpr (k == 0) {
                m1 = 0u;
                if constexpr (BITS == 2) {
                    m0 = cw[n][0];
                } else if constexpr (BITS == 3) {
                    m0 = perm_bytes(cw[n][1], cw[n][0], h == 0 ? 0x04030100u : 0x06050302u);
                    m1 = perm_bytes(cw[n][1], cw[n][0], h == 0 ? 0x05040201u : 0x07060403u);
                } else {
                    m0 = perm_bytes(cw[n][1], cw[n][0], 0x05040100u);
                    m1 = perm_bytes(cw[n][1], cw[n][0], 0x07060302u);
                }
            }
            const xq_f16x2 v = __builtin_bit_cast(xq_f16x2, fold_code<BITS, k>(m0, m1, fold_pc_add<BITS>()));
            F[t & 1][k] = __builtin_bit_cast(uint32_t, v * __builtin_bit_cast(xq_f16x2, fac[h][nb][k]));
        };
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
        static_for<0, NL>([&](auto K) XQ_INLINE_LAMBDA { load_codes(slab0, K); });
        load_fac(slab0, 0);
        static_for<0, 4 * RT>([&](auto I) XQ_INLINE_LAMBDA { load_u(slab0, std::integral_constant<int, 0>{}, I); });
        write_codes();
#pragma unroll
        for (int n = 0; n < NB; ++n) to_fp16(rs[n], fs[n], fac[0][n]);
        read_unit(std::integral_constant<int, 0>{});
        read_unit(std::integral_constant<int, 1>{});
        static_for<0, 8>([&](auto K) XQ_INLINE_LAMBDA { unpack(std::integral_constant<int, 0>{}, K); });
        for (int slab = slab0; slab < slab1; slab += o.step) {
            const int snext = slab + o.step < slab1 ? slab + o.step : slab;
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, 16>([&](auto T) XQ_INLINE_LAMBDA {
                constexpr int t = decltype(T)::value, h = t >> 3, i = t & 7;
                if constexpr (i == 0) {
                    static_for<0, 4 * RT>([&](auto I) XQ_INLINE_LAMBDA { load_u(h == 0 ? slab : snext, std::integral_constant<int, h ^ 1>{}, I); });
                    load_z(slab, h);
                    load_fac(h == 0 ? slab : snext, h ^ 1);
                }
                if constexpr (t >= 2 && t < 2 + NL) load_codes(snext, std::integral_constant<int, t - 2>{});
                if constexpr (t == 14) write_codes();                // (units 14 and 15 of this slab have been read)
                read_unit(std::integral_constant<int, t + 2>{});
                if constexpr (i == 5) to_fp16(rz, zfac, zf);
                if constexpr (i == 6)
#pragma unroll
                    for (int n = 0; n < NB; ++n) to_fp16(rs[n], fs[n], fac[h ^ 1][n]);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, 4 * RT>([&](auto M) XQ_INLINE_LAMBDA {
                    constexpr int m = decltype(M)::value, rt = m % RT, k = 1 - (m / RT) % 2, tick = m / (2 * RT);
                    const uint32_t* f = &F[t & 1][4 * tick];
                    S[rt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, u[h][rt][tick][k]), as_frag(f[0], f[1], f[2], f[3]), S[rt][i], 0, 0, 0);
                    static_for<0, 2 / RT>([&](auto E) XQ_INLINE_LAMBDA {
                        unpack(std::integral_constant<int, t + 1>{}, std::integral_constant<int, m * (2 / RT) + decltype(E)::value>{});
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (i == 7)
                    static_for<0, 4 * RT>([&](auto M) XQ_INLINE_LAMBDA {
                        constexpr int m = decltype(M)::value, rt = m % RT, k = 1 - (m / RT) % 2, tick = m / (2 * RT);
                        const uint32_t* f = &zf[4 * tick];
                        Z[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, u[h][rt][tick][k]), as_frag(f[0], f[1], f[2], f[3]), Z[rt], 0, 0, 0);
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        // to the unit of the codes: scales out, z + c0 s in
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    const float z = __shfl(Z[rt][r], (lane & 48) + 2 * n), sc = __shfl(Z[rt][r], (lane & 48) + 2 * n + 1);
                    const float off = (z * ifz[n] + sc * (ifs[n] * (float)FOLD_PC_CENTRE<BITS>)) * (1.0f / FOLD_CODE_UNIT);
#pragma unroll
                    for (int i = 8 / NB * n; i < 8 / NB * (n + 1); ++i) S[rt][i][r] = __builtin_fmaf(S[rt][i][r], ifs[n], off);
                }
    }
    fold_scores_finish<RT>(s, a.rowfac, a.p, a.mtile, S, reinterpret_cast<float*>(lds), o, lane, wave);
}

template <int RT>
struct FoldValuePcLds {
    static constexpr int W_BYTES = 8 * RT * 2 * 1024;                           // [tile32][rt][hi, lo][lane 64][16 B]
    static constexpr int M_OFF = 2 * W_BYTES;
    static constexpr int F_BYTES = 4 * 16 * RT * 4;                             // factors of a tile's rows, per 64 tokens
    static constexpr int F_OFF = M_OFF + 16 * RT * 4 * 34;
    static constexpr int L_OFF = F_OFF + 2 * F_BYTES;
    static constexpr int LOOP = L_OFF + 8 * 16 * RT * 4;
    static constexpr int RED = 8 * RT * 8 * 1024;
    static constexpr int TOTAL = LOOP > RED ? LOOP : RED;
};

// Workgroup and waves as in fold_values_kernel: two slab ways, four token ways of 64 of the 256 tokens staged at a time.
template <int BITS, int RT>
__global__ __launch_bounds__(512) void fold_values_pc_kernel(const FoldValueArgs a)
{
    typedef FoldValuePcLds<RT> L;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const FoldShape& s = a.s;
    if ((int)blockIdx.x < a.n_window) {
        fold_values_dense<RT>(a, a.window, true, lds);
        return;
    }
    FoldValuePlace o;
    if (!fold_value_place(s, false, a.cblocks, (int)blockIdx.x - a.n_window, o)) return;
    const FoldSource& x = a.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, q = lane >> 4;
    const int sw = wave & 1, tw = wave >> 1;
    const int slab = o.cblk * 2 + sw;
    const bool live = slab < x.n_slabs;
    const long long seq = s.b0 + o.b;
    float* mrow = reinterpret_cast<float*>(lds + L::M_OFF) + 32 * 16 * RT;
    fold_row_maxima<RT, FOLD_RANGE_LOW>(s, a.mtile, o.b, o.rb, reinterpret_cast<float*>(lds + L::M_OFF), mrow, (2 * o.t0) << s.mhalf, (2 * o.t1) << s.mhalf);
    // does the range hold a block far below its row's maximum?
    const int any_row = lane % (16 * RT);
    const bool apart = __ballot(mrow[16 * RT + any_row] - mrow[any_row] < -16.0f && o.rb * 16 * RT + any_row < s.R) != 0;

    constexpr int NP = 2 * RT;
    constexpr float UP = 32768.0f;                                  // the weights are at most 1: fp16 parts below 2^15
    const float* psrc = a.p + (((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) * 4 * FOLD_P_TILE32<RT>;
    const int prow = RT == 2 ? ((wave >> 1) & 1) * 16 + c16 : c16;
    const float M = mrow[prow];
    const float* msrc = a.mtile + ((((long long)o.b * s.nrb + o.rb) * s.tiles + o.tile0) << s.mhalf) * 16 * RT + prow;
    float4 pv[NP];
    float fm[NP];
    auto load_stage = [&](int t) XQ_INLINE_LAMBDA {
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const int g64 = RT == 2 ? e : 2 * e + (wave >> 2);
            fm[e] = t * FOLD_VTILE + g64 * 64 < o.len ? msrc[(long long)((4 * t + g64) >> (1 - s.mhalf)) * 16 * RT] : -INFINITY;
            pv[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if ((2 * t + e / RT) * FOLD_TILE < o.len) pv[e] = *reinterpret_cast<const float4*>(psrc + (long long)t * 8 * FOLD_P_TILE32<RT> + (e * 512 + tid) * 4);
        }
    };
    float lacc = 0.0f;
    // (a piece belongs to one row and 64 tokens: the first lanes of four waves, RT = 1, or two hold all the factors)
    auto write_stage = [&](auto APART, int buf) XQ_INLINE_LAMBDA {
        constexpr bool apart = decltype(APART)::value;
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const float f = fm[e] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(fm[e] - M);
            if constexpr (apart) {
                if (q == 0 && (RT == 2 ? wave == 0 || wave == 2 : (wave & 3) == 0))
                    reinterpret_cast<float*>(lds + L::F_OFF + buf * L::F_BYTES)[(RT == 2 ? e : 2 * e + (wave >> 2)) * 16 * RT + prow] = f;
                lacc += ((pv[e].x + pv[e].y) + (pv[e].z + pv[e].w)) * f;
            }
            const float v[4] = {apart ? pv[e].x : pv[e].x * f, apart ? pv[e].y : pv[e].y * f, apart ? pv[e].z : pv[e].z * f, apart ? pv[e].w : pv[e].w * f};
            if constexpr (!apart) lacc += (v[0] + v[1]) + (v[2] + v[3]);
            uint32_t hi[2], lo[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float w0 = v[2 * i] * UP, w1 = v[2 * i + 1] * UP;
                const xq_f16x2 hh = {(_Float16)w0, (_Float16)w1};
                const xq_f16x2 ll = {(_Float16)(w0 - (float)hh.x), (_Float16)(w1 - (float)hh.y)};
                hi[i] = __builtin_bit_cast(uint32_t, hh);
                lo[i] = __builtin_bit_cast(uint32_t, ll);
            }
            // piece e 512 + tid of [tile32][rt][half of the slots][lane]
            const int idx = e * 512 + tid, hs = (idx >> 6) & 1, blk = idx >> 7;
            uint8_t* dst = lds + buf * L::W_BYTES + blk * 2048 + lane * 16 + hs * 8;
            *reinterpret_cast<uint2*>(dst) = make_uint2(hi[0], hi[1]);
            *reinterpret_cast<uint2*>(dst + 1024) = make_uint2(lo[0], lo[1]);
        }
    };
    // codes: octet n = c16 of the wave's slab for tokens 4 i + q of its 32
    const uint8_t* cbase = x.codes + seq * x.cap * x.row_bytes + (live ? slab : 0) * (16 * BITS);
    const uint32_t oct = BITS == 3 ? 3 * c16 - (c16 > 0) : BITS * c16;
    uint32_t voff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) voff[i] = (uint32_t)(4 * i + q) * (uint32_t)x.row_bytes + oct;
    auto load_codes = [&](int k32, uint32_t (&r)[8]) XQ_INLINE_LAMBDA {
        const uint8_t* base = cbase + (long long)k32 * 32 * x.row_bytes;
        uint32_t off[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) off[i] = voff[i];
        if (k32 * 32 + 32 > o.len) {                                // past the length: the last row again
            base = cbase;
#pragma unroll
            for (int i = 0; i < 8; ++i) off[i] = (uint32_t)min(k32 * 32 + 4 * i + q, o.len - 1) * (uint32_t)x.row_bytes + oct;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (BITS == 2) r[i] = *reinterpret_cast<const uint16_t*>(base + off[i]);
            else if constexpr (BITS == 4) r[i] = *reinterpret_cast<const uint32_t*>(base + off[i]);
            else __builtin_memcpy(&r[i], base + off[i], 4);         // three of these four bytes (lane 0: the first three)
        }
    };
    const uint32_t sel0 = c16 ? 0x06050201u : 0x05040100u, sel1 = c16 ? 0x07060302u : 0x06050201u;
    // scales and zero-points of the lane's eight channels in the block of the wave's 64 tokens
    const int nblk = o.len / s.block, d = x.n_slabs * 128;
    const long long meta0 = seq * (x.cap / s.block) * d + (live ? slab : 0) * 128 + 8 * c16;
    uint4 sv, zv;
    auto load_meta = [&](int t) XQ_INLINE_LAMBDA {
        const long long at = meta0 + (long long)min((t * FOLD_VTILE + tw * 64) / s.block, nblk - 1) * d;
        sv = *reinterpret_cast<const uint4*>(x.scale + at);
        zv = *reinterpret_cast<const uint4*>(x.zero + at);
    };
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 y[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int k = 0; k < 8; ++k) y[rt][k] = zero4;
    uint32_t raw[2][8];
    const f16x8 ones = as_frag(0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u);
    auto walk = [&](auto APART) XQ_INLINE_LAMBDA {
        constexpr bool apart = decltype(APART)::value;
        load_stage(o.t0);
        load_codes(o.t0 * 8 + tw * 2, raw[0]);
        load_codes(o.t0 * 8 + tw * 2 + 1, raw[1]);
        load_meta(o.t0);
        write_stage(APART, 0);
        __syncthreads();
        for (int t = o.t0; t < o.t1; ++t) {
            const int buf = (t - o.t0) & 1, next = min(t + 1, o.t1 - 1);
            const bool more = t + 1 < o.t1;
            if (more) load_stage(t + 1);
            const uint8_t* wb = lds + buf * L::W_BYTES;
            f32x4 acc[RT][8], psum[RT];
            static_for<0, 2>([&](auto ST) XQ_INLINE_LAMBDA {
                constexpr int st = decltype(ST)::value;
                uint4 w[RT][2];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int k = 0; k < 2; ++k) w[rt][k] = *reinterpret_cast<const uint4*>(wb + (((tw * 2 + st) * RT + rt) * 2 + k) * 1024 + lane * 16);
                uint32_t m0[4], m1[4];
                const uint32_t (&r)[8] = raw[st];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (BITS == 2) { m0[j] = r[2 * j] | (r[2 * j + 1] << 16); m1[j] = 0u; }
                    else if constexpr (BITS == 3) { m0[j] = perm_bytes(r[2 * j + 1], r[2 * j], sel0); m1[j] = perm_bytes(r[2 * j + 1], r[2 * j], sel1); }
                    else { m0[j] = perm_bytes(r[2 * j + 1], r[2 * j], 0x05040100u); m1[j] = perm_bytes(r[2 * j + 1], r[2 * j], 0x07060302u); }
                }
                load_codes(next * 8 + tw * 2 + st, raw[st]);
                static_for<0, 9>([&](auto K) XQ_INLINE_LAMBDA {          // eight column tiles, and one of ones
                    constexpr int k = decltype(K)::value;
                    f16x8 f = ones;
                    if constexpr (k < 8) {
                        uint32_t F[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) F[j] = fold_code<BITS, k>(m0[j], m1[j], fold_pc_add<BITS>());
                        f = as_frag(F[0], F[1], F[2], F[3]);
                    }
#pragma unroll
                    for (int p = 1; p >= 0; --p)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) {
                            f32x4& to = *(k < 8 ? &acc[rt][k & 7] : &psum[rt]);
                            to = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[rt][p]), f, st == 0 && p == 1 ? zero4 : to, 0, 0, 0);
                        }
                });
            });
            if constexpr (apart)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const float4 fv = *reinterpret_cast<const float4*>(lds + L::F_OFF + buf * L::F_BYTES + (tw * 16 * RT + rt * 16 + 4 * q) * 4);
                    const float fac[4] = {fv.x, fv.y, fv.z, fv.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        psum[rt][r] *= fac[r];
#pragma unroll
                        for (int k = 0; k < 8; ++k) acc[rt][k][r] *= fac[r];
                    }
                }
            const uint32_t s4[4] = {sv.x, sv.y, sv.z, sv.w}, z4[4] = {zv.x, zv.y, zv.z, zv.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float sc = (k & 1) ? bf16_hi_to_f32(s4[k >> 1]) : bf16_lo_to_f32(s4[k >> 1]);
                const float z = (k & 1) ? bf16_hi_to_f32(z4[k >> 1]) : bf16_lo_to_f32(z4[k >> 1]);
                const float off = __builtin_fmaf(sc, (float)FOLD_PC_CENTRE<BITS>, z), f = sc * FOLD_CODE_UNIT;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[rt][k][r] = __builtin_fmaf(acc[rt][k][r], f, __builtin_fmaf(psum[rt][r], off, y[rt][k][r]));
            }
            load_meta(next);
            if (more) write_stage(APART, buf ^ 1);
            __syncthreads();
        }
    };
    if (apart) walk(std::true_type{});
    else walk(std::false_type{});
    if (o.cblk == 0) {
        fold_denominators<RT>(a, o, lacc, 1.0f, reinterpret_cast<float*>(lds + L::L_OFF));
        __syncthreads();
    }
    // the four token ways meet in LDS; token way tw sums half a row tile (rt, four column tiles) of its slab
    f32x4 t[1][4];
    fold_meet<RT, 8>(y, lds, wave, lane, t);
    if (live && tw < 2 * RT) {
        const long long yrow0 = ((long long)o.split * s.nb + o.b) * s.R;
        const int rt = tw >> 1, kg = tw & 1;
        constexpr float down = 1.0f / UP;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = o.rb * 16 * RT + rt * 16 + 4 * q + r;
            if (row < s.R)
                *reinterpret_cast<float4*>(a.y + (yrow0 + row) * (x.n_slabs * 128) + slab * 128 + 8 * c16 + 4 * kg) =
                    make_float4(t[0][0][r] * down, t[0][1][r] * down, t[0][2][r] * down, t[0][3][r] * down);
        }
    }
}
