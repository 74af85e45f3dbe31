// GeMM^quant of a few rows (a decode step of few sequences): every weight byte is read once, by one wave, and there is
// nothing else to do, so the kernel is a stream of the weights with the matrix instructions hung behind it.
//
// A workgroup owns CT tiles of 16 columns and all M <= 32 rows; its eight waves share K (an eighth each).  A wave streams its
// part through a ring of its OWN in LDS (global_load_lds_dwordx4), so the main loop has no barrier at all: a wave waits
// for its own oldest loads and nothing else.  A unit of the ring is 16 rows of 128 bytes (two 1 KB loads of 8 whole cache
// lines): per step of 128 bytes of K, TM units of activation rows and CT units of weight rows.  v_mfma_*_16x16x64 (16-bit:
// x32, E4M3: x128) with the weight rows as first operand: lane l holds, for row l % 16, four consecutive columns 4 (l / 16)
// .. + 3 of each tile.  The eight partial sums meet in LDS once, in the order of the waves, and the epilogue runs on them in
// the order of the other kernels.
// Against 32-column tiles (the ring kernel of gemm_ring.h), 16-column ones give every CU its share at N = 4096 without a split
// of K over workgroups, i.e. without partial planes in memory and the launch that adds them.
//
// What bounds it: HBM, as far as the order of the requests lets it.  The waves' steps interleave, so that a workgroup walks its
// rows in order, eight lines at a time; an XCD's workgroups take neighbouring tiles and stand at the same K (the activations'
// lines are in its L2 then), and the XCDs start an eighth of K apart.  Against an eighth of K in one piece per wave and tiles dealt
// round-robin, us: INT8 3 x 12288 x 4096 12.7 -> 11.0, 3 x 16384 x 4096 15.8 -> 13.6 (5.0 TB/s with the launch), 3 x 8192 x 8192 15.8
// -> 13.2, BF16 3 x 4096 x 16384 40.9 -> 26.2; six units per wave rather than nine: 2 % on average.
//
// LN form: the activation rows are LN^quant of a 16-bit residual stream (the layer in front of QKV and FC1), computed by
// every workgroup for itself, a wave per row, under the first weights' latency: up to eight rows that costs less than the launch it
// replaces.  The codes stay in LDS; the ring then carries weights only.  us, three rows: LN^quant + QKV 3.7 + 11.2 -> 12.4, LN^quant +
// FC1 3.6 + 14.0 -> 15.4.
#include "gemm_common.h"

using namespace hero_gemm;

namespace {

// the residual's rows: none, four elements as one vector, element by element (16-bit products take any stride and address)
enum { RES_NONE = 0, RES_ALIGNED = 1, RES_ANY = 2 };
struct SkinnyArgs {
    GemmArgs g;
    int epi, c_dt, has_res;
    const void* h; const float* gamma; const float* beta; float eps;     // LN form: 16-bit rows [M][K], contiguous
};

constexpr int SKINNY_WAVES = 8, UNIT = 16 * 128;

// both 16-byte fragments of a 128-byte step
template <int ADT, typename ACC>
__device__ __forceinline__ ACC mfma_16(const v4i (&w)[2], const v4i (&a)[2], ACC c) {
    if constexpr (ADT == HERO_F8E4M3) {
        const v8i w8 = {w[0][0], w[0][1], w[0][2], w[0][3], w[1][0], w[1][1], w[1][2], w[1][3]};
        const v8i a8 = {a[0][0], a[0][1], a[0][2], a[0][3], a[1][0], a[1][1], a[1][2], a[1][3]};
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w8, a8, c, 0, 0, 0, 0, 0, 0);
    } else {
#pragma unroll
        for (int s = 0; s < 2; ++s) c = mfma16_step<ADT>(w[s], a[s], c);
        return c;
    }
}

// at most min(left, N) units of two loads outstanding
template <int N>
__device__ __forceinline__ void unit_wait(int left) {
    if constexpr (N > 0) {
        if (left >= N) { __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * N)); return; }
        unit_wait<N - 1>(left);
    } else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

// HDT: type of the rows in front of the fused LN^quant; -1: the activation rows are codes (or 16-bit values) in memory
template <int ADT, int CT, int TM, int HDT>
__global__ __launch_bounds__(SKINNY_WAVES * 64, 2) void skinny_gemm_kernel(SkinnyArgs sa) {
    using ACC = typename Acc4Of<ADT>::type;
    const GemmArgs& g = sa.g;
    constexpr bool LN = HDT >= 0, HP = ADT == HERO_BF16 || ADT == HERO_F16;
    constexpr int LN_ROWS = 8, LN_K = 4096;                         // the fused form's limits
    static_assert(!LN || (TM == 1 && !HP), "the fused LN^quant makes 8-bit codes of at most eight rows");
    constexpr int AU = LN ? 0 : TM, PER = AU + CT;                  // units of a step: activation rows first
    constexpr int NU = 6;                                           // units of a wave's ring
    constexpr int RING = NU * UNIT, POOL = SKINNY_WAVES * RING;
    static_assert(SKINNY_WAVES * CT * TM * 1024 <= POOL, "the partial sums fit the rings");
    __shared__ __attribute__((aligned(1024))) int8_t smem[POOL + (LN ? LN_ROWS * LN_K : 0)];
    __shared__ float srow[LN_ROWS];
    int8_t* const scode = smem + POOL;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD takes neighbouring tiles
    const int xcd = blockIdx.x % NUM_XCD, n0 = (xcd * g.per_xcd + (int)(blockIdx.x / NUM_XCD)) * (CT * 16);
    if (n0 >= g.N) return;
    const int steps = g.K >> 10;                                    // 128-byte steps of a wave: K is a multiple of 8 * 128
    const int kbeg = wave * 128, KSTEP = SKINNY_WAVES * 128;     // the waves' steps interleave: together they walk each row in order

    // the epilogue's vectors of this thread's four columns, on their way before everything else
    constexpr int SLOTS = CT * TM * 64;
    const int ct_e = wave / TM, m_e = (wave % TM) * 16 + (lane & 15), n_e = min(n0 + ct_e * 16 + (lane >> 4) * 4, g.N - 4);
    const bool out = tid < SLOTS && m_e < g.M && n0 + ct_e * 16 < g.N;
    v4f cs = {1, 1, 1, 1}, bs = {0, 0, 0, 0}, os = {1, 1, 1, 1};
    float rs = 1.0f;
    if (tid < SLOTS) {                                              // (uniform branches, clamped addresses: nothing waits here)
        if (!HP)
#pragma unroll
            for (int t = 0; t < 4; ++t) cs[t] = g.b_col_scale[n_e + t];       // (the vectors need no alignment of their own)
        if (g.bias)
#pragma unroll
            for (int t = 0; t < 4; ++t) bs[t] = g.bias[n_e + t];
        if (sa.epi == HERO_EPI_GELU_REQUANT)
#pragma unroll
            for (int t = 0; t < 4; ++t) os[t] = g.out_col_scale[n_e + t];
        if (!LN && !HP && g.a_row_scale) rs = g.a_row_scale[min(m_e, g.M - 1)];
    }

    // loader: a load takes 8 rows of 128 bytes; lane l owns row l / 8 of them and stores chunk (l % 8) ^ (row & 7) of it
    const int lrow = lane >> 3;
    const uint32_t lc = (uint32_t)(((lane & 7) ^ lrow) * 16);
    uint32_t ow[CT][2], oa[TM][2];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u) ow[c][u] = (uint32_t)min(c * 16 + u * 8 + lrow, g.N - 1 - n0) * (uint32_t)g.ldb + lc;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) oa[i][u] = (uint32_t)min(i * 16 + u * 8 + lrow, g.M - 1) * (uint32_t)g.lda + lc;
    const int8_t* const wb = g.Bt + (int64_t)n0 * g.ldb + kbeg;
    const int8_t* const ab = g.A + kbeg;
    const uint32_t ring = __builtin_amdgcn_readfirstlane(lds_offset(smem) + wave * RING);
    // the issue stream: unit j of step is (both known at compile time but for the slot)
    const int rot = xcd * steps / NUM_XCD;
    int is = rot, islot = 0;
    auto issue = [&](auto J) {
        constexpr int j = decltype(J)::value;
        const uint32_t dst = ring + islot * UNIT;
        if constexpr (j < AU) {
            dma16s(oa[j][0], ab + is * KSTEP, dst);
            dma16s(oa[j][1], ab + is * KSTEP, dst + 1024);
        } else {
            dma16s(ow[j - AU][0], wb + is * KSTEP, dst);
            dma16s(ow[j - AU][1], wb + is * KSTEP, dst + 1024);
        }
        islot = islot + 1 == NU ? 0 : islot + 1;
        if constexpr (j == PER - 1) is = is + 1 == steps ? 0 : is + 1;
    };
    const int total = steps * PER;
    auto fill = [&]() {                                             // NU units, or all there are
        static_for<NU>([&](auto U) { if (decltype(U)::value < total) issue(std::integral_constant<int, decltype(U)::value % PER>{}); });
    };

    if constexpr (LN) {
        // LN^quant of row `wave` (ln_quant_row_kernel's arithmetic; the sums in the order of a wave's lanes).  The row and its
        // gains are here before this wave's first weights are requested: the loads return in order.  (The waves without a
        // row request theirs at once.)
        constexpr int NC = LN_K / 512;                              // chunks of 8 values per lane
        if (wave < g.M) {
            const int D = g.K;
            const float* const beta = sa.beta ? sa.beta : sa.gamma;
            const bool has_beta = sa.beta != nullptr;
            const uint16_t* const xp = (const uint16_t*)sa.h + (int64_t)wave * D;
            v4i rx[NC];
            v4f ga[NC][2], be[NC][2];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int j0 = min((c * 64 + lane) * 8, D - 8);     // beyond the row: its end again, taken out below
                rx[c] = *reinterpret_cast<const v4i*>(xp + j0);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    ga[c][e] = *reinterpret_cast<const v4f*>(sa.gamma + j0 + 4 * e);
                    be[c][e] = *reinterpret_cast<const v4f*>(beta + j0 + 4 * e);
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                asm volatile("" : "+v"(rx[c]));
#pragma unroll
                for (int e = 0; e < 2; ++e) { asm volatile("" : "+v"(ga[c][e])); asm volatile("" : "+v"(be[c][e])); }
            }
            fill();
            const float inv_d = 1.0f / (float)D;
            float v[NC][8], s = 0.0f, q = 0.0f, amax = 0.0f;
            bool in[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) in[c] = (c * 64 + lane) * 8 < D;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[c][e] = in[c] ? hp_to_f32<HDT>(((uint32_t)rx[c][e >> 1] >> (16 * (e & 1))) & 0xffffu) : 0.0f;
                    s += v[c][e];
                }
            const float mean = wave_reduce<false>(s) * inv_d;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const float mean_c = in[c] ? mean : 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) { v[c][e] -= mean_c; q = fmaf(v[c][e], v[c][e], q); }
            }
            const float rstd = __builtin_amdgcn_rsqf(wave_reduce<false>(q) * inv_d + sa.eps);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[c][e] = fmaf(v[c][e] * rstd, ga[c][e >> 2][e & 3], has_beta ? be[c][e >> 2][e & 3] : 0.0f);
                    amax = fmaxf(amax, in[c] ? fabsf(v[c][e]) : 0.0f);
                }
            amax = wave_reduce<true>(amax);
            constexpr bool F8 = ADT == HERO_F8E4M3;
            const float sc = amax == 0.0f ? 1.0f : __fdiv_rn(amax, F8 ? 448.0f : 127.0f), inv_sc = __builtin_amdgcn_rcpf(sc);
            if (lane == 0) srow[wave] = sc;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int j0 = (c * 64 + lane) * 8;
                if (j0 >= D) continue;
                uint32_t pk[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) pk[e] = ln_codes4(v[c] + 4 * e, sc, inv_sc, F8);
                *reinterpret_cast<v2i*>(scode + wave * LN_K + (((j0 >> 4) ^ (wave & 7)) << 4) + (j0 & 8)) = v2i{(int)pk[0], (int)pk[1]};
            }
        } else {
            fill();
        }
        // the codes are in LDS for every wave; no wait for the weights in flight (a __syncthreads() would do as well, but for
        // the compiler's own idea of what is outstanding)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
        fill();
    }

    ACC acc[CT][TM];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[c][i] = ACC{0, 0, 0, 0};
    // fragment s of unit row r = lane % 16: chunk 4 s + lane / 16
    const int fr = lane & 15, fg = lane >> 4;
    const int fo0 = fr * 128 + ((fg ^ (fr & 7)) << 4), fo1 = fr * 128 + (((4 + fg) ^ (fr & 7)) << 4);
    const int8_t* const base = smem + wave * RING;
    const int8_t* const arow = scode + (fr & 7) * LN_K;
    int slot = 0, left = total - 1;
    for (int st = 0; st < steps; ++st) {
        v4i a[TM][2];
        if constexpr (LN) {
            const int kc = (kbeg + (st + rot < steps ? st + rot : st + rot - steps) * KSTEP) >> 4;
            a[0][0] = *reinterpret_cast<const v4i*>(arow + ((kc + (fg ^ (fr & 7))) << 4));
            a[0][1] = *reinterpret_cast<const v4i*>(arow + ((kc + ((4 + fg) ^ (fr & 7))) << 4));
        }
        static_for<PER>([&](auto J) {
            constexpr int j = decltype(J)::value;
            unit_wait<NU - 1>(left);                                // this unit has landed
            __builtin_amdgcn_sched_barrier(0);
            const int8_t* u = base + slot * UNIT;
            v4i f[2] = {*reinterpret_cast<const v4i*>(u + fo0), *reinterpret_cast<const v4i*>(u + fo1)};
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]) :: "memory");       // read: its slot is free
            if (left >= NU) issue(std::integral_constant<int, (j + NU) % PER>{});
            if constexpr (j < AU) { a[j][0] = f[0]; a[j][1] = f[1]; }
            else {
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j - AU][i] = mfma_16<ADT>(f, a[i], acc[j - AU][i]);
            }
            slot = slot + 1 == NU ? 0 : slot + 1;
            --left;
        });
    }
    // the eight partial sums: [wave][tile][64 lanes] of four columns, added in the order of the waves
    __syncthreads();
    ACC* const part = reinterpret_cast<ACC*>(smem);
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < TM; ++i) part[(wave * (CT * TM) + c * TM + i) * 64 + lane] = acc[c][i];
    __syncthreads();
    if (!out) return;
    ACC sum = part[tid];
#pragma unroll
    for (int w = 1; w < SKINNY_WAVES; ++w) {
        const ACC p = part[w * SLOTS + tid];
#pragma unroll
        for (int t = 0; t < 4; ++t) sum[t] += p[t];
    }
    if (LN) rs = srow[m_e & 7];
    const bool has_rs = LN || g.a_row_scale != nullptr, gelu = sa.epi == HERO_EPI_DEQUANT_GELU || sa.epi == HERO_EPI_GELU_REQUANT;
    float y[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float v = (float)sum[t];
        if (HP) v = v + bs[t];
        else {
            if (has_rs) v = v * rs;
            v = fmaf(v, cs[t], bs[t]);
        }
        if (gelu) v = gelu_erf(v);
        if (sa.epi == HERO_EPI_GELU_REQUANT) v = v * __fdiv_rn(1.0f, os[t]);
        y[t] = v;
    }
    const int64_t o = (int64_t)m_e * g.ldc + n_e;
    if (sa.c_dt == HERO_I8 || sa.c_dt == HERO_F8E4M3) {
        *reinterpret_cast<uint32_t*>((int8_t*)g.C + o) = sa.c_dt == HERO_I8 ? quant4_sat(y[0], y[1], y[2], y[3]) : fp8x4_sat(y[0], y[1], y[2], y[3]);
        return;
    }
    const bool bf = sa.c_dt == HERO_BF16;
    if (sa.has_res) {
        const uint16_t* const rp = (const uint16_t*)g.residual + (int64_t)m_e * g.ldr + n_e;
        v2i r;
        if (sa.has_res == RES_ALIGNED) r = *reinterpret_cast<const v2i*>(rp);
        else r = v2i{(int)(rp[0] | (uint32_t)rp[1] << 16), (int)(rp[2] | (uint32_t)rp[3] << 16)};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t b = ((uint32_t)r[t >> 1] >> (16 * (t & 1))) & 0xffffu;
            y[t] += bf ? hp_to_f32<HERO_BF16>(b) : hp_to_f32<HERO_F16>(b);
        }
    }
    *reinterpret_cast<v2i*>((uint16_t*)g.C + o) =
        bf ? v2i{(int)pack2_hp<HERO_BF16>(y[0], y[1]), (int)pack2_hp<HERO_BF16>(y[2], y[3])}
           : v2i{(int)pack2_hp<HERO_F16>(y[0], y[1]), (int)pack2_hp<HERO_F16>(y[2], y[3])};
}

template <int ADT, int TM, int HDT>
hero_status launch_tiles(const SkinnyArgs& sa, hipStream_t st) {
    const int64_t nt = sa.g.N / 16;
    const int ct = nt <= 256 ? 1 : (nt <= 512 ? 2 : (nt <= 768 ? 3 : 4));
    SkinnyArgs a = sa;
    a.g.per_xcd = (int)(((nt + ct - 1) / ct + NUM_XCD - 1) / NUM_XCD);
    const dim3 grid((unsigned)(a.g.per_xcd * NUM_XCD)), block(SKINNY_WAVES * 64);
    switch (ct) {
    case 1: hipLaunchKernelGGL((skinny_gemm_kernel<ADT, 1, TM, HDT>), grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL((skinny_gemm_kernel<ADT, 2, TM, HDT>), grid, block, 0, st, a); break;
    case 3: hipLaunchKernelGGL((skinny_gemm_kernel<ADT, 3, TM, HDT>), grid, block, 0, st, a); break;
    default:                                                        // beyond 12288 columns: the LN form only (skinny_ok)
        if constexpr (HDT >= 0) hipLaunchKernelGGL((skinny_gemm_kernel<ADT, 4, TM, HDT>), grid, block, 0, st, a);
        else return HERO_ERR_UNSUPPORTED;
    }
    return hero_launch_status();
}

}  // namespace

namespace hero_gemm {

hero_status launch_skinny(const GemmArgs& g, hero_dtype adt, hero_epilogue epi, hero_dtype c_dt, hipStream_t st) {
    SkinnyArgs a;
    a.g = g; a.epi = epi; a.c_dt = c_dt;
    a.has_res = !g.residual ? RES_NONE : (g.ldr % 4 == 0 && ((uintptr_t)g.residual & 7) == 0 ? RES_ALIGNED : RES_ANY);
    a.h = nullptr; a.gamma = a.beta = nullptr; a.eps = 0.0f;
    const bool one = g.M <= 16;
    switch (adt) {
    case HERO_I8: return one ? launch_tiles<HERO_I8, 1, -1>(a, st) : launch_tiles<HERO_I8, 2, -1>(a, st);
    case HERO_F8E4M3: return one ? launch_tiles<HERO_F8E4M3, 1, -1>(a, st) : launch_tiles<HERO_F8E4M3, 2, -1>(a, st);
    case HERO_BF16: return one ? launch_tiles<HERO_BF16, 1, -1>(a, st) : launch_tiles<HERO_BF16, 2, -1>(a, st);
    case HERO_F16: return one ? launch_tiles<HERO_F16, 1, -1>(a, st) : launch_tiles<HERO_F16, 2, -1>(a, st);
    default: return HERO_ERR_UNSUPPORTED;
    }
}

}  // namespace hero_gemm

// LN^quant of the residual stream and the linear behind it in one launch (a decode step of up to eight sequences), or
// HERO_ERR_UNSUPPORTED: the caller then runs the two.  8-bit operands; not part of the C ABI.
hero_status hero_ln_gemm(const void* h, hero_dtype h_dt, const float* gamma, const float* beta, float eps,
                         const void* Wt, const float* w_scale, const float* bias, hero_epilogue epi, const float* out_col_scale,
                         void* C, hero_dtype c_dt, int64_t ldc, int64_t M, int64_t N, int64_t K, bool fp8, void* stream) {
    if (M > 8 || K > 4096 || !skinny_ok(M, N, K, K, K, 16384) || !gamma || !hero_aligned16(gamma) || !hero_aligned16(beta)) return HERO_ERR_UNSUPPORTED;
    SkinnyArgs a;
    GemmArgs& g = a.g;
    g.A = (const int8_t*)Wt; g.lda = 0; g.a_row_scale = nullptr;         // (no activation rows in memory)
    g.Bt = (const int8_t*)Wt; g.ldb = K; g.b_col_scale = w_scale; g.bias = bias; g.residual = nullptr; g.ldr = 0;
    g.out_col_scale = out_col_scale; g.C = C; g.ldc = ldc; g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.ntm = g.ntn = g.per_xcd = 0; g.ksplit = 1; g.kslabs = 0;
    a.epi = epi; a.c_dt = c_dt; a.has_res = RES_NONE; a.h = h; a.gamma = gamma; a.beta = beta; a.eps = eps;
    hipStream_t st = (hipStream_t)stream;
    if (fp8) return h_dt == HERO_BF16 ? launch_tiles<HERO_F8E4M3, 1, HERO_BF16>(a, st) : HERO_ERR_UNSUPPORTED;
    return h_dt == HERO_BF16 ? launch_tiles<HERO_I8, 1, HERO_BF16>(a, st) : launch_tiles<HERO_I8, 1, HERO_F16>(a, st);
}
