// The ring kernel (see the comment in front of it) and its forms; instantiated once per operand type, in gemm_ring_*.hip.
#pragma once
#include "gemm_common.h"

namespace hero_gemm {

// =====================================================================================
// Direct-to-LDS ring with K groups (small and middling problems).  One tile per workgroup; slabs of 128 bytes of K (one
// cache line of every row) go global -> LDS through a ring of NS stages, one barrier per slab.  KG groups of WM x WN waves
// share the tile: group k takes the k-th range of the slabs through a ring of its own (so KG rings are in flight), and the
// groups' accumulators are added through LDS, in the fixed order 0, 1, .., KG-1, before the epilogue.  PART: blockIdx.y
// picks a range of g.kslabs slabs (of 128 bytes) and the raw accumulators go to a plane of g.C.
// A slab row is 128 bytes, its eight 16-byte chunks stored at position c ^ ((row >> 1) & 7).  The LDS serves a 128-bit read in four turns of
// 16 lanes (lanes 0-3, 12-15 and 20-27 in the first); two rows share the 16 bank groups, so the eight rows of one parity in a
// turn have to differ in row / 2.  (By row & 7 they met in pairs: half of the cycles of every fragment read were conflicts; us, INT8 2000 x
// 1024 x 4096 15.2 -> 15.0, E4M3 3817 x 1024 x 4096 21.1 -> 20.7, BF16 602 x 4096 x 8192 61.1 -> 60.0, weights from memory 17.1 -> 16.9, 23.1 -> 22.7, 66.8 -> 66.0.)  A
// wave-level load still covers whole lines.
// =====================================================================================
template <int N, int NU>
__device__ __forceinline__ void ring_wait(int left) {                // at most min(left, N) slabs of NU loads outstanding
    if constexpr (N > 0) {
        if (left >= N) { __builtin_amdgcn_s_waitcnt(vmcnt_imm(N * NU)); return; }
        ring_wait<N - 1, NU>(left);
    } else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

template <int BM, int BN, int WM, int WN, int KG, int NS, int EPI, int CDT, int RDT, int ADT, bool PART, bool HALF>
__global__ __launch_bounds__(WM * WN * 64 * KG) void int8_gemm_ring_kernel(GemmArgs g) {
    using ACC = typename AccOf<ADT>::type;
    constexpr bool UNIT = ADT == HERO_BF16 || ADT == HERO_F16;      // 16-bit operands: no scales, y = acc + bias
    constexpr int SK = 2 * BK;                                      // bytes of K per slab
    constexpr int NWAVE = WM * WN, NT = NWAVE * 64;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int STAGE = (BM + BN) * SK, RING = NS * STAGE;
    constexpr int AU = BM / 8 / NWAVE, BU = BN / 8 / NWAVE, NU = AU + BU;   // 1 KB loads per wave and slab: 8 rows each
    static_assert(BM % (8 * NWAVE) == 0 && BN % (8 * NWAVE) == 0, "whole loads per wave");
    static_assert((NS - 1) * NU < 64, "vmcnt");
    static_assert(KG == 1 || (KG - 1) * BM * BN * 4 <= KG * RING, "accumulators of the other groups fit the rings");
    static_assert(KG * RING + 3 * BN * 4 <= 160 * 1024, "LDS budget");
    __shared__ __attribute__((aligned(1024))) int8_t smem[KG * RING + 3 * BN * 4];
    float* const sv = reinterpret_cast<float*>(smem + KG * RING);

    int m0, n0;
    if (!tile_origin<BM, BN>(g, m0, n0)) return;
    const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int tid = KG == 1 ? (int)threadIdx.x : (int)threadIdx.x % NT, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    // this group's slabs [k0, k0 + KT); every group passes the same number of barriers
    const int kall = HALF ? g.K / SK + 1 : g.K / SK, kbeg = PART ? (int)blockIdx.y * g.kslabs : 0, kwg = PART ? min(g.kslabs, kall - kbeg) : kall;
    const int kper = (kwg + KG - 1) / KG, k0 = kbeg + min(kg * kper, kwg), KT = min(kper, kbeg + kwg - k0);

    // HALF: K is an odd number of 64-byte pieces and ends in half a slab.  The group that owns it takes it FIRST, its lanes of the
    // upper half repeating the lower one (the memory behind a row's end is not the kernel's to read), and leaves out the matrix
    // instructions of that half.  A kernel of its own: tests for it in the other one cost 2-5 % of a small product.  Measured with
    // cold weights, us, register-staged tile -> here: INT8 1 x 4096 x 4160 20.5 -> 8, 64 x 4096 x 16448 with the K split 72 -> 24,
    // E4M3 64 x 4096 x 16448 100 -> 27, BF16 1000 x 4096 x 8256 bytes 92 -> 46.
    const int half = HALF && KT > 0 && k0 + KT == kall ? 1 : 0;
    const int8_t* ia = g.A + (int64_t)m0 * g.lda + (int64_t)(k0 - half) * SK;        // slab kt of this group: + kt * SK
    const int8_t* ib = g.Bt + (int64_t)n0 * g.ldb + (int64_t)(k0 - half) * SK;
    const int lrow = wave * 8 + (lane >> 3);                        // row of this lane in a load's 8 rows; the next load: + 8 * NWAVE
    auto lc = [&](int u) { return (uint32_t)(((lane & 7) ^ (((lrow + u * 8 * NWAVE) >> 1) & 7)) * 16); };    // this lane's chunk of load u
    uint32_t oa[AU], ob[BU];
#pragma unroll
    for (int u = 0; u < AU; ++u) oa[u] = (uint32_t)min(lrow + u * 8 * NWAVE, g.M - 1 - m0) * (uint32_t)g.lda + lc(u);
#pragma unroll
    for (int u = 0; u < BU; ++u) ob[u] = (uint32_t)min(lrow + u * 8 * NWAVE, g.N - 1 - n0) * (uint32_t)g.ldb + lc(u);
    const uint32_t ring = __builtin_amdgcn_readfirstlane(lds_offset(smem) + kg * RING);
    auto issue = [&](int kt, int stage) {
        const uint32_t dst = ring + stage * STAGE + wave * 1024;
        const int8_t* a = ia + (int64_t)kt * SK;
        const int8_t* b = ib + (int64_t)kt * SK;
#pragma unroll
        for (int u = 0; u < BU; ++u) dma16s(ob[u], b, dst + BM * SK + u * NWAVE * 1024);
#pragma unroll
        for (int u = 0; u < AU; ++u) dma16s(oa[u], a, dst + u * NWAVE * 1024);
    };
    // the epilogue's vectors are requested first (loads return in order: the waits below cover them) and wait in registers,
    // one entry per thread, until the main loop is over
    static_assert(NT * KG >= BN, "one entry per thread");
    constexpr bool VECS = !PART && EPI != HERO_EPI_RAW_I32;         // raw sums: the caller may have no vectors at all
    float vcs = 0.0f, vbs = 0.0f, vos = 1.0f;
    if (VECS && (int)threadIdx.x < BN) {
        const int n = min(n0 + (int)threadIdx.x, g.N - 1);
        if (!UNIT) vcs = g.b_col_scale[n];
        if (g.bias) vbs = g.bias[n];
        if (EPI == HERO_EPI_GELU_REQUANT) vos = g.out_col_scale[n];
    }
    float rsr[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
        rsr[i] = (VECS && !UNIT && g.a_row_scale) ? g.a_row_scale[min(m0 + wm * TM * 32 + i * 32 + (lane & 31), g.M - 1)] : 1.0f;
    if (HALF && half) {
#pragma unroll
        for (int u = 0; u < BU; ++u) dma16s(ob[u] - (lc(u) & (uint32_t)BK), ib + (int64_t)KT * SK, ring + wave * 1024 + BM * SK + u * NWAVE * 1024);
#pragma unroll
        for (int u = 0; u < AU; ++u) dma16s(oa[u] - (lc(u) & (uint32_t)BK), ia + (int64_t)KT * SK, ring + wave * 1024 + u * NWAVE * 1024);
    }
#pragma unroll
    for (int p = 0; p < NS; ++p) if (p >= half && p < KT) issue(p, p);

    const int hh = lane >> 5, ml = lane & 31;
    const int8_t* const base = smem + kg * RING;
    // row rr of the stage: rr & 15 == ml & 15, so the swizzle of k-step ks is one constant per lane
    const int8_t* const fa = base + (wm * TM * 32 + ml) * SK;
    const int8_t* const fb = base + BM * SK + (wn * TN * 32 + ml) * SK;
    int sw[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) sw[ks] = ((2 * ks + hh) ^ ((ml >> 1) & 7)) * 16;
    ACC acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // Half a slab (two k-steps) of fragments is read ahead: the reads of one half are under way during the matrix
    // instructions of the other, and the barrier that publishes the next slab sits between the two halves.  (Against reading
    // a whole slab behind its barrier: 602 x 4096 x 16384 BF16 143 -> 130 us, 3 x 4096 x 4096 INT8 6.5 -> 5.7.)
    v4i f0[2][TN + TM], f1[2][TN + TM];
    auto read = [&](int st, int half, v4i (&f)[2][TN + TM]) {
        const int so = st * STAGE;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int j = 0; j < TN; ++j) f[k][j] = *reinterpret_cast<const v4i*>(fb + so + j * 32 * SK + sw[2 * half + k]);
#pragma unroll
            for (int i = 0; i < TM; ++i) f[k][TN + i] = *reinterpret_cast<const v4i*>(fa + so + i * 32 * SK + sw[2 * half + k]);
        }
    };
    auto multiply = [&](const v4i (&f)[2][TN + TM]) {
        if constexpr (ADT == HERO_F8E4M3) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i][j] = mfma_wide_f8(f[0][j], f[1][j], f[0][TN + i], f[1][TN + i], acc[i][j]);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][j] = mfma_step<ADT>(f[k][j], f[k][TN + i], acc[i][j]);
        }
    };
    ring_wait<NS - 1, NU>(KT - 1);                                  // slab 0 is here
    __syncthreads();
    if (KT > 0) read(0, 0, f0);
    int stage = 0;
    for (int kt = 0; kt < kper; ++kt) {
        const int next = stage + 1 == NS ? 0 : stage + 1;
        if (kt < KT) { read(stage, 1, f1); multiply(f0); }
        ring_wait<NS - 2, NU>(KT - 2 - kt);                         // slab kt + 1 is here (mine) ...
        __syncthreads();                                            // ... and everybody's; slab kt has been read by every wave
        if (kt + 1 < KT) read(next, 0, f0);
        if (kt + NS < KT) issue(kt + NS, stage);
        if (kt < KT && kt >= half) multiply(f1);
        stage = next;
    }
    if (VECS && (int)threadIdx.x < BN) {
        sv[threadIdx.x] = vcs;
        sv[BN + threadIdx.x] = vbs;
        if (EPI == HERO_EPI_GELU_REQUANT) sv[2 * BN + threadIdx.x] = __fdiv_rn(1.0f, vos);      // 1 / S_a[j]
    }
    if constexpr (KG == 1 && VECS) __syncthreads();
    if constexpr (KG > 1) {
        using V4 = typename std::conditional<ADT == HERO_I8, v4i, v4f>::type;
        constexpr int NV = TM * TN * 4;
        __syncthreads();                                            // every group is done reading its ring; no load is outstanding
        if (kg > 0) {
            V4* const mine = reinterpret_cast<V4*>(smem + (kg - 1) * BM * BN * 4) + (wave * NV) * 64 + lane;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int ij = v >> 2, c = (v & 3) * 4;
                mine[v * 64] = V4{acc[ij / TN][ij % TN][c], acc[ij / TN][ij % TN][c + 1], acc[ij / TN][ij % TN][c + 2], acc[ij / TN][ij % TN][c + 3]};
            }
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int k = 0; k < KG - 1; ++k) {
            const V4* other = reinterpret_cast<const V4*>(smem + k * BM * BN * 4) + (wave * NV) * 64 + lane;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int ij = v >> 2, c = (v & 3) * 4;
                const V4 o = other[v * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[ij / TN][ij % TN][c + e] += o[e];
            }
        }
    }
    if constexpr (PART) {
        static_assert(EPI == HERO_EPI_RAW_I32, "a part writes raw accumulators");
        GemmArgs gp = g;
        gp.C = (int32_t*)g.C + (int64_t)blockIdx.y * g.M * g.ldc;
        epilogue_direct<BM, BN, WM, WN, EPI, CDT, RDT, false, false>(gp, acc, sv, rsr, m0, n0, tid);
    } else {
        epilogue_direct<BM, BN, WM, WN, EPI, CDT, RDT, false, UNIT>(g, acc, sv, rsr, m0, n0, tid);
    }
}

template <int ADT, int EPI, int CDT, int RDT, bool HALF>
hero_status launch_ring_slabs(const GemmArgs& g, RingForm f, hipStream_t st) {
#define HERO_RING(BM, BN, WM, WN, KG, NS) \
    return launch_grid(g, BM, BN, WM * WN * KG * 64, int8_gemm_ring_kernel<BM, BN, WM, WN, KG, NS, EPI, CDT, RDT, ADT, false, HALF>, st)
    switch (f) {
    case RING_32x32_K8: HERO_RING(32, 32, 1, 1, 8, 2);
    case RING_32x32_K4: HERO_RING(32, 32, 1, 1, 4, 4);
    case RING_32x64_K2: HERO_RING(32, 64, 1, 2, 2, 4);
    case RING_32x64_K4: HERO_RING(32, 64, 1, 2, 4, 3);
    case RING_64x32_K4: HERO_RING(64, 32, 2, 1, 4, 3);
    case RING_64x64_K2: HERO_RING(64, 64, 2, 2, 2, 3);
    case RING_64x64:    HERO_RING(64, 64, 2, 2, 1, 3);
    case RING_128x64_K2: HERO_RING(128, 64, 2, 2, 2, 3);
    case RING_128x64:   HERO_RING(128, 64, 2, 2, 1, 3);
    case RING_128x128:  HERO_RING(128, 128, 4, 2, 1, 4);
    default: return HERO_ERR_UNSUPPORTED;
    }
#undef HERO_RING
}

template <int ADT, bool HALF>
hero_status launch_ring_part_slabs(GemmArgs g, RingForm f, hipStream_t st) {
    auto go = [&](int BM, int BN, int threads, auto kernel) -> hero_status {
        g.ntm = (g.M + BM - 1) / BM;
        g.ntn = (g.N + BN - 1) / BN;
        g.per_xcd = (int)(((int64_t)g.ntm * g.ntn + NUM_XCD - 1) / NUM_XCD);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(g.per_xcd * NUM_XCD), (unsigned)g.ksplit), dim3(threads), 0, st, g);
        return hero_launch_status();
    };
    if (f == RING_64x64_K2) return go(64, 64, 512, int8_gemm_ring_kernel<64, 64, 2, 2, 2, 3, HERO_EPI_RAW_I32, HERO_I32, -1, ADT, true, HALF>);
    if (f == RING_128x64_K2) return go(128, 64, 512, int8_gemm_ring_kernel<128, 64, 2, 2, 2, 3, HERO_EPI_RAW_I32, HERO_I32, -1, ADT, true, HALF>);
    if constexpr (ADT == HERO_BF16 || ADT == HERO_F16)
        if (f == RING_128x256) return go(128, 256, 256, int8_gemm_ring_kernel<128, 256, 2, 2, 1, 3, HERO_EPI_RAW_I32, HERO_I32, -1, ADT, true, HALF>);
    return HERO_ERR_UNSUPPORTED;
}

// what gemm_ring_*.hip (K of whole slabs) and gemm_ring_*_half.hip instantiate for their operand type
#define HERO_RING_8BIT(ADT, CDT8, HALF) \
    template hero_status launch_ring_part_slabs<ADT, HALF>(GemmArgs, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_REQUANT, CDT8, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_GELU_REQUANT, CDT8, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT, HERO_BF16, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT, HERO_F16, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT, HERO_F16, HERO_F16, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<ADT, HERO_EPI_DEQUANT_GELU, HERO_F16, -1, HALF>(const GemmArgs&, RingForm, hipStream_t);
#define HERO_RING_16BIT(DT, HALF) \
    template hero_status launch_ring_part_slabs<DT, HALF>(GemmArgs, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<DT, HERO_EPI_DEQUANT, DT, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<DT, HERO_EPI_DEQUANT, DT, DT, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<DT, HERO_EPI_DEQUANT_GELU, DT, -1, HALF>(const GemmArgs&, RingForm, hipStream_t); \
    template hero_status launch_ring_slabs<DT, HERO_EPI_DEQUANT_GELU, DT, DT, HALF>(const GemmArgs&, RingForm, hipStream_t);

}  // namespace hero_gemm
