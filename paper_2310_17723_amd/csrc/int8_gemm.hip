// hero_int8_gemm: GeMM^quant, INT8 x INT8 -> INT32 on the gfx950 matrix cores with the
// dequantization / static-scale / bias / GELU / residual / requantization epilogue fused
// behind the accumulators (paper Sec. 2.1 GEMM convention and column-wise weight scales;
// Sec. 2.2.2 fused dequantization and the bare Round after folding; Sec. 2.2.3 GELU^quant).
//
// Both operands are K-contiguous ([M][K] activations, [N][K] weights), so every MFMA
// operand fragment is one 128-bit LDS read.  The WEIGHT fragment is the matrix instruction's first operand and the
// activation fragment its second, so an accumulator holds, for ONE output row per lane, groups of 4 consecutive
// columns: the per-row scale is one register.  The persistent kernel multiplies INT8 and 16-bit operands on 16 x 16 tiles
// (mfma16_step), whose weight rows are taken in an order that gives a lane 16 consecutive columns; the others use 32 x 32
// tiles (columns 8g + 4(l/32) + t of row l % 32) and exchange halves in the epilogue (v_permlane32_swap).
//
// The main loops; all but the skinny one's share one epilogue (gemm_common.h):
//   * int8_gemm_persistent_kernel (gemm_persistent.h; large problems): 256x256 block tile, 8 waves of 128x64,
//     slabs of 64 bytes of K copied global -> LDS directly (global_load_lds_dwordx4) through
//     two rings, of four slots for the activations and five for the weights; one workgroup per CU walks its tiles and the
//     rings run through the tile boundaries.  Tiles of 224, 192 and 160 rows and a second form, 128x128 with 4 waves of 64x64 and two workgroups per CU,
//     serve the sizes at which the large tile would leave CUs idle (128x128: twice the L2 -> LDS traffic per tile area).
//   * int8_gemm_dma_kernel: the same tile, one tile per workgroup (short K, huge strides).
//   * int8_gemm_ring_kernel (gemm_ring.h; small and middling problems): 32x32 .. 128x128 tiles, 128-byte slabs, K groups.
//   * skinny_gemm_kernel (gemm_skinny.hip; up to 32 rows): a stream of the weights.
//   * int8_gemm_kernel (rows too far apart for 32-bit offsets; a short K that ends in half a slab, over many rows): 128x128 /
//     64x64 tile staged through registers.
// The epilogue works in registers: every lane ends with a contiguous piece of one output row, written with 128-bit stores.
#include "gemm_common.h"
#include <atomic>
#include <cstdlib>

using namespace hero_gemm;

namespace {

// =====================================================================================
// Register-staged main loop (small / ragged problems).  BK-byte slabs, double-buffered in
// LDS with an 80-byte padded row stride, PD slabs in flight in registers.
// =====================================================================================
template <int BM, int BN, int WM, int WN, int PD, int MINW, int EPI, int CDT, int RDT, int ADT = HERO_I8>
__global__ __launch_bounds__(WM * WN * 64, MINW) void int8_gemm_kernel(GemmArgs g) {
    using ACC = typename AccOf<ADT>::type;
    constexpr int NT = WM * WN * 64;
    constexpr int CPR = BK / 16;                              // 16-byte chunks per slab row
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;      // 32x32 MFMA tiles per wave
    constexpr int A_UNITS = BM * CPR / NT, B_UNITS = BN * CPR / NT;
    static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
    static_assert(PD % 2 == 0, "prefetch distance must be even (LDS buffer parity is compile-time)");
    constexpr int POOL = 2 * (BM + BN) * LDS_LD;
    __shared__ __attribute__((aligned(16))) int8_t smem[POOL + 3 * BN * 4];
    int8_t* const sA0 = smem;                                 // [2][BM * LDS_LD]
    int8_t* const sB0 = sA0 + 2 * BM * LDS_LD;                // [2][BN * LDS_LD]
    float* const sv = reinterpret_cast<float*>(smem + POOL);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    int m0, n0;
    if (!tile_origin<BM, BN>(g, m0, n0)) return;
    const int KT = g.K / BK;

    constexpr bool UNIT = ADT == HERO_BF16 || ADT == HERO_F16;      // 16-bit operands: no scales, y = acc + bias
    stage_col_vectors<BN, NT, EPI, UNIT>(g, sv, n0, tid);
    float rsr[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
        rsr[i] = (EPI != HERO_EPI_RAW_I32 && g.a_row_scale) ? g.a_row_scale[min(m0 + wm * TM * 32 + i * 32 + (lane & 31), g.M - 1)] : 1.0f;

    // global -> register -> LDS staging.  Unit u of this thread is slab row idx / CPR,
    // 16-byte chunk idx % CPR.  PD slabs are in flight in registers ahead of the one in LDS.
    const int8_t* pa[A_UNITS];
    const int8_t* pb[B_UNITS];
#pragma unroll
    for (int u = 0; u < A_UNITS; ++u) {
        int idx = tid + u * NT, row = idx / CPR, ch = idx % CPR;
        pa[u] = g.A + (int64_t)min(m0 + row, g.M - 1) * g.lda + ch * 16;   // clamp: ragged M
    }
#pragma unroll
    for (int u = 0; u < B_UNITS; ++u) {
        int idx = tid + u * NT, row = idx / CPR, ch = idx % CPR;
        pb[u] = g.Bt + (int64_t)min(n0 + row, g.N - 1) * g.ldb + ch * 16;
    }
    const int lds_unit0 = (tid / CPR) * LDS_LD + (tid % CPR) * 16;                // + u * (NT / CPR) * LDS_LD
    v4i ra[PD][A_UNITS], rb[PD][B_UNITS];
    auto load_slab = [&](int kt, int p) {
#pragma unroll
        for (int u = 0; u < A_UNITS; ++u) ra[p][u] = *reinterpret_cast<const v4i*>(pa[u] + (int64_t)kt * BK);
#pragma unroll
        for (int u = 0; u < B_UNITS; ++u) rb[p][u] = *reinterpret_cast<const v4i*>(pb[u] + (int64_t)kt * BK);
    };
    auto store_slab = [&](int buf, int p) {
#pragma unroll
        for (int u = 0; u < A_UNITS; ++u)
            *reinterpret_cast<v4i*>(sA0 + buf * BM * LDS_LD + lds_unit0 + u * (NT / CPR) * LDS_LD) = ra[p][u];
#pragma unroll
        for (int u = 0; u < B_UNITS; ++u)
            *reinterpret_cast<v4i*>(sB0 + buf * BN * LDS_LD + lds_unit0 + u * (NT / CPR) * LDS_LD) = rb[p][u];
    };

    ACC acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // Every load is unconditional (slab indices are clamped to the last slab, whose
    // redundant copies are never read): with no branch between a load and its use the
    // compiler can wait for exactly the oldest register set and leave the younger ones
    // in flight.
    const int last = KT - 1;
    load_slab(0, 0);
    store_slab(0, 0);
#pragma unroll
    for (int p = 0; p < PD; ++p) load_slab(min(1 + p, last), p);  // slab s waits in register set (s-1) % PD
    __syncthreads();
    const int frag_a = (wm * TM * 32 + (lane & 31)) * LDS_LD + (lane >> 5) * 16;
    const int frag_b = (wn * TN * 32 + (lane & 31)) * LDS_LD + (lane >> 5) * 16;
    // One slab.  The body is written in the issue order wanted and pinned with scheduling
    // barriers: every MFMA is followed by at most one LDS read, one LDS write or one global
    // load.  A wave issues in order, and a burst of vector-memory instructions stalls it in
    // front of its next MFMA while the address unit drains; spread out, the memory
    // instructions issue in the shadow of the 32-cycle MFMAs.
    constexpr int NM = TM * TN, NFR = TM + TN, NW = A_UNITS + B_UNITS;
    auto iteration = [&](int kt, int buf, auto U) {
        constexpr int u = decltype(U)::value;
        const int8_t* sa = sA0 + buf * BM * LDS_LD + frag_a;
        const int8_t* sb = sB0 + buf * BN * LDS_LD + frag_b;
        int8_t* wa = sA0 + (buf ^ 1) * BM * LDS_LD + lds_unit0;
        int8_t* wb = sB0 + (buf ^ 1) * BN * LDS_LD + lds_unit0;
        const int64_t koff = (int64_t)min(kt + 1 + PD, last) * BK;
        v4i f0[NFR], f1[NFR];                                     // fragments of k-step 0 / 1: B tiles first, then A tiles
#pragma unroll
        for (int t = 0; t < NFR; ++t)
            f0[t] = *reinterpret_cast<const v4i*>((t < TN ? sb + t * 32 * LDS_LD : sa + (t - TN) * 32 * LDS_LD));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NM; ++n) {                             // k-step 0; memory instructions dealt round-robin
            const int jj = n / TM, ii = n % TM;
            acc[ii][jj] = mfma_step<ADT>(f0[jj], f0[TN + ii], acc[ii][jj]);
#pragma unroll
            for (int t = n; t < NFR; t += NM)
                f1[t] = *reinterpret_cast<const v4i*>((t < TN ? sb + t * 32 * LDS_LD : sa + (t - TN) * 32 * LDS_LD) + 32);
#pragma unroll
            for (int t = n; t < NW; t += NM) {                     // slab kt + 1 from register set u into LDS
                if (t < A_UNITS) *reinterpret_cast<v4i*>(wa + t * (NT / CPR) * LDS_LD) = ra[u][t];
                else *reinterpret_cast<v4i*>(wb + (t - A_UNITS) * (NT / CPR) * LDS_LD) = rb[u][t - A_UNITS];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < NM; ++n) {                             // k-step 1
            const int jj = n / TM, ii = n % TM;
            acc[ii][jj] = mfma_step<ADT>(f1[jj], f1[TN + ii], acc[ii][jj]);
#pragma unroll
            for (int t = n; t < NW; t += NM) {                     // slab kt + 1 + PD into the freed register set
                if (t < A_UNITS) ra[u][t] = *reinterpret_cast<const v4i*>(pa[t] + koff);
                else rb[u][t - A_UNITS] = *reinterpret_cast<const v4i*>(pb[t - A_UNITS] + koff);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    // PD iterations per trip, one per register set (the set index and the LDS buffer parity are compile-time);
    // the tail runs the first KT % PD of them
    int kt = 0;
    auto trip = [&](auto FULL) {
        static_for<PD>([&](auto U) {
            constexpr int u = decltype(U)::value;
            if (decltype(FULL)::value || kt + u < KT) iteration(kt + u, u & 1, U);
        });
    };
    for (; kt + PD <= KT; kt += PD) trip(std::true_type{});
    if (kt < KT) trip(std::false_type{});
    epilogue_direct<BM, BN, WM, WN, EPI, CDT, RDT, false, UNIT>(g, acc, sv, rsr, m0, n0, tid);
}

// =====================================================================================
// Direct-to-LDS main loop (large problems).  A wave-level global_load_lds_dwordx4 writes
// 1 KB of consecutive LDS, so slab rows are 64 bytes, unpadded, and the four 16-byte chunks
// of row r are stored at position c ^ ((r >> 2) & 3): the 128-bit fragment reads of 16
// consecutive rows then fall into 16 different 16-byte bank groups.
// =====================================================================================
template <int BM, int BN, int WM, int WN, int NS, int MINW, int EPI, int CDT, int RDT>
__global__ __launch_bounds__(WM * WN * 64, MINW) void int8_gemm_dma_kernel(GemmArgs g) {
    constexpr int NT = WM * WN * 64, NWAVE = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE = A_BYTES + B_BYTES;
    constexpr int A_UNITS = A_BYTES / 16 / NT, B_UNITS = B_BYTES / 16 / NT, NW = A_UNITS + B_UNITS;
    constexpr int NM = TM * TN, NFR = TM + TN;
    static_assert(NS >= 3, "ring needs at least three stages");
    static_assert(NW <= NM && NFR <= NM, "interleave plan needs one slot per memory instruction");
    constexpr int POOL = NS * STAGE;
    __shared__ __attribute__((aligned(1024))) int8_t smem[POOL + 3 * BN * 4];
    float* const sv = reinterpret_cast<float*>(smem + POOL);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    int m0, n0;
    if (!tile_origin<BM, BN>(g, m0, n0)) return;
    const int KT = g.K / BK, last = KT - 1;

    stage_col_vectors<BN, NT, EPI>(g, sv, n0, tid);
    float rsr[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
        rsr[i] = (EPI != HERO_EPI_RAW_I32 && g.a_row_scale) ? g.a_row_scale[min(m0 + wm * TM * 32 + i * 32 + (lane & 31), g.M - 1)] : 1.0f;

    // loader: unit u of wave w fills LDS granules [(u * NWAVE + w) * 64, +64) of the A (or B)
    // part of a stage; lane l owns granule q = that + l  ->  row q / 4, stored chunk q % 4,
    // which holds global chunk (q % 4) ^ ((row >> 2) & 3).
    const int8_t* pa[A_UNITS];
    const int8_t* pb[B_UNITS];
#pragma unroll
    for (int u = 0; u < A_UNITS; ++u) {
        const int q = (u * NWAVE + wave) * 64 + lane, row = q >> 2, c = (q & 3) ^ ((row >> 2) & 3);
        pa[u] = g.A + (int64_t)min(m0 + row, g.M - 1) * g.lda + c * 16;
    }
#pragma unroll
    for (int u = 0; u < B_UNITS; ++u) {
        const int q = (u * NWAVE + wave) * 64 + lane, row = q >> 2, c = (q & 3) ^ ((row >> 2) & 3);
        pb[u] = g.Bt + (int64_t)min(n0 + row, g.N - 1) * g.ldb + c * 16;
    }
    const uint32_t wbase = __builtin_amdgcn_readfirstlane(lds_offset(smem) + wave * 1024);   // + stage * STAGE + unit offset
    auto issue = [&](int n, int kt, int stage) {        // the n-th direct load of slab kt
        const int64_t koff = (int64_t)min(kt, last) * BK;
        if (n < A_UNITS) dma16(pa[n] + koff, wbase + stage * STAGE + n * NWAVE * 1024);
        else dma16(pb[n - A_UNITS] + koff, wbase + stage * STAGE + A_BYTES + (n - A_UNITS) * NWAVE * 1024);
    };
    // fragment offsets inside a stage (row rr, k-step ks, half hh): rr*64 + ((2ks+hh) ^ ((rr>>2)&3))*16
    const int hh = lane >> 5, ml = lane & 31;
    int fo[2][NFR];
#pragma unroll
    for (int t = 0; t < NFR; ++t) {
        const int rr = (t < TN ? wn * TN * 32 + t * 32 : wm * TM * 32 + (t - TN) * 32) + ml;
        const int base = (t < TN ? A_BYTES : 0) + rr * 64;
        fo[0][t] = base + (((0 + hh) ^ ((rr >> 2) & 3)) << 4);
        fo[1][t] = base + (((2 + hh) ^ ((rr >> 2) & 3)) << 4);
    }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // prologue: slabs 0 .. NS-2 in flight, slab 0 landed, its k-step-0 fragments in registers
#pragma unroll
    for (int s0 = 0; s0 < NS - 1; ++s0)
#pragma unroll
        for (int n = 0; n < NW; ++n) issue(n, s0, s0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * NW));
    __syncthreads();
    v4i f0[NFR], f1[NFR];
#pragma unroll
    for (int t = 0; t < NFR; ++t) f0[t] = *reinterpret_cast<const v4i*>(smem + fo[0][t]);

    // One slab per iteration; the barrier sits in the MIDDLE: k-step 0 runs on fragments read
    // during the previous slab, the barrier then makes slab kt+1 visible, and k-step 1 runs
    // while the first fragments of slab kt+1 and the direct loads of slab kt+NS-1 are issued,
    // one memory instruction per MFMA.
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
        const int8_t* st = smem + stage * STAGE;
        const int nstage = stage + 1 == NS ? 0 : stage + 1;      // slab kt + 1
        const int pstage = stage == 0 ? NS - 1 : stage - 1;      // slab kt - 1 == slab kt + NS - 1
        const int8_t* stn = smem + nstage * STAGE;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NM; ++n) {                             // k-step 0
            const int jj = n / TM, ii = n % TM;
            acc[ii][jj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0[jj], f0[TN + ii], acc[ii][jj], 0, 0, 0);
            if (n < NFR) f1[n] = *reinterpret_cast<const v4i*>(st + fo[1][n]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 3) * NW));     // slab kt + 1 has landed (mine)
        __syncthreads();                                           // ... and everybody's
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NM; ++n) {                             // k-step 1
            const int jj = n / TM, ii = n % TM;
            acc[ii][jj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1[jj], f1[TN + ii], acc[ii][jj], 0, 0, 0);
            if (n < NFR) f0[n] = *reinterpret_cast<const v4i*>(stn + fo[0][n]);
            if (n < NW) issue(n, kt + NS - 1, pstage);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = nstage;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                      // the redundant tail loads
    __syncthreads();
    epilogue_direct<BM, BN, WM, WN, EPI, CDT, RDT>(g, acc, sv, rsr, m0, n0, tid);
}

// Split-K for skinny M with a long K (M <= 128, 64 slabs of 128 bytes or more): the weights are streamed once, and too few
// tiles exist to do that from every CU.  Pass 1: the ring kernel with a second grid dimension over K ranges writes raw
// partial sums, one [M][ldp] plane per range, into the caller's scratch, as many ranges as give every CU one
// workgroup of 64 columns.  Pass 2 (splitk_reduce_kernel) adds the planes and runs the epilogue: its arithmetic is the one-pass
// kernels', in the same order; INT8 sums are exact, fp32 ones (E4M3, 16 bits) are added in the fixed order of the ranges.
// The kernel boundary is the only synchronisation (device-wide fences inside one
// kernel measured 4x slower than no split at all).  Measured with cold weights, one pass -> split: INT8 64 x 4096 x 16384
// 23.6 -> 19.7 us, 3 rows 19.7 -> 17.6, 100 rows 26.3 -> 24.1; BF16 64 rows 44.4 -> 35.6, 3 rows 36.2 -> 30.5; with
// K = 4096 the second launch costs more than the split gives.
struct SplitK { int ksplit, kslabs; int64_t ldp; size_t bytes; int rows = 0; };      // ranges, 128-byte slabs of each, the planes' stride and size; rows: below
inline SplitK split_ranges(int64_t M, int64_t N, int64_t kb, int64_t want) {
    const int64_t slabs = (kb + 2 * BK - 1) / (2 * BK), kslabs = (slabs + want - 1) / want;
    SplitK p;
    p.kslabs = (int)kslabs;
    p.ksplit = (int)((slabs + kslabs - 1) / kslabs);                   // every range non-empty
    p.ldp = (N + 3) & ~(int64_t)3;
    p.bytes = (size_t)p.ksplit * M * p.ldp * 4;
    return p;
}
inline SplitK splitk_plan(int64_t M, int64_t N, int64_t kb) {           // kb: bytes of K
    const int64_t b = M <= 64 ? 64 : 128, tiles = (N + b - 1) / b, want = 256 / ((N + 63) / 64 > 0 ? (N + 63) / 64 : 1);
    if (M <= 0 || N <= 0 || M > 128 || kb % BK != 0 || tiles > 128 || kb < 128 * BK || N * kb < (4 << 20) /* launch-bound anyway */ || want < 2)
        return SplitK{1, 0, 0, 0};
    return split_ranges(M, N, kb, want < 16 ? want : 16);
}

// A middling product with a very long K (FC2 of a prompt chunk, 16 KB and more): one round of 128 x 128 tiles leaves a part of the CUs
// without work, and so do few large ones.  Tiles of `rows` x 256 of the persistent kernel, or 16-bit ones of 128 x 256 of the ring's (rows 0; 256 slabs or
// more), times as many K ranges as fill the 256 CUs, where an estimate in us says so: a range's share of a 256 x 256 tile's time over the
// whole K, 9.4 ns per byte of it, plus the planes' way out and back, 0.9 us per MB, and 6 us for the second launch and the ranges' start, against 128 x 128
// tiles in one round (0.43) or two (0.8), or large ones.  Measured, N = 4096, K = 16384, best form in one pass -> split: BF16 M = 150 67 -> 52 us (ring), 300 83 -> 69
// (ring), 602 128 -> 93 (ring 99), 700 124 -> 108, 900 135 -> 131, 1100 236 -> 153, 1400 231 -> 180;  INT8 602 68 -> 63, 1100 119 -> 93, 1400
// 118 -> 112, but 900 74 -> 83;  a quarter of that K: nowhere ahead (INT8 602 20.8 -> 38, BF16 1100 64 -> 60).
inline SplitK mid_split_plan(int64_t M, int64_t N, int64_t kb, bool hp) {
    SplitK best{1, 0, 0, 0};
    if (M <= 128 || N <= 0 || kb % BK != 0) return best;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t t128 = tiles(128, 256);
    const double whole = 9.4e-3 * (double)kb;
    double t = 0;
    auto offer = [&](int rows, double part) {
        const int64_t n = tiles(rows ? rows : 128, 256);
        if (n > 128) return;
        SplitK p = split_ranges(M, N, kb, 256 / n < 8 ? 256 / n : 8);
        p.rows = rows;
        if (p.ksplit < 2 || (rows && kb / (2 * BK) - (int64_t)(p.ksplit - 1) * p.kslabs < 3)) return;      // (the rings: six slabs or more)
        const double e = part * whole * (double)p.kslabs * (2 * BK) / (double)kb + 0.9e-6 * (double)p.bytes + 6;
        if (best.ksplit == 1 || e < t) { t = e; best = p; }
    };
    const bool ring = hp && kb >= 256 * 2 * BK && t128 * 3 <= 256;
    if (ring) offer(0, 0.66);
    const RingForm form = ring_form(M, N, kb, HERO_EPI_DEQUANT);
    if ((form != RING_NONE && form != RING_128x128) || kb < 128 * 2 * BK || kb % (2 * BK) != 0) return best;
    const int64_t small = tiles(128, 128);
    auto rounds = [&](int64_t bm) { return (double)((tiles(bm, 256) + 255) / 256); };
    double one = small <= 256 ? 0.43 : small <= 512 ? 0.8 : 1e9;
    for (const double o : {rounds(256), 0.91 * rounds(224), 0.80 * rounds(192), 0.71 * rounds(160)}) one = o < one ? o : one;
    offer(160, 0.70);
    offer(192, 0.82);
    offer(224, 0.95);
    offer(256, 1.00);
    if (!ring && t > 0.93 * one * whole) return SplitK{1, 0, 0, 0};
    return best;
}
inline SplitK split_plan(bool hp, int64_t M, int64_t N, int64_t kb) { return M <= 128 ? splitk_plan(M, N, kb) : mid_split_plan(M, N, kb, hp); }

// Pass 2 of split-K: one thread per 4 consecutive columns of a row.
// Integer sums are exact in any order; fp32 partial sums (E4M3 and 16-bit operands) are added in the fixed order of the
// ranges, so a result does not vary from run to run.
template <int EPI, int CDT, int RDT, int ADT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs g, const int32_t* part, int64_t ldp) {
    constexpr bool UNIT = ADT == HERO_BF16 || ADT == HERO_F16;
    using V4 = typename std::conditional<ADT == HERO_I8, v4i, v4f>::type;
    constexpr int ES = ElemSize<CDT>::v;
    const int nq = (g.N + 3) / 4;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)g.M * nq) return;
    const int m = (int)(idx / nq), n = (int)(idx % nq) * 4;
    V4 a = {0, 0, 0, 0};
#pragma unroll 4
    for (int ks = 0; ks < g.ksplit; ++ks) {
        const V4 p = *reinterpret_cast<const V4*>(part + ((int64_t)ks * g.M + m) * ldp + n);
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] += p[t];
    }
    const int nv = min(4, g.N - n);                                    // valid columns
    uint32_t e[4];                                                     // outputs as element bit patterns
    if constexpr (EPI == HERO_EPI_RAW_I32) {
#pragma unroll
        for (int t = 0; t < 4; ++t) e[t] = (uint32_t)a[t];
    } else {
        const float rs = g.a_row_scale ? g.a_row_scale[m] : 1.0f;
        float y[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int nn = min(n + t, g.N - 1);
            float v = (float)a[t];
            if (UNIT) v = v + (g.bias ? g.bias[nn] : 0.0f);
            else {
                if (g.a_row_scale) v = v * rs;
                v = fmaf(v, g.b_col_scale[nn], g.bias ? g.bias[nn] : 0.0f);
            }
            if (EPI == HERO_EPI_DEQUANT_GELU || EPI == HERO_EPI_GELU_REQUANT) v = gelu_erf(v);
            if (EPI == HERO_EPI_GELU_REQUANT) v = v * __fdiv_rn(1.0f, g.out_col_scale[nn]);
            if (RDT >= 0 && t < nv) v += hp_to_f32<RDT>(((const uint16_t*)g.residual)[(int64_t)m * g.ldr + n + t]);
            y[t] = v;
        }
        if constexpr (ES == 1) {
            const uint32_t w = CDT == HERO_F8E4M3 ? fp8x4_sat(y[0], y[1], y[2], y[3]) : quant4_sat(y[0], y[1], y[2], y[3]);
#pragma unroll
            for (int t = 0; t < 4; ++t) e[t] = (w >> (8 * t)) & 0xffu;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) e[t] = f32_to_hp<CDT>(y[t]);
        }
    }
    int8_t* cp = (int8_t*)g.C + ((int64_t)m * g.ldc + n) * ES;
    if (nv == 4) {
        if constexpr (ES == 1) *reinterpret_cast<uint32_t*>(cp) = e[0] | (e[1] << 8) | (e[2] << 16) | (e[3] << 24);
        else if constexpr (ES == 2) *reinterpret_cast<v2i*>(cp) = v2i{(int)(e[0] | (e[1] << 16)), (int)(e[2] | (e[3] << 16))};
        else *reinterpret_cast<v4i*>(cp) = v4i{(int)e[0], (int)e[1], (int)e[2], (int)e[3]};
    } else {
        for (int t = 0; t < nv; ++t) {
            if (ES == 1) cp[t] = (int8_t)e[t];
            else if (ES == 2) reinterpret_cast<uint16_t*>(cp)[t] = (uint16_t)e[t];
            else reinterpret_cast<uint32_t*>(cp)[t] = e[t];
        }
    }
}

// Runs the split where it is one (true: *status is the outcome).
template <int EPI, int CDT, int RDT, int ADT>
bool launch_splitk(const GemmArgs& g, void* ws, size_t ws_bytes, hipStream_t st, hero_status* status) {
    if (!ws || !ring_ok(g.lda, g.ldb)) return false;
    const SplitK p = ADT == HERO_F8E4M3 ? splitk_plan(g.M, g.N, g.K) : split_plan(ADT != HERO_I8, g.M, g.N, g.K);
    if (p.ksplit <= 1 || ws_bytes < p.bytes) return false;
    const RingForm f = g.M > 128 ? RING_128x256 : (g.M <= 64 ? RING_64x64_K2 : RING_128x64_K2);     // skinny: 64 columns, one workgroup per CU
    GemmArgs g1 = g;                                                   // pass 1: raw partial planes in the scratch
    g1.a_row_scale = nullptr; g1.b_col_scale = nullptr; g1.bias = nullptr; g1.residual = nullptr; g1.out_col_scale = nullptr;
    g1.C = ws; g1.ldc = p.ldp;
    g1.kslabs = p.kslabs; g1.ksplit = p.ksplit;
    if constexpr (ADT != HERO_F8E4M3) if (p.rows) *status = launch_persistent_part<ADT>(g1, p.rows, st);
    if (!p.rows) *status = launch_ring_part<ADT>(g1, f, st);
    if (*status != HERO_OK) return true;
    GemmArgs g2 = g;                                                   // pass 2: sum of the planes + epilogue
    g2.ksplit = p.ksplit;
    const int64_t threads = (int64_t)g.M * ((g.N + 3) / 4);
    hipLaunchKernelGGL((splitk_reduce_kernel<EPI, CDT, RDT, ADT>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                       g2, (const int32_t*)ws, p.ldp);
    *status = hero_launch_status();
    return true;
}

// Tile choice (choose() below): the ring kernel where ring_form (gemm_common.h) has a form (everything small, and a short K), the
// persistent kernels beyond (persistent_choice).
// Only regions of at most 8 MB are requested: a BERT-large weight matrix (1-4 MB) waits in the memory-side cache until
// its kernel starts and saves it 5-7 us of simultaneous first misses; GPT's 16-64 MB matrices are pushed out again by
// the activations written in between (FC1 alone writes 268 MB), and requesting them cost 0.3 % of the layer.
inline void set_prefetch(GemmArgs& g, const void* prefetch, size_t prefetch_bytes) {
    if (prefetch && prefetch_bytes >= 128 && prefetch_bytes <= ((size_t)8 << 20) && ((uintptr_t)prefetch & 3) == 0) {
        g.pf = (const int8_t*)prefetch;
        g.pf_lines = (int)(prefetch_bytes / 128);                // whole lines inside the region
    }
}

// What runs a product.  The codes of the kernels are those of the test hooks (include/hero_debug.h).
enum Kernel { K_REG128 = 0, K_DMA256 = 1, K_RING = 2, K_REG64 = 3, K_SKINNY = 4, K_PERS256 = 7, K_PERS128 = 8 };
struct Choice { Kernel kernel; RingForm form; int rows = 256; };       // rows: K_PERS256's tile is rows x 256

// The persistent kernel's tile: 256, 224, 192 or 160 rows (E4M3, whose matrix instructions take 32 rows of a wave's half: 256 or 192) by 256
// columns, one workgroup per CU, or 128 x 128, two per CU.  A CU is handed ceil(tiles / 256) of them; what one takes, in parts of a
// 256 x 256 tile's time, is below: more than its share of the area (0.875, 0.75, 0.625, 0.25), since the weights' 256 rows are loaded for every
// height and a 128 x 128 tile loads twice as much for its area, which a long K does not hide.  Measured over 265 products (INT8, E4M3, BF16;
// 300 .. 14000 rows, K of 768 .. 16384) the choice is 0.4 % from the best of the five on average and was ahead of choosing between 256 and 128
// by 4 % on average, by 40 % at most.  Single ones are further off: behind a short K how full the last round is counts too (8-bit operands, 16-bit result, 160 x 256 /
// 128 x 128: 4184 x 4096 x 1024 26.7 / 30.5, but 4931 rows 31.0 / 28.7, 6616 x 3072 x 1024 29.9 / 27.7; 8187 x 3072 x 768 is best in 224 rows, 28.5 / 33.4).  us, 256 / 224 / 192 / 160 / 128: INT8 GELU^quant 602 x 16384 x 4096 52.1 / 49.6 / 47.5 / 43.3 / 58.5, 16-bit result
// 2500 x 4096 x 16384 160 / 152 / 141 / 134 / 174, REQUANT 3817 x 3072 x 1024 17.0 / 16.7 / 15.0 / 23.4 / 15.9, 9000 x 1024 x 4096 43.8 / 41.4 / 36.3 / 35.4 / 46.0, 14000 x
// 3072 x 1024 47.0 / 44.1 / 49.4 / 53.4 / 47.6;  BF16 602 x 16384 x 4096 94 / 90 / 83 / 76 / 109, 9000 x 1024 x 4096 81 / 78 / 67 / 65 / 88.
// (256 rows by the loop with branches.  Where launch_persistent_tile takes the one without, they take 0.94 to 0.98 of that, which is not weighed here.)
inline Choice persistent_choice(hero_dtype adt, hero_epilogue epi, int64_t M, int64_t N, int64_t kb) {
    const bool f8 = adt == HERO_F8E4M3, gelu = epi == HERO_EPI_DEQUANT_GELU || epi == HERO_EPI_GELU_REQUANT;
    auto rounds = [&](int64_t bm, int64_t bn) { return (double)((((M + bm - 1) / bm) * ((N + bn - 1) / bn) + 255) / 256); };
    const double n256 = rounds(256, 256);
    // Behind a K of 8 KB and more 128 x 128 tiles are nearer to their share of the area while all are resident at once (512 at most) and an eighth of the CUs have one only.
    // us, weights and activations from memory, 160 x 256 / 128 x 128: BF16 5943 x 768 x 8192 126 / 111, 301 x 12288 x 4096 70.8 / 61.5, 4637 x 1024 x 4096 71.0 / 60.5, INT8
    // 1313 x 4096 x 16384 123 / 112;  GPT layer, 1300 and 1700 tokens, M3 396 / 387, 442 / 436.  Not with more of them (480: 630 tokens, M0 327 / 332; 512: 2040 tokens, M2 600 / 619), nor with four or eight rows of
    // tiles, the last one more than half full (BF16 431 x 12288 x 4096 70.0 / 68.5, 480 rows 71.8 / 74.4, 505 rows 69.9 / 79.2, 1000 x 8192 x 4096 69.0 / 75.2;
    // layer, 505 tokens, M0 293 / 314): consecutive workgroups then differ in their row of tiles in steps of four, which is slower by a fifth than with six.
    const int64_t m128 = (M + 127) / 128;
    const bool resident = m128 * ((N + 127) / 128) <= 448 && !(m128 % 4 == 0 && m128 <= 8 && (M - 1) % 128 >= 64);
    const double small = rounds(128, 128) * (kb <= 2048 ? (gelu ? 0.27 : 0.30) : f8 && n256 > 1 ? 0.325 : kb < 8192 || resident ? 0.34 : 0.36);
    // (E4M3 behind a long K: from the second large round on 128 x 128 keeps what it is ahead of 256 x 256 in, 192 rows serve the rest.  us, 256 / 192 / 128:
    // REQUANT 3000 x 12288 x 4096 143 / 124 / 140, 1900 x 12288 x 4096 94 / 83 / 102, 10500 x 1024 x 4096 43.7 / 39.6 / 45.7.)
    if (f8 && kb > 2048 && n256 > 1 && small < n256) return {K_PERS128, RING_NONE};
    Choice c = {K_PERS256, RING_NONE};
    double t = n256;
    auto offer = [&](int rows, double part) { const double o = rounds(rows, 256) * part; if (o < t) { t = o; c.rows = rows; } };
    offer(192, f8 ? 0.87 : 0.80);
    if (!f8) {
        offer(224, 0.91);
        if (kb >= 6 * BK) offer(160, 0.71);                            // (its weights' ring of six slots)
    }
    if (small < t) return {K_PERS128, RING_NONE};
    return c;
}

// kb, lda, ldb in bytes.  tile: -1 chooses, otherwise the code a test hook
// forces (a forced kernel that cannot run the shape gives way to its closest relative).
inline Choice choose(hero_dtype adt, hero_epilogue epi, int64_t M, int64_t N, int64_t kb, int64_t lda, int64_t ldb, int tile = -1) {
    const bool i8 = adt == HERO_I8, ring = ring_ok(lda, ldb);
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256), t128 = ((M + 127) / 128) * ((N + 127) / 128);
    // persistent kernels: K long enough that the slab ring never runs more than one tile ahead, whole pairs of slabs, 32-bit
    // per-lane offsets
    const bool pers_ok = ring && kb >= 4 * BK && kb % (2 * BK) == 0 && t128 <= 0x7fffff00LL;
    const RingForm form = ring ? ring_form(M, N, kb, epi) : RING_NONE;
    const Choice small = {ring ? K_RING : (M <= 64 || t128 < 192 ? K_REG64 : K_REG128), form == RING_NONE ? RING_128x64 : form};
    if (tile >= 0) {
        const int rows = tile == 10 ? 224 : tile == 11 || (tile == 12 && kb < 6 * BK) ? 192 : tile == 12 ? 160 : 256;
        if (rows < 256) tile = K_PERS256;
        if (tile == K_PERS256 || tile == K_PERS128) {
            if (pers_ok) return {tile == K_PERS128 ? K_PERS128 : K_PERS256, RING_NONE, rows};
            if (i8) return {tile == K_PERS128 ? K_REG128 : K_DMA256, RING_NONE};
            return small;
        }
        if (tile == K_RING || (tile == 0 && (adt == HERO_BF16 || adt == HERO_F16))) return small;
        return {tile == K_DMA256 ? K_DMA256 : K_REG128, RING_NONE};
    }
    if (epi != HERO_EPI_RAW_I32 && skinny_ok(M, N, kb, lda, ldb)) return {K_SKINNY, RING_NONE};
    if (form != RING_NONE) return small;
    if (pers_ok) return persistent_choice(adt, epi, M, N, kb);
    // K that ends in half a slab: the one-tile-per-workgroup 256 x 256 kernel (INT8) once its grid fills the chip, else 128 x 128
    // tiles, through the ring from 32 slabs on.  us, ring / registers: 2048 x 4096 x 4160 INT8 52.1 / 54.8, E4M3 51.0 / 55.7,
    // x 8256 bytes of BF16 90.4 / 99.7, but 2048 x 4096 x 2112 INT8 32.6 / 31.1, 8192 x 1024 x 1056 BF16 28.5 / 26.8.
    if (i8 && t256 >= 160) return {K_DMA256, RING_NONE};
    if (ring && kb >= 32 * 2 * BK) return {K_RING, RING_128x128};
    return {M <= 64 || t128 < 192 ? K_REG64 : K_REG128, RING_NONE};
}

// May K be split over workgroups, given scratch?  Few rows stream the weights without that, unless K is long (in bytes beyond 8192, all
// that N <= 512 asks) and the columns few: a workgroup of the weight-streaming kernel takes the whole K of its columns and of all
// rows, so that its time grows with both and most CUs are idle, while the split's grows with the slabs of a range, more so where an XCD
// is handed more of its workgroups than it has CUs.  Two estimates in us, fitted to 800 products of 576 .. 4096 columns, and the split
// where they are close (within 7 %, up to 2048 columns): 1 % behind the better one on average, nowhere 5 % behind the split.  us, split / whole K: INT8 16 x 512 x 16384 10.5 / 11.6, 32 x 640 x 16384 11.1 / 15.5, 32 x 1024 x 16384 12.0 / 15.2, 8
// rows 11.2 / 10.4, 24 x 2048 x 24576 16.8 / 20.2, 32 x 1280 x 16384 (36 workgroups on an XCD) 15.2 / 14.3;  BF16 32 x 1024 x 8192 11.8 / 14.9.
inline bool may_split(Kernel kernel, int64_t M, int64_t N, int64_t kb) {
    if (kernel != K_SKINNY) return true;
    if (kb <= 8192) return false;
    if (N <= 512) return true;
    const SplitK p = splitk_plan(M, N, kb);
    const double k = (double)kb / 1024, on_xcd = (double)((N + 511) / 512) * p.ksplit;
    const double whole = 4.7 + k * (0.28 + 0.009 * (double)M + (M > 16 ? 0.06 : 0.0)) + (double)N * k * 4e-5;
    const double split = 7.0 + 0.35e-3 * (double)N + 0.09 * p.ksplit + p.kslabs * (on_xcd > 32 ? 0.46 : 0.29) + (on_xcd > 32 ? 1.8 : 0.0);
    return split < (N <= 2048 ? 1.07 : 1.0) * whole;
}

template <int ADT, int EPI, int CDT, int RDT>
hero_status launch_choice(const GemmArgs& g, Choice c, hipStream_t st) {
    switch (c.kernel) {
    case K_PERS256: return launch_persistent_tile<ADT, EPI, CDT, RDT>(g, c.rows, st);
    case K_PERS128: return launch_persistent_tile<ADT, EPI, CDT, RDT>(g, 128, st);
    case K_DMA256:
        if constexpr (ADT == HERO_I8) return launch_grid(g, 256, 256, 512, int8_gemm_dma_kernel<256, 256, 2, 4, 4, 2, EPI, CDT, RDT>, st);
        else return HERO_ERR_UNSUPPORTED;
    case K_RING: return launch_ring<ADT, EPI, CDT, RDT>(g, c.form, st);
    case K_SKINNY: return launch_skinny(g, (hero_dtype)ADT, (hero_epilogue)EPI, (hero_dtype)CDT, st);
    case K_REG64: return launch_grid(g, 64, 64, 256, int8_gemm_kernel<64, 64, 2, 2, 2, 2, EPI, CDT, RDT, ADT>, st);
    default: return launch_grid(g, 128, 128, 256, int8_gemm_kernel<128, 128, 2, 2, 2, 2, EPI, CDT, RDT, ADT>, st);
    }
}

template <int ADT, int EPI, int CDT, int RDT>
hero_status launch_epi(const GemmArgs& g, void* ws, size_t ws_bytes, hipStream_t st, int tile) {
    hero_status split;
    const Choice c = choose((hero_dtype)ADT, (hero_epilogue)EPI, g.M, g.N, g.K, g.lda, g.ldb, tile);
    if (tile < 0 && may_split(c.kernel, g.M, g.N, g.K) && launch_splitk<EPI, CDT, RDT, ADT>(g, ws, ws_bytes, st, &split)) return split;
    return launch_choice<ADT, EPI, CDT, RDT>(g, c, st);
}

}  // namespace

// 16-bit operands (bf16 or fp16: the 16-bit side of a switched module).  Same kernels, same choice as for INT8 operands, K
// counted in bytes.
namespace {
template <int DT>
hero_status launch_hp(const GemmArgs& g, bool gelu, void* ws, size_t wsb, hipStream_t st, int tile) {
    if (gelu) return g.residual ? launch_epi<DT, HERO_EPI_DEQUANT_GELU, DT, DT>(g, ws, wsb, st, tile) : launch_epi<DT, HERO_EPI_DEQUANT_GELU, DT, -1>(g, ws, wsb, st, tile);
    return g.residual ? launch_epi<DT, HERO_EPI_DEQUANT, DT, DT>(g, ws, wsb, st, tile) : launch_epi<DT, HERO_EPI_DEQUANT, DT, -1>(g, ws, wsb, st, tile);
}

hero_status run_hp_gemm(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                        const float* bias, const void* residual, int64_t ldr, int gelu,
                        void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, hero_dtype dt, void* ws, size_t ws_bytes, void* stream, int tile) {
    if (dt != HERO_BF16 && dt != HERO_F16) return HERO_ERR_UNSUPPORTED;
    if (M < 0 || N < 0 || K <= 0 || M > 0x7fffffffLL || N > 0x7fffffffLL || K > 0x3fffffffLL) return HERO_ERR_SHAPE;
    if (K % 32 != 0) return HERO_ERR_UNSUPPORTED;
    if (lda < K || ldb < K || ldc < N || (residual && ldr < N)) return HERO_ERR_SHAPE;
    if (M == 0 || N == 0) return HERO_OK;
    if (!A || !Wt || !C) return HERO_ERR_NULL;
    if (lda % 8 || ldb % 8 || ldc % 4 || !hero_aligned16(A) || !hero_aligned16(Wt) || !hero_aligned16(C)) return HERO_ERR_ALIGN;
    GemmArgs g;
    g.A = (const int8_t*)A; g.lda = lda * 2; g.a_row_scale = nullptr; g.Bt = (const int8_t*)Wt; g.ldb = ldb * 2;
    g.b_col_scale = nullptr; g.bias = bias; g.residual = residual; g.ldr = ldr; g.out_col_scale = nullptr;
    g.C = C; g.ldc = ldc; g.M = (int)M; g.N = (int)N; g.K = (int)(K * 2);
    g.ksplit = 1; g.kslabs = 0;
    // more than 2^23 rows: the persistent kernels only (INT8 operands end there altogether)
    if (M > 65535 * 128LL) {
        const Kernel k = choose(dt, gelu ? HERO_EPI_DEQUANT_GELU : HERO_EPI_DEQUANT, M, N, g.K, g.lda, g.ldb, tile).kernel;
        if (k != K_PERS256 && k != K_PERS128) return HERO_ERR_UNSUPPORTED;
    }
    return dt == HERO_BF16 ? launch_hp<HERO_BF16>(g, gelu != 0, ws, ws_bytes, (hipStream_t)stream, tile)
                           : launch_hp<HERO_F16>(g, gelu != 0, ws, ws_bytes, (hipStream_t)stream, tile);
}
}  // namespace

size_t hero_hp_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) { return split_plan(true, M, N, 2 * K).bytes; }

// hero_hp_gemm with scratch for the K split (hero_layer_fwd).  Not part of the C ABI.
hero_status hero_hp_gemm_ws(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                            const float* bias, const void* residual, int64_t ldr, int gelu,
                            void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, hero_dtype dt,
                            void* workspace, size_t workspace_bytes, void* stream) {
    return run_hp_gemm(A, lda, Wt, ldb, bias, residual, ldr, gelu, C, ldc, M, N, K, dt, workspace, workspace_bytes, stream, -1);
}

extern "C" hero_status hero_hp_gemm(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                                    const float* bias, const void* residual, int64_t ldr, int gelu,
                                    void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, hero_dtype dt, void* stream) {
    return run_hp_gemm(A, lda, Wt, ldb, bias, residual, ldr, gelu, C, ldc, M, N, K, dt, nullptr, 0, stream, -1);
}

extern "C" hero_status hero_bf16_gemm(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                                      const float* bias, const void* residual, int64_t ldr, int gelu,
                                      void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, void* stream) {
    return run_hp_gemm(A, lda, Wt, ldb, bias, residual, ldr, gelu, C, ldc, M, N, K, HERO_BF16, nullptr, 0, stream, -1);
}

// Test and tuning hook (include/hero_debug.h).
extern "C" hero_status hero_hp_gemm_tile(const void* A, int64_t lda, const void* Wt, int64_t ldb,
                                         const float* bias, const void* residual, int64_t ldr, int gelu,
                                         void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, hero_dtype dt, void* stream, int tile) {
    if (tile != 0 && tile != 7 && tile != 8 && (tile < 10 || tile > 12)) return HERO_ERR_UNSUPPORTED;
    return run_hp_gemm(A, lda, Wt, ldb, bias, residual, ldr, gelu, C, ldc, M, N, K, dt, nullptr, 0, stream, tile);
}

// Test hook (include/hero_debug.h): what the product entry points run without scratch.
extern "C" int hero_gemm_kernel(hero_dtype dt, hero_epilogue epi, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
    const int64_t es = dt == HERO_BF16 || dt == HERO_F16 ? 2 : 1;
    const Choice c = choose(dt, epi, M, N, K * es, lda * es, ldb * es);
    return c.kernel == K_RING ? 16 + (int)c.form : (int)c.kernel;
}

// The FP8 variant: the same kernels and the same choice with E4M3 operands.
static hero_status run_fp8_gemm(const void* A, int64_t lda, const float* a_row_scale,
                                const void* Bt, int64_t ldb, const float* b_col_scale,
                                const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                hero_epilogue epi, const float* out_col_scale,
                                void* C, hero_dtype c_dt, int64_t ldc,
                                int64_t M, int64_t N, int64_t K, void* workspace, size_t workspace_bytes, void* stream, int tile,
                                const void* prefetch = nullptr, size_t prefetch_bytes = 0) {
    if (M < 0 || N < 0 || K <= 0) return HERO_ERR_SHAPE;
    if (M > 0x7fffffffLL || N > 0x7fffffffLL || K > 0x7fffffffLL) return HERO_ERR_SHAPE;
    if (K % KMULT != 0) return HERO_ERR_UNSUPPORTED;
    if (lda < K || ldb < K || ldc < N) return HERO_ERR_SHAPE;
    if (M == 0 || N == 0) return HERO_OK;
    if (!A || !Bt || !C || !b_col_scale) return HERO_ERR_NULL;
    if (epi == HERO_EPI_GELU_REQUANT && !out_col_scale) return HERO_ERR_NULL;
    const bool c16 = c_dt == HERO_F16 || c_dt == HERO_BF16;
    switch (epi) {
    case HERO_EPI_DEQUANT: case HERO_EPI_DEQUANT_GELU: if (!c16) return HERO_ERR_UNSUPPORTED; break;
    case HERO_EPI_REQUANT: case HERO_EPI_GELU_REQUANT: if (c_dt != HERO_F8E4M3) return HERO_ERR_UNSUPPORTED; break;
    default: return HERO_ERR_UNSUPPORTED;
    }
    if (residual) {
        if (epi != HERO_EPI_DEQUANT || res_dt != c_dt) return HERO_ERR_UNSUPPORTED;
        if (ldr < N) return HERO_ERR_SHAPE;
        if (ldr % 4 != 0 || !hero_aligned16(residual)) return HERO_ERR_ALIGN;
    }
    if (lda % 16 != 0 || ldb % 16 != 0 || ldc % 4 != 0) return HERO_ERR_ALIGN;
    if (!hero_aligned16(A) || !hero_aligned16(Bt) || !hero_aligned16(C)) return HERO_ERR_ALIGN;
    GemmArgs g;
    g.A = (const int8_t*)A; g.lda = lda; g.a_row_scale = a_row_scale; g.Bt = (const int8_t*)Bt; g.ldb = ldb; g.b_col_scale = b_col_scale;
    g.bias = bias; g.residual = residual; g.ldr = ldr; g.out_col_scale = out_col_scale;
    g.C = C; g.ldc = ldc; g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.ksplit = 1; g.kslabs = 0;
    set_prefetch(g, prefetch, prefetch_bytes);
    hipStream_t st = (hipStream_t)stream;
    switch (epi) {
    case HERO_EPI_REQUANT: return launch_epi<HERO_F8E4M3, HERO_EPI_REQUANT, HERO_F8E4M3, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_GELU_REQUANT: return launch_epi<HERO_F8E4M3, HERO_EPI_GELU_REQUANT, HERO_F8E4M3, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_DEQUANT_GELU:
        return c_dt == HERO_BF16 ? launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1>(g, workspace, workspace_bytes, st, tile)
                                 : launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT_GELU, HERO_F16, -1>(g, workspace, workspace_bytes, st, tile);
    default:
        if (!residual)
            return c_dt == HERO_BF16 ? launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_BF16, -1>(g, workspace, workspace_bytes, st, tile)
                                     : launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_F16, -1>(g, workspace, workspace_bytes, st, tile);
        return c_dt == HERO_BF16 ? launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16>(g, workspace, workspace_bytes, st, tile)
                                 : launch_epi<HERO_F8E4M3, HERO_EPI_DEQUANT, HERO_F16, HERO_F16>(g, workspace, workspace_bytes, st, tile);
    }
}

size_t hero_fp8_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) { return splitk_plan(M, N, K).bytes; }

// The size callers have always been asked for, and by which hero_int8_gemm_static refuses: two tiles of 64 x 64 (M > 64: 128 x
// 128) per CU, at most 16 ranges.  An upper bound of the plan's own; 0 where the plan does not split.
extern "C" size_t hero_int8_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const SplitK p = splitk_plan(M, N, K);
    if (p.ksplit <= 1) return 0;
    const int64_t b = M <= 64 ? 64 : 128, tiles = (N + b - 1) / b, kt = K / BK, want = (512 + tiles - 1) / tiles;
    const int64_t kslabs = (kt + (want < 16 ? want : 16) - 1) / (want < 16 ? want : 16);
    return (size_t)((kt + kslabs - 1) / kslabs) * M * p.ldp * 4;
}

// What hero_layer_fwd offers an INT8 linear: as much as any split of it takes.
size_t hero_int8_gemm_split_bytes(int64_t M, int64_t N, int64_t K) { return M <= 128 ? hero_int8_gemm_workspace_bytes(M, N, K) : split_plan(false, M, N, K).bytes; }

// What hero_layer_fwd insists on for an INT8 linear (contiguous rows): nothing where no plane is written.
size_t hero_int8_gemm_scratch_needed(int64_t M, int64_t N, int64_t K) {
    return may_split(choose(HERO_I8, HERO_EPI_DEQUANT, M, N, K, K, K).kernel, M, N, K) ? hero_int8_gemm_workspace_bytes(M, N, K) : 0;
}

extern "C" hero_status hero_int8_gemm(const int8_t* A, int64_t lda, const float* a_row_scale,
                                      const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                      const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                      hero_epilogue epi, const float* out_col_scale,
                                      void* C, hero_dtype c_dt, int64_t ldc,
                                      int64_t M, int64_t N, int64_t K, void* stream) {
    return hero_int8_gemm_ws(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                             C, c_dt, ldc, M, N, K, nullptr, 0, stream);
}

namespace {
// Everything that can be checked about a GeMM^quant request, before anything is launched.  *noop: nothing to do.
hero_status check_gemm_args(const int8_t* A, int64_t lda, const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                            const void* residual, hero_dtype res_dt, int64_t ldr, hero_epilogue epi,
                            const float* out_col_scale, void* C, hero_dtype c_dt, int64_t ldc,
                            int64_t M, int64_t N, int64_t K, bool* noop) {
    *noop = false;
    if (M < 0 || N < 0 || K <= 0) return HERO_ERR_SHAPE;
    if (M >= (1LL << 23) || N > 0x7fffffffLL || K > 0x7fffffffLL) return HERO_ERR_SHAPE;
    if (K % KMULT != 0) return HERO_ERR_UNSUPPORTED;
    if (lda < K || ldb < K || ldc < N) return HERO_ERR_SHAPE;
    if (M == 0 || N == 0) { *noop = true; return HERO_OK; }
    if (!A || !Bt || !C) return HERO_ERR_NULL;
    if (epi != HERO_EPI_RAW_I32 && !b_col_scale) return HERO_ERR_NULL;
    if (epi == HERO_EPI_GELU_REQUANT && !out_col_scale) return HERO_ERR_NULL;
    const bool c16 = c_dt == HERO_F16 || c_dt == HERO_BF16;
    switch (epi) {
    case HERO_EPI_RAW_I32: if (c_dt != HERO_I32) return HERO_ERR_UNSUPPORTED; break;
    case HERO_EPI_DEQUANT: case HERO_EPI_DEQUANT_GELU: if (!c16) return HERO_ERR_UNSUPPORTED; break;
    case HERO_EPI_REQUANT: case HERO_EPI_GELU_REQUANT: if (c_dt != HERO_I8) return HERO_ERR_UNSUPPORTED; break;
    default: return HERO_ERR_UNSUPPORTED;
    }
    if (residual) {
        if (epi != HERO_EPI_DEQUANT) return HERO_ERR_UNSUPPORTED;
        if (res_dt != HERO_F16 && res_dt != HERO_BF16) return HERO_ERR_UNSUPPORTED;
        if (res_dt != c_dt) return HERO_ERR_UNSUPPORTED;
        if (ldr < N) return HERO_ERR_SHAPE;
        if (ldr % 4 != 0 || !hero_aligned16(residual)) return HERO_ERR_ALIGN;
    }
    if (lda % 16 != 0 || ldb % 16 != 0 || ldc % 4 != 0) return HERO_ERR_ALIGN;
    if (!hero_aligned16(A) || !hero_aligned16(Bt) || !hero_aligned16(C)) return HERO_ERR_ALIGN;
    return HERO_OK;
}
}  // namespace

static hero_status run_int8_gemm(const int8_t* A, int64_t lda, const float* a_row_scale,
                                 const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                 const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                 hero_epilogue epi, const float* out_col_scale,
                                 void* C, hero_dtype c_dt, int64_t ldc,
                                 int64_t M, int64_t N, int64_t K,
                                 void* workspace, size_t workspace_bytes, void* stream, int tile,
                                 const void* prefetch = nullptr, size_t prefetch_bytes = 0) {
    if (workspace && ((uintptr_t)workspace & 255)) return HERO_ERR_WORKSPACE;
    bool noop = false;
    const hero_status cs = check_gemm_args(A, lda, Bt, ldb, b_col_scale, residual, res_dt, ldr, epi, out_col_scale,
                                           C, c_dt, ldc, M, N, K, &noop);
    if (cs != HERO_OK || noop) return cs;

    GemmArgs g;
    g.A = A; g.lda = lda; g.a_row_scale = a_row_scale; g.Bt = Bt; g.ldb = ldb; g.b_col_scale = b_col_scale;
    g.bias = bias; g.residual = residual; g.ldr = ldr; g.out_col_scale = out_col_scale;
    g.C = C; g.ldc = ldc; g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.ksplit = 1; g.kslabs = 0;
    set_prefetch(g, prefetch, prefetch_bytes);
    hipStream_t st = (hipStream_t)stream;
    switch (epi) {
    case HERO_EPI_RAW_I32: return launch_epi<HERO_I8, HERO_EPI_RAW_I32, HERO_I32, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_REQUANT: return launch_epi<HERO_I8, HERO_EPI_REQUANT, HERO_I8, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_GELU_REQUANT: return launch_epi<HERO_I8, HERO_EPI_GELU_REQUANT, HERO_I8, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_DEQUANT_GELU:
        return c_dt == HERO_BF16 ? launch_epi<HERO_I8, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1>(g, workspace, workspace_bytes, st, tile)
                                 : launch_epi<HERO_I8, HERO_EPI_DEQUANT_GELU, HERO_F16, -1>(g, workspace, workspace_bytes, st, tile);
    case HERO_EPI_DEQUANT:
        if (!residual)
            return c_dt == HERO_BF16 ? launch_epi<HERO_I8, HERO_EPI_DEQUANT, HERO_BF16, -1>(g, workspace, workspace_bytes, st, tile)
                                     : launch_epi<HERO_I8, HERO_EPI_DEQUANT, HERO_F16, -1>(g, workspace, workspace_bytes, st, tile);
        if (c_dt == HERO_BF16) return launch_epi<HERO_I8, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16>(g, workspace, workspace_bytes, st, tile);
        return launch_epi<HERO_I8, HERO_EPI_DEQUANT, HERO_F16, HERO_F16>(g, workspace, workspace_bytes, st, tile);
    default: return HERO_ERR_UNSUPPORTED;
    }
}

// hero_int8_gemm_ws for a caller that knows what its chain reads next (hero_layer_fwd: the next module's weights):
// the large-problem kernels request that memory while they run, the others ignore the hint.  The workspace is scratch for any split
// (hero_int8_gemm_split_bytes).  Not part of the C ABI.
hero_status hero_int8_gemm_prefetching(const int8_t* A, int64_t lda, const float* a_row_scale,
                                       const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                       const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                       hero_epilogue epi, const float* out_col_scale,
                                       void* C, hero_dtype c_dt, int64_t ldc,
                                       int64_t M, int64_t N, int64_t K,
                                       void* workspace, size_t workspace_bytes, void* stream,
                                       const void* prefetch, size_t prefetch_bytes) {
    return run_int8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                         C, c_dt, ldc, M, N, K, workspace, workspace_bytes, stream, -1, prefetch, prefetch_bytes);
}

hero_status hero_fp8_gemm_prefetching(const void* A, int64_t lda, const float* a_row_scale,
                                      const void* Bt, int64_t ldb, const float* b_col_scale,
                                      const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                      hero_epilogue epi, const float* out_col_scale,
                                      void* C, hero_dtype c_dt, int64_t ldc,
                                      int64_t M, int64_t N, int64_t K,
                                      void* workspace, size_t workspace_bytes, void* stream,
                                      const void* prefetch, size_t prefetch_bytes) {
    return run_fp8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                        C, c_dt, ldc, M, N, K, workspace, workspace_bytes, stream, -1, prefetch, prefetch_bytes);
}

extern "C" hero_status hero_int8_gemm_ws(const int8_t* A, int64_t lda, const float* a_row_scale,
                                         const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                         const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                         hero_epilogue epi, const float* out_col_scale,
                                         void* C, hero_dtype c_dt, int64_t ldc,
                                         int64_t M, int64_t N, int64_t K,
                                         void* workspace, size_t workspace_bytes, void* stream) {
    // a buffer for a product whose size query is 0 need not be scratch (the split of a middling one is hero_layer_fwd's, which asks for it)
    if (hero_int8_gemm_workspace_bytes(M, N, K) == 0) workspace_bytes = 0;
    return run_int8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                         C, c_dt, ldc, M, N, K, workspace, workspace_bytes, stream, -1);
}

extern "C" hero_status hero_fp8_gemm(const void* A, int64_t lda, const float* a_row_scale,
                                     const void* Bt, int64_t ldb, const float* b_col_scale,
                                     const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                     hero_epilogue epi, const float* out_col_scale,
                                     void* C, hero_dtype c_dt, int64_t ldc,
                                     int64_t M, int64_t N, int64_t K, void* stream) {
    return run_fp8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                        C, c_dt, ldc, M, N, K, nullptr, 0, stream, -1);
}

// Test and tuning hooks (include/hero_debug.h): the same calls with the kernel choice forced.
extern "C" hero_status hero_int8_gemm_tile(const int8_t* A, int64_t lda, const float* a_row_scale,
                                           const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                           const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                           hero_epilogue epi, const float* out_col_scale,
                                           void* C, hero_dtype c_dt, int64_t ldc,
                                           int64_t M, int64_t N, int64_t K, void* stream, int tile) {
    if (tile == 9) tile = K_PERS256;                                   // (a former kernel's code, still accepted)
    if (tile != 0 && tile != 1 && tile != 2 && tile != 7 && tile != 8 && (tile < 10 || tile > 12)) return HERO_ERR_UNSUPPORTED;
    return run_int8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                         C, c_dt, ldc, M, N, K, nullptr, 0, stream, tile);
}

extern "C" hero_status hero_fp8_gemm_tile(const void* A, int64_t lda, const float* a_row_scale,
                                          const void* Bt, int64_t ldb, const float* b_col_scale,
                                          const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                          hero_epilogue epi, const float* out_col_scale,
                                          void* C, hero_dtype c_dt, int64_t ldc,
                                          int64_t M, int64_t N, int64_t K, void* stream, int tile) {
    if (tile != 0 && tile != 7 && tile != 8 && tile != 11) return HERO_ERR_UNSUPPORTED;
    return run_fp8_gemm(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                        C, c_dt, ldc, M, N, K, nullptr, 0, stream, tile);
}

// ---- hero_int8_gemm_static: the split-K scratch lives in the library ---------------------------------------
// For callers that cannot allocate (HIP graph capture, serving loops, harnesses that forbid hipMalloc).  The
// array below exists once per GPU the library is loaded on, until the process ends.  Its name is a host-side
// stand-in, not a device address: the address is asked for once per device (hipGetSymbolAddress with that
// device current) and only that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[HERO_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::atomic<void*> g_scratch_ptr[MAX_DEVICES];                         // per device; racing first calls store the same value

hero_status static_scratch_ptr(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return HERO_ERR_LAUNCH;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return HERO_ERR_LAUNCH;
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return HERO_OK;
}
}  // namespace

extern "C" hero_status hero_int8_gemm_static(const int8_t* A, int64_t lda, const float* a_row_scale,
                                             const int8_t* Bt, int64_t ldb, const float* b_col_scale,
                                             const float* bias, const void* residual, hero_dtype res_dt, int64_t ldr,
                                             hero_epilogue epi, const float* out_col_scale,
                                             void* C, hero_dtype c_dt, int64_t ldc,
                                             int64_t M, int64_t N, int64_t K, void* stream) {
    bool noop = false;
    const hero_status cs = check_gemm_args(A, lda, Bt, ldb, b_col_scale, residual, res_dt, ldr, epi, out_col_scale,
                                           C, c_dt, ldc, M, N, K, &noop);
    if (cs != HERO_OK || noop) return cs;
    const size_t need = hero_int8_gemm_workspace_bytes(M, N, K);
    if (need > (size_t)HERO_STATIC_SCRATCH_BYTES) return HERO_ERR_WORKSPACE;   // beyond the built-in scratch
    void* ws = nullptr;
    if (need) {
        const hero_status ss = static_scratch_ptr(&ws);
        if (ss != HERO_OK) return ss;
    }
    return hero_int8_gemm_ws(A, lda, a_row_scale, Bt, ldb, b_col_scale, bias, residual, res_dt, ldr, epi, out_col_scale,
                             C, c_dt, ldc, M, N, K, ws, need, stream);
}
