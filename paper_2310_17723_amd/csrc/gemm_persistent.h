// int8_gemm_persistent_kernel: large problems of every operand type (instantiated per type in gemm_persistent_*.hip).
#pragma once
#include "gemm_common.h"

namespace hero_gemm {

// =====================================================================================
// Persistent variant of the direct-to-LDS kernel (large problems): one
// workgroup per CU walks a strided list of tiles, and the slab ring runs straight through
// the tile boundaries, so the first slabs of the next tile (and its per-column / per-row
// epilogue vectors, fetched by the same direct loads into a double-buffered LDS area) are
// already resident when the epilogue of the current tile ends.  Slab addresses are a wave-uniform tile base in SGPRs
// plus a per-lane 32-bit offset, so advancing along K is scalar arithmetic.
// A and B have rings of their own, of four and five slots (144 KB), and take turns: B's pair of slabs goes out in even iterations and has
// three to arrive in, A's in odd ones and has two.  One ring of four slots for both sent 64 KB at once and then waited for the last of them: a
// pair of slabs took the time from its first load to its last one's arrival, 2500 to 3200 clocks against 2048 of matrix instructions.  us,
// one ring -> two: BERT-large layer 32 x 512 300 both ways, in M1 404 -> 385, GPT prefill 8 x 2048 3387 -> 3263;  INT8 16384 x 12288 x 4096 641 -> 610 (2.70 POP/s), 16384 x 4096 x 16384 888 -> 815, 16384 x 1024 x 4096 55.3 -> 53.2, 16384 x
// 3072 x 1024 49.8 -> 48.8;  BF16 8192 x 4096 x 4096 208 -> 199;  E4M3 8192 x 4096 x 4096 111 -> 102.  (Both operands in the same iteration: -7 %.)
// The clock under matrix load is set by power, and 16 x 16 instructions multiply more per watt than 32 x 32 ones; their lanes also
// write 16 (32) consecutive bytes next to their neighbours'.  us, 32 x 32 -> 16 x 16 tiles: INT8 16384 x 12288 x 4096 694 -> 642
// (2.57 POP/s), 8192 x 4096 x 16384 451 -> 411, 8192 x 4096 x 4096 120 -> 111, 16384 x 4096 x 1024 REQUANT 71.5 -> 69.2, GELU^quant 16384 x
// 16384 x 4096 1013 -> 921, 16-bit result 8192 x 4096 x 1024 53.9 -> 40.4;  BF16 8192 x 4096 x 4096 234 -> 208, 16384 x 4096 x 1024 156 -> 128.
// (A kernel of its own for GELU^quant behind a short K, its epilogue spread over the next tile's main loop, fell behind with
// that: 16384 x 4096 x 1024 91 -> 84 us, 16-bit result 152 -> 98.5, 2500 rows 27.9 -> 20.5.)
// =====================================================================================
// How many of a wave's direct loads may be out when the barrier of an iteration publishes the next slab: those issued behind the ones
// that bring it.  la, lb: loads of a pair of A, B.  Times are iterations before this one (0); a ring of n slots is given a pair for the slabs
// n - 1 and n ahead in odd iterations (n even) or even ones (n odd), A before B.  Behind an odd iteration the pair's first slab is
// needed, whose loads alternate with the second one's, so that the very last may be out as well.
constexpr int pair_loads_behind(bool odd, int na, int nb, int la, int lb) {
    const int first = odd ? 2 : 1;
    const int last = 2 * (first - nb) + 1 > 2 * (first - na) ? 2 * (first - nb) + 1 : 2 * (first - na);     // 2 * time (+ 1: B)
    int c = odd ? 1 : 0;
    for (int t = -6; t < 0; ++t) {
        const bool t_odd = ((t + (odd ? 1 : 0)) & 1) != 0;
        if ((nb % 2 == 0) == t_odd && 2 * t + 1 > last) c += lb;
        if ((na % 2 == 0) == t_odd && 2 * t > last) c += la;
    }
    return c;
}

template <int BM, int BN, int WM, int WN, int NSA, int NSB, int EPI, int CDT, int RDT, int ADT = HERO_I8, bool PART = false, bool STEADY = false>
__global__ __launch_bounds__(WM * WN * 64, 2) void int8_gemm_persistent_kernel(GemmArgs g) {
    constexpr bool UNIT = ADT == HERO_BF16 || ADT == HERO_F16;      // 16-bit operands: no scales, y = acc + bias
    constexpr bool WIDE = ADT == HERO_F8E4M3;                       // 32 x 32 tiles; INT8 and 16 bits: 16 x 16 (mfma16_step)
    using ACC = typename std::conditional<WIDE, v16f, typename Acc4Of<ADT>::type>::type;
    constexpr int NT = WM * WN * 64, NWAVE = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;            // (32 x 32 tiles)
    constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK;
    // 1 KB loads per wave and slab: 16 rows each; with BM no multiple of 128 the last one is for the first A_LAST waves only
    constexpr int A_UNITS = (BM / 16 + NWAVE - 1) / NWAVE, A_LAST = BM / 16 - (A_UNITS - 1) * NWAVE, B_UNITS = BN / 16 / NWAVE;
    constexpr bool A_EVEN = A_LAST == NWAVE;
    constexpr bool ONE = NSA == NSB && BM == BN;                    // rings alike, filled in the same iterations: B's stream and offsets are A's too
    constexpr int NM = TM * TN, NFR = TM + TN;
    static_assert(NSA >= 4 && NSA <= 6 && NSB >= 4 && NSB <= 6 && BM % (16 * WM) == 0 && BN % (16 * NWAVE) == 0 && (!WIDE || (NFR <= 2 * NM && BM % (32 * WM) == 0)), "rings / interleave plan");
    static_assert(!PART || (EPI == HERO_EPI_RAW_I32 && !WIDE), "a part writes raw accumulators");
    constexpr int A_RING = NSA * A_BYTES, B_RING = NSB * B_BYTES, RING = A_RING + B_RING;
    constexpr int SVF = 4 * BN;                                  // floats per vector set: column scale, bias, S_a, row scale
    static_assert(BM <= BN, "the row-scale vector shares the column vectors' length");
    constexpr int PF_OFF = RING + 2 * SVF * 4;                   // 256 bytes per wave where the prefetch requests land (never read)
    static_assert(PF_OFF + NWAVE * 256 <= 160 * 1024, "LDS budget");
    __shared__ __attribute__((aligned(1024))) int8_t smem[PF_OFF + NWAVE * 256];
    float* const sv0 = reinterpret_cast<float*>(smem + RING);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int xcd = blockIdx.x % NUM_XCD, slot = blockIdx.x / NUM_XCD, nslot = gridDim.x / NUM_XCD;
    const int ntiles = g.ntm * g.ntn;
    const int seq_end = min((xcd + 1) * g.per_xcd, PART ? ntiles * g.ksplit : ntiles);
    int seq = xcd * g.per_xcd + slot;                            // this workgroup's tiles: seq, seq + nslot, ...
    if (seq >= seq_end) return;
    // PART: sequence number s is tile s % ntiles of K range s / ntiles (g.kslabs pairs of slabs, the last range may be shorter)
    auto range_slabs = [&](int s) { return PART ? 2 * min(g.kslabs, g.K / (2 * BK) - s / ntiles * g.kslabs) : g.K / BK; };
    const bool has_last = A_EVEN || wave < A_LAST;
    const bool has_rs = g.a_row_scale != nullptr, has_bias = g.bias != nullptr;
    if (!has_bias)                                               // the bias vectors are read by the epilogue either way
        for (int c = tid; c < 2 * BN; c += NT) sv0[(c / BN) * SVF + BN + c % BN] = 0.0f;

    // loader: unit u of wave w fills LDS granules [(u * NWAVE + w) * 64, +64) of a slot of A (or B); lane l owns row u * 128 + lrow, stored chunk l % 4 = global chunk (l % 4) ^ ((row >> 2) & 3).
    const int lrow = wave * 16 + (lane >> 2);
    // 16 x 16 tiles swizzle by swz4(row / 4), the weight rows, taken in another order, by swz4(row / 16).  The LDS serves a 128-bit
    // read in four turns of 16 lanes, lanes 0-3, 12-15 and 20-27 in the first, so a turn meets rows 0-3 and 12-15 of one chunk and rows 4-11 of
    // the chunk beside it; with row / 4 itself half of every read's cycles were bank conflicts, with 0, 3, 2, 1 there are none.
    // us: BERT-large layer 32 x 512 304 -> 300, in M1 405 both ways, GPT prefill 8 x 2048 3418 -> 3376.
    auto swz4 = [](int q) { return (q ^ (q << 1)) & 3; };
    const uint32_t lc = (uint32_t)(((lane & 3) ^ (WIDE ? (lrow >> 2) & 3 : swz4(lrow >> 2))) * 16);
    const uint32_t lcb = WIDE ? lc : (uint32_t)(((lane & 3) ^ swz4(lrow >> 4)) * 16);
    const uint32_t wbase = __builtin_amdgcn_readfirstlane(lds_offset(smem) + wave * 1024);
    const uint32_t svbase = __builtin_amdgcn_readfirstlane(lds_offset(sv0));

    // ---- the two issue streams, of A and of B: the tile / slab their next direct loads belong to
    int aseq = seq, akt = 0, aKT, bseq = seq, bkt = 0, bKT, bpar = 0;
    const int8_t* ia; const int8_t* ib;                          // wave-uniform: tile base + slab offset
    uint32_t oa[A_UNITS], ob[B_UNITS];
    int m0b = 0, n0b = 0;                                        // origin of B's tile
    auto range_start = [&](int s) { return PART ? (int64_t)(s / ntiles) * g.kslabs * (2 * BK) : (int64_t)0; };
    auto set_tile_a = [&](int s) {
        if constexpr (!ONE) {
            int m0, n0;
            tile_from_seq<BM, BN>(g, PART ? s % ntiles : s, m0, n0);
            aKT = range_slabs(s);
            ia = g.A + (int64_t)m0 * g.lda + range_start(s);
#pragma unroll
            for (int u = 0; u < A_UNITS; ++u) oa[u] = (uint32_t)min(lrow + u * (NWAVE * 16), g.M - 1 - m0) * (uint32_t)g.lda + lc;
        }
    };
    auto set_tile_b = [&](int s) {
        tile_from_seq<BM, BN>(g, PART ? s % ntiles : s, m0b, n0b);
        if constexpr (ONE) {
            ia = g.A + (int64_t)m0b * g.lda + range_start(s);
#pragma unroll
            for (int u = 0; u < A_UNITS; ++u) oa[u] = (uint32_t)min(lrow + u * (NWAVE * 16), g.M - 1 - m0b) * (uint32_t)g.lda + lc;
        }
        bKT = range_slabs(s);
        ib = g.Bt + (int64_t)n0b * g.ldb + range_start(s);
#pragma unroll
        for (int u = 0; u < B_UNITS; ++u) ob[u] = (uint32_t)min(lrow + u * (NWAVE * 16), g.N - 1 - n0b) * (uint32_t)g.ldb + lcb;
    };
    // The epilogue vectors of B's tile go out together with its FIRST pair, not when the stream
    // moves on to the tile: their buffer (parity of the tile) is still being read by the epilogue of the tile
    // two back until every wave has started the tile in between.
    auto issue_tile_vectors = [&](int par) {
        // wave w fetches 64 entries (chunk w % CH) of vectors w / CH and 2 + w / CH
        constexpr int CH = BN / 64;
        static_assert(NWAVE == 2 * CH, "two vectors per wave");
        const int ch = (wave % CH) * 64, which = wave / CH;
        const uint32_t dst = svbase + par * SVF * 4 + ch * 4;
        const uint32_t cn = (uint32_t)min(ch + lane, g.N - 1 - n0b) * 4u, cm = (uint32_t)min(ch + lane, g.M - 1 - m0b) * 4u;
        if (EPI == HERO_EPI_RAW_I32) return;
        if (which == 0) {
            if (!UNIT) dma4s(cn, g.b_col_scale + n0b, dst);
            if (EPI == HERO_EPI_GELU_REQUANT) dma4s(cn, g.out_col_scale + n0b, dst + 2 * BN * 4);
        } else {
            if (has_bias) dma4s(cn, g.bias + n0b, dst + BN * 4);
            if (has_rs) dma4s(cm, g.a_row_scale + m0b, dst + 3 * BN * 4);
        }
    };
    // A stream moves in PAIRS of slabs (128 bytes of every row = one cache line): the two 64-byte halves of a line are requested back
    // to back and the second one is served by the line the first one brought in.  In a loop of nothing else, as many workgroups sharing panels as here, a CU
    // takes 57 B/clk from its L2 that way, 43 with the halves one slab apart, 60 in whole lines;  38, 28 and 46 where the panels come from beyond the L2, at any
    // depth from 16 KB per wave on (a 256 x 256 tile needs 32 at the matrix cores' peak, a 128 x 128 tile 64).
    // issue_a(u) / issue_b(u): unit u of both slabs; wra, wrb: LDS offset of the pair's first slot (the second is the next one, round the ring).
    uint32_t wra = 0, wrb = 0;
    auto next_slot = [](uint32_t o, uint32_t bytes, uint32_t ring) { const uint32_t n = o + bytes; return n == ring ? 0u : n; };
    auto issue_a = [&](int u) {
        if (A_EVEN || u + 1 < A_UNITS || has_last) {
            dma16s(oa[u], ia, wbase + (ONE ? wrb : wra) + u * NWAVE * 1024);
            // (the second slab through its own scalar base: an instruction offset would move the LDS side too)
            dma16s(oa[u], ia + BK, wbase + next_slot(ONE ? wrb : wra, A_BYTES, A_RING) + u * NWAVE * 1024);
        }
    };
    auto issue_b = [&](int u) {
        if (!STEADY && u == 0 && bkt == 0) issue_tile_vectors(bpar);
        dma16s(ob[u], ib, wbase + A_RING + wrb + u * NWAVE * 1024);
        dma16s(ob[u], ib + BK, wbase + A_RING + next_slot(wrb, B_BYTES, B_RING) + u * NWAVE * 1024);
    };
    auto advance_a = [&]() {                                     // next pair; past the last tile the last pair repeats (never read)
        if constexpr (ONE) return;
        wra = next_slot(next_slot(wra, A_BYTES, A_RING), A_BYTES, A_RING);
        if constexpr (STEADY) { ia += 2 * BK; return; }
        akt += 2;
        if (akt < aKT) { ia += 2 * BK; return; }
        if (aseq + nslot < seq_end) {
            aseq += nslot; akt = 0;
            set_tile_a(aseq);
        } else akt = aKT - 2;
    };
    auto advance_b = [&]() {
        wrb = next_slot(next_slot(wrb, B_BYTES, B_RING), B_BYTES, B_RING);
        if constexpr (STEADY) { ib += 2 * BK; return; }
        bkt += 2;
        if (bkt < bKT) { ib += 2 * BK; if constexpr (ONE) ia += 2 * BK; return; }
        if (bseq + nslot < seq_end) {
            bseq += nslot; bkt = 0; bpar ^= 1;
            set_tile_b(bseq);
        } else bkt = bKT - 2;
    };

    // fragment offsets inside a slot (row rr, k-step ks, half hh): rr*64 + ((2ks+hh) ^ ((rr>>2)&3))*16
    const int hh = lane >> 5, ml = lane & 31;
    // 16 x 16 tiles: row r = l % 16, chunk l / 16; weight row r of tile j is column 16 (r / 4) + 4 j + r % 4 of the wave's 64
    constexpr int TI = BM / WM / 16, TJ = 2 * TN;
    static_assert(WIDE || TJ == 4, "16 x 16 tiles: 64 columns per wave");
    const int r16 = lane & 15, ch16 = ((lane >> 4) ^ swz4(r16 >> 2)) << 4;
    const int foa = (wm * TI * 16 + r16) * 64 + ch16, fob = A_RING + (wn * 64 + 16 * (r16 >> 2) + (r16 & 3)) * 64 + ch16;
    int fo[2][NFR];
#pragma unroll
    for (int t = 0; t < NFR; ++t) {
        const int rr = (t < TN ? wn * TN * 32 + t * 32 : wm * TM * 32 + (t - TN) * 32) + ml;
        const int base = (t < TN ? A_RING : 0) + rr * 64;
        fo[0][t] = base + (((0 + hh) ^ ((rr >> 2) & 3)) << 4);
        fo[1][t] = base + (((2 + hh) ^ ((rr >> 2) & 3)) << 4);
    }

    // prologue: what the iterations before the first would have issued, in their order; slab 0 landed
    constexpr int LA = 2 * A_UNITS, LB = 2 * B_UNITS;
    set_tile_a(seq);
    set_tile_b(seq);
#pragma unroll
    for (int t = -5; t < 0; ++t) {
        const int pb = t + NSB - 1, pa = t + NSA - 1;              // twice the pair whose turn it is
        if (pa >= 0 && pa % 2 == 0) {
#pragma unroll
            for (int u = 0; u < A_UNITS; ++u) issue_a(u);
            advance_a();
        }
        if (pb >= 0 && pb % 2 == 0) {
            if (STEADY && pb == 0) issue_tile_vectors(0);
#pragma unroll
            for (int u = 0; u < B_UNITS; ++u) issue_b(u);
            advance_b();
        }
    }
    if (has_last) __builtin_amdgcn_s_waitcnt(vmcnt_imm(pair_loads_behind(false, NSA, NSB, LA, LB) + 1));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(pair_loads_behind(false, NSA, NSB, LA - 2, LB) + 1));
    __syncthreads();

    int rda = 0, rdb = 0, par = 0;                                  // LDS offsets of the current slab
    for (;;) {
        int m0, n0;
        tile_from_seq<BM, BN>(g, PART ? seq % ntiles : seq, m0, n0);
        const int KT = range_slabs(seq);
        constexpr int CI = WIDE ? TM : TI, CJ = WIDE ? TN : TJ, CR = WIDE ? 16 : 4;
        ACC acc[CI][CJ];
#pragma unroll
        for (int i = 0; i < CI; ++i)
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int r = 0; r < CR; ++r) acc[i][j][r] = 0;
        v4i f0[NFR], f1[NFR], fa[TI], fb[TJ];
        if constexpr (WIDE) {
#pragma unroll
            for (int t = 0; t < NFR; ++t) {
                f0[t] = *reinterpret_cast<const v4i*>(smem + (t < TN ? rdb : rda) + fo[0][t]);
                f1[t] = *reinterpret_cast<const v4i*>(smem + (t < TN ? rdb : rda) + fo[1][t]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < TJ; ++t) fb[t] = *reinterpret_cast<const v4i*>(smem + rdb + fob + t * 256);
#pragma unroll
            for (int t = 0; t < TI; ++t) fa[t] = *reinterpret_cast<const v4i*>(smem + rda + foa + t * 1024);
        }

        // One slab per iteration with the barrier in the middle (see int8_gemm_dma_kernel).  Behind the barrier of iteration i every
        // wave has read the last fragment of slab i, so both its slots are free: a ring of five slots has
        // one to spare and takes the pair (i + 4, i + 5) in even iterations, rings of four and six wait for the odd one
        // and take (i + 3, i + 4), (i + 5, i + 6).  The pairs may already belong to the next tile.
        auto iteration = [&](auto ODD) {
            constexpr bool odd = decltype(ODD)::value;
            constexpr bool put_a = odd == (NSA % 2 == 0), put_b = odd == (NSB % 2 == 0);
            constexpr int NU = (put_a ? A_UNITS : 0) + (put_b ? B_UNITS : 0);      // units to issue: A's, then B's
            const int nda = rda + A_BYTES == A_RING ? 0 : rda + A_BYTES, ndb = ONE ? nda : (rdb + B_BYTES == B_RING ? 0 : rdb + B_BYTES);
            auto issue_unit = [&](int u) { if (put_a && u < A_UNITS) issue_a(u); else issue_b(u - (put_a ? A_UNITS : 0)); };
            // slab i + 1 has landed (mine); what the loads behind the barrier overwrite has been read.  (16 x 16 tiles: the last of the weights'
            // fragments was an operand in front of the barrier, a row's may still be under way.)
            auto wait_next_slab = [&]() {
                constexpr int all = pair_loads_behind(odd, NSA, NSB, LA, LB), part = pair_loads_behind(odd, NSA, NSB, LA - 2, LB);
                constexpr bool lds = put_a || WIDE;
                if (has_last) __builtin_amdgcn_s_waitcnt(lds ? vmcnt_lds_imm(all) : vmcnt_imm(all));
                else __builtin_amdgcn_s_waitcnt(lds ? vmcnt_lds_imm(part) : vmcnt_imm(part));
            };
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (WIDE) {
                // FP8: one 32x32x64 matrix instruction per accumulator and slab (both k halves of a fragment
                // side by side: any K grouping shared by the two operands is the same contraction).  A
                // fragment is reloaded from the next slab right after its last use; the barrier that
                // publishes that slab sits after the first TM instructions.
#pragma unroll
                for (int n = 0; n < NM; ++n) {
                    const int jj = n / TM, ii = n % TM;
                    acc[ii][jj] = mfma_wide_f8(f0[jj], f1[jj], f0[TN + ii], f1[TN + ii], acc[ii][jj]);
                    if (n == TM - 1) {
                        wait_next_slab();
                        __syncthreads();
                    }
                    if (n >= TM - 1) {
#pragma unroll
                        for (int t = 0; t < NFR; ++t) {
                            const int last = t < TN ? t * TM + TM - 1 : (TN - 1) * TM + (t - TN);
                            if ((last < TM - 1 ? TM - 1 : last) == n) {
                                f0[t] = *reinterpret_cast<const v4i*>(smem + (t < TN ? ndb : nda) + fo[0][t]);
                                f1[t] = *reinterpret_cast<const v4i*>(smem + (t < TN ? ndb : nda) + fo[1][t]);
                            }
                        }
                        constexpr int SLOTS = NM - TM + 1, PPS = (NU + SLOTS - 1) / SLOTS;      // units per instruction slot
#pragma unroll
                        for (int u = (n - (TM - 1)) * PPS; u < (n - (TM - 1) + 1) * PPS; ++u)
                            if (u < NU) issue_unit(u);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // 16 x 16 tiles: one instruction takes a whole slab of a row, so every fragment of a slab is read during the slab
                // before, right after its register's last use: the first half of the rows (dead by the barrier) and the weights one by
                // one as the second half is done with them, that half itself at the end.  At least three times TI / 2, rounded down, instructions lie
                // between a read and its use: twelve with 256 rows, nine with 224 and 192, six with 160 and in 128 x 128 tiles.
                // The rows run there and back, so that an instruction shares an operand with the one before it: nothing changes but what toggles, and the clock
                // is what the power limit allows.  us, rows always upwards / this: INT8 16384 x 12288 x 4096 600.8 / 594.0, GELU^quant 16384 x 4096 x 1024
                // 82.8 / 81.8, BF16 109.6 / 108.9;  BERT-large layer 32 x 512 270.9 / 269.0 (282.4 / 280.1 on another card), in M1 357.0 / 356.3, GPT prefill 0 to 1 %
                // by the card.  (The columns there and back as well, over the two iterations of a pair: 631 / 623 us for the first of these, no gain.)
                auto there_and_back = [](int jj, int r, int rows) { return jj & 1 ? rows - 1 - r : r; };
                constexpr int HI = TI / 2, HS = TI - HI, NH = HS * TJ;
                static_assert(NU <= NH, "a slot of the second half for every unit");
#pragma unroll
                for (int n = 0; n < HI * TJ; ++n) {
                    const int jj = n / HI, ii = there_and_back(jj, n % HI, HI);
                    acc[ii][jj] = mfma16_step<ADT>(fb[jj], fa[ii], acc[ii][jj]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                wait_next_slab();
                __syncthreads();                                       // ... and everybody's
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < NH; ++n) {
                    const int jj = n / HS, ii = HI + there_and_back(jj, n % HS, HS);
                    acc[ii][jj] = mfma16_step<ADT>(fb[jj], fa[ii], acc[ii][jj]);
                    if (n < HI) fa[n] = *reinterpret_cast<const v4i*>(smem + nda + foa + n * 1024);
                    if (n % HS == HS - 1) fb[jj] = *reinterpret_cast<const v4i*>(smem + ndb + fob + jj * 256);
                    if (n >= NH - HS) fa[ii] = *reinterpret_cast<const v4i*>(smem + nda + foa + ii * 1024);
                    if constexpr (NU > 0) {                            // evenly over the half
                        constexpr int EV = NH / NU;
                        if (n % EV == 0 && n / EV < NU) issue_unit(n / EV);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (put_b) advance_b();
            if (put_a) advance_a();
            rda = nda; rdb = ndb;
        };
        // STEADY: the streams are D pairs ahead, so that the last D pairs of iterations, in front of which they move on to the next tile, are code of their own
        // and the loop of the others holds no branch but its own.  Past the last tile the last pair repeats (never read).
        constexpr int D = STEADY ? NSA / 2 : 0;
        static_assert(!STEADY || (NSB / 2 == D && !ONE && !WIDE && EPI != HERO_EPI_GELU_REQUANT), "both streams move on together");
        const int KS = KT - 2 * D;
        for (int kt = 0; kt < KS; kt += 2) {
            iteration(std::false_type{});
            iteration(std::true_type{});
            // S_a -> 1 / S_a once per tile (IEEE division): the vectors landed before the first barrier, KT >= 4 leaves another
            if (!WIDE && EPI == HERO_EPI_GELU_REQUANT && kt == 0 && tid < BN) {
                float* const s = sv0 + par * SVF + 2 * BN + tid;
                *s = __fdiv_rn(1.0f, *s);
            }
        }
        if constexpr (STEADY) {
            const bool last = seq + nslot >= seq_end;
            const int back = last ? 2 * BK : 0;
            if (!last) {
                bpar ^= 1;
                set_tile_a(seq + nslot);
                set_tile_b(seq + nslot);
                issue_tile_vectors(bpar);                              // (every wave is past the epilogue that read their buffer)
            }
            static_for<D>([&](auto) {
                ia -= back; ib -= back;
                iteration(std::false_type{});
                iteration(std::true_type{});
            });
        }
        // Prefetch for the caller's next kernel: this tile's share of the lines, one dword of each, through the same
        // direct loads into a scratch corner of the LDS (no register is written, so nothing has to wait for them; the
        // waits of the next main loop only count loads issued after these, and the epilogue in between is far
        // longer than a miss).  What the request brings is the line: into this XCD's L2 and, on its way, into the
        // memory-side cache, where the next kernel's first tiles would otherwise all miss at once.
        if (g.pf_lines > 0) {
            const int w0 = wave * 64;
            if (w0 < g.pf_lpt) {
                const uint32_t line = (uint32_t)min(seq * g.pf_lpt + w0 + lane, g.pf_lines - 1);
                dma4s(line * 128u, reinterpret_cast<const float*>(g.pf),
                      __builtin_amdgcn_readfirstlane(lds_offset(smem + PF_OFF)) + (uint32_t)w0 * 4u);
            }
        }
        // epilogue of this tile; the ring keeps filling with the next tile's slabs meanwhile
        const float* sv = sv0 + par * SVF;
        // STEADY, 16-bit results behind GELU or of 128 x 128 tiles: what hangs on the lane's number is worked out per tile, from a number the compiler cannot carry over
        // the main loop.  Not in front of other 16-bit results: no gain, and it is what a short launch ends with.  us, before the path for whole tiles / per tile / this: FP16
        // 7000 x 1500 x 512 18.4 / 18.6 / 18.4, 9000 x 1000 x 512 17.6 / 17.8 / 17.6, INT8 -> FP16 4000 x 4100 x 4096 68.1 / 68.8 / 68.4, BF16 with a residual 4000 x 4100 x 2048 70.6 / 71.1 /
        // 69.6;  GELU the other way round (FP16 1500 x 3001 x 512 12.4 / 12.4 / 12.5), 128 x 128 too (INT8 -> BF16 1500 x 3001 x 4096 29.3 / 29.3 / 29.4).
        constexpr bool HP = !WIDE && ElemSize<CDT>::v == 2, ANEW = STEADY || (HP && (EPI == HERO_EPI_DEQUANT_GELU || BM == 128));
        int el = lane;
        if constexpr (ANEW) asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(el));
        float rsr[CI];
#pragma unroll
        for (int i = 0; i < CI; ++i)
            rsr[i] = (EPI != HERO_EPI_RAW_I32 && has_rs) ? sv[3 * BN + wm * (BM / WM) + i * (WIDE ? 32 : 16) + (HP || STEADY ? el & 15 : WIDE ? ml : r16)] : 1.0f;
        if constexpr (WIDE) epilogue_direct<BM, BN, WM, WN, EPI, CDT, RDT, true, UNIT>(g, acc, sv, rsr, m0, n0, tid);
        else if constexpr (HP) epilogue_rows16_hp<BM, BN, WM, WN, EPI, CDT, RDT, UNIT>(g, acc, sv, rsr, m0, n0, wave, el);
        else if constexpr (PART) {
            GemmArgs gp = g;
            gp.C = (int32_t*)g.C + (int64_t)(seq / ntiles) * g.M * g.ldc;
            epilogue_rows16<BM, BN, WM, WN, EPI, CDT, UNIT>(gp, acc, sv, rsr, m0, n0, tid);
        } else epilogue_rows16<BM, BN, WM, WN, EPI, CDT, UNIT>(g, acc, sv, rsr, m0, n0, STEADY ? wave * 64 + el : tid);
        seq += nslot;
        par ^= 1;
        if (seq >= seq_end) break;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                      // the redundant tail loads
}

// the prefetch hint's share per tile: at most one request per lane
inline void share_prefetch(GemmArgs& g, int64_t tiles, int lanes) {
    if (g.pf_lines <= 0) return;
    const int64_t lpt = (g.pf_lines + tiles - 1) / tiles;
    g.pf_lpt = (int)(lpt < lanes ? lpt : lanes);
}
// Slots of the two rings, A and B, for a tile of BM x 256: what 160 KB hold.  Both operands in the same
// iteration lose what the slots give: 2500 x 4096 x 4096 in tiles of 192 rows 48.0 us with five and five, 42.9 with four and five.
template <int BM> struct PersRing { static constexpr int A = BM == 160 ? 5 : 4, B = BM == 160 ? 6 : 5; };
template <int BM, int BN, int WM, int WN, int NSA, int NSB, int EPI, int CDT, int RDT, int ADT, bool STEADY = false>
hero_status launch_persistent(const GemmArgs& g, int wg_per_cu, hipStream_t st) {
    GemmArgs gp = g;
    gp.ntm = (g.M + BM - 1) / BM; gp.ntn = (g.N + BN - 1) / BN;
    const int64_t tiles = (int64_t)gp.ntm * gp.ntn;
    if (tiles > 0x7fffff00LL) return HERO_ERR_SHAPE;
    gp.per_xcd = (int)((tiles + NUM_XCD - 1) / NUM_XCD);
    share_prefetch(gp, tiles, WM * WN * 64);
    const int cap = 32 * wg_per_cu;                                   // 32 CUs per XCD
    const int nslot = gp.per_xcd < cap ? gp.per_xcd : cap;
    hipLaunchKernelGGL((int8_gemm_persistent_kernel<BM, BN, WM, WN, NSA, NSB, EPI, CDT, RDT, ADT, false, STEADY>), dim3((unsigned)(nslot * NUM_XCD)), dim3(WM * WN * 64), 0, st, gp);
    return hero_launch_status();
}

// a tile of `rows` x 256, or 128 x 128
template <int ADT, int EPI, int CDT, int RDT>
hero_status launch_persistent_tile(const GemmArgs& g, int rows, hipStream_t st) {
    auto wide = [&](auto R) {
        constexpr int BM = decltype(R)::value;
        return launch_persistent<BM, 256, 2, 4, PersRing<BM>::A, PersRing<BM>::B, EPI, CDT, RDT, ADT>(g, 1, st);
    };
    // The branch-free loop where a launch has four tiles per CU and more of 64 slabs and more.  It takes 1223 cycles per slab of 1024 cycles of matrix instructions
    // where the other takes 1405 (the same at any clock: what waits is not memory), and the clock falls by half of that.  us, other / this: INT8 16384 x
    // 12288 x 4096 608.8 / 584.0 (2.82 POP/s), 16-bit result 16384 x 4096 x 4096 217.8 / 211.3, x 16384 829.7 / 796.5, BF16 16384 x 12288 x 4096 1188 /
    // 1149;  GPT prefill 8 x 2048 3055 / 3004.  Not for less, though by itself it is ahead there too (one to eight tiles per CU of 16 slabs 0.96 to 1.01 of the other's time,
    // of 32 and more 0.94 to 0.98: REQUANT 16384 x 1024 x 4096 55.6 / 53.5, x 16384 209.0 / 201.8, 16384 x 3072 x 2048 88.1 / 83.0): the BERT-large layer, whose other kernels pay for
    // the clock, was 2 % slower with it everywhere, and with it for FC2 alone (one tile per CU, 64 slabs; in M1 128) 284.9 / 286.6, in M1 361.0 / 360.9.
    // GELU^quant 16384 x 16384 x 4096 921 / 900 by itself, but GPT prefill as long with it.  All but one of the twelve INT8 and BF16 forms spill two to six registers,
    // which come back where the streams move on to the next tile and wait there for the loads under way (GPT's QKV writes 202.9 MB, its result is 201.3).
    if constexpr (ADT != HERO_F8E4M3 && EPI != HERO_EPI_GELU_REQUANT)
        if (rows == 256 && g.K >= 64 * BK && ((int64_t)(g.M + 255) / 256) * ((g.N + 255) / 256) >= 4 * 256)
            return launch_persistent<256, 256, 2, 4, PersRing<256>::A, PersRing<256>::B, EPI, CDT, RDT, ADT, true>(g, 1, st);
    if (rows == 256) return wide(std::integral_constant<int, 256>{});
    if (rows == 192) return wide(std::integral_constant<int, 192>{});
    if constexpr (ADT != HERO_F8E4M3) {
        if (rows == 224) return wide(std::integral_constant<int, 224>{});
        if (rows == 160) return wide(std::integral_constant<int, 160>{});
    }
    if (rows != 128) return HERO_ERR_UNSUPPORTED;
    // While a workgroup has one tile, four slots each, filled by one stream: it waits for its weights as long either way, and both operands in one go (the
    // activations first: the other order +3 to 9 %) take fewer requests at a time.  us, weights and activations from memory, four and four / five and four: BF16
    // 301 x 12288 x 4096 61.5 / 65.7, 1100 x 4096 x 4096 60.4 / 63.4, 1310 x 4096 x 16384 224 / 244, INT8 33.7 / 35.0, 33.2 / 34.4, 112 / 118;  beyond, E4M3 6144 x
    // 4096 x 4096 100.8 / 99.6, 12500 x 4096 x 1024 62.0 / 61.5, INT8 60.8 / 61.1, BF16 112.0 / 113.4.  (Two streams for the four and four: E4M3 1693 x 4096 x 16384
    // in cache 121.1 us, one 117.4, BF16 1395 x 4096 x 4096 56.7 and 55.3.)
    if (((int64_t)(g.M + 127) / 128) * ((g.N + 127) / 128) <= 512) return launch_persistent<128, 128, 2, 2, 4, 4, EPI, CDT, RDT, ADT>(g, 2, st);
    return launch_persistent<128, 128, 2, 2, 5, 4, EPI, CDT, RDT, ADT>(g, 2, st);
}

// Pass 1 of a K split: g.ksplit ranges of g.kslabs slabs (of 128 bytes) into planes of g.C, tiles of `rows` x 256.
template <int ADT>
hero_status launch_persistent_part(const GemmArgs& g, int rows, hipStream_t st) {
    auto go = [&](auto R) {
        constexpr int BM = decltype(R)::value;
        GemmArgs gp = g;
        gp.ntm = (g.M + BM - 1) / BM; gp.ntn = (g.N + 255) / 256;
        gp.per_xcd = (gp.ntm * gp.ntn * g.ksplit + NUM_XCD - 1) / NUM_XCD;
        const int nslot = gp.per_xcd < 32 ? gp.per_xcd : 32;
        hipLaunchKernelGGL((int8_gemm_persistent_kernel<BM, 256, 2, 4, PersRing<BM>::A, PersRing<BM>::B, HERO_EPI_RAW_I32, HERO_I32, -1, ADT, true>),
                           dim3((unsigned)(nslot * NUM_XCD)), dim3(512), 0, st, gp);
        return hero_launch_status();
    };
    switch (rows) {
    case 160: return go(std::integral_constant<int, 160>{});
    case 192: return go(std::integral_constant<int, 192>{});
    case 224: return go(std::integral_constant<int, 224>{});
    case 256: return go(std::integral_constant<int, 256>{});
    default: return HERO_ERR_UNSUPPORTED;
    }
}

// what gemm_persistent_*.hip instantiate for their operand type
#define HERO_PERSISTENT_8BIT(ADT, CDT8) \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_REQUANT, CDT8, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_GELU_REQUANT, CDT8, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT, HERO_BF16, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT, HERO_F16, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT, HERO_BF16, HERO_BF16>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT, HERO_F16, HERO_F16>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT_GELU, HERO_BF16, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<ADT, HERO_EPI_DEQUANT_GELU, HERO_F16, -1>(const GemmArgs&, int, hipStream_t);
#define HERO_PERSISTENT_16BIT(DT) \
    template hero_status launch_persistent_part<DT>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<DT, HERO_EPI_DEQUANT, DT, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<DT, HERO_EPI_DEQUANT, DT, DT>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<DT, HERO_EPI_DEQUANT_GELU, DT, -1>(const GemmArgs&, int, hipStream_t); \
    template hero_status launch_persistent_tile<DT, HERO_EPI_DEQUANT_GELU, DT, DT>(const GemmArgs&, int, hipStream_t);

}  // namespace hero_gemm
