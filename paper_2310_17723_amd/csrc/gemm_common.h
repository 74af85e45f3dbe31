// What the GEMM kernels share: arguments, matrix instructions per operand type, tile order, the epilogue behind the
// accumulators, direct global -> LDS loads.
#pragma once
#include "hero_common.h"
#include <type_traits>

namespace hero_gemm {

constexpr int KMULT = 64;       // K must be a multiple of this
constexpr int BK = 64;          // bytes of K per LDS slab
constexpr int LDS_LD = BK + 16; // padded slab row stride of the register-staged kernel
constexpr int GROUP_M = 8;      // tile order: 8 row panels x 8 column panels run together on one XCD
constexpr int NUM_XCD = 8;

struct GemmArgs {
    const int8_t* A; int64_t lda; const float* a_row_scale;
    const int8_t* Bt; int64_t ldb; const float* b_col_scale;
    const float* bias; const void* residual; int64_t ldr;
    const float* out_col_scale;
    void* C; int64_t ldc;
    int M, N, K;
    int ntm, ntn, per_xcd;      // tile grid and tiles per XCD
    // split-K (skinny M): blockIdx.y picks a range of kslabs slabs and writes raw int32 partial sums
    // to its own [M][ldc] plane of C (plane stride M * ldc elements); a second kernel adds the planes
    int ksplit, kslabs;
    // optional (persistent kernels only): memory the NEXT kernel of the caller's chain will read (a layer's next weight
    // matrix).  Every tile requests pf_lpt of its pf_lines 128-byte lines once, at the start of its epilogue.  (The ring kernel
    // does not: requests behind its first slabs changed 24 layers of BERT-large at 1500 .. 6000 tokens by +-0.3 %, -1.4 % at most.)
    const int8_t* pf = nullptr; int pf_lines = 0, pf_lpt = 0;
};

// Operand types of the main loops.  ADT = HERO_I8: INT8 operands, int32 accumulators.  ADT = HERO_BF16: bf16
// operands (the BF16 side of a switched module, Sec. 2.3 / Table 1), fp32 accumulators, no scales; K, lda and ldb
// are then in BYTES, and a 64-byte slab holds two v_mfma_f32_32x32x16_bf16 steps exactly as it holds two INT8
// steps.  ADT = HERO_F8E4M3: the FP8 variant (Sec. 2.1), fp32 accumulators, the INT8 epilogue; a 16-byte
// fragment feeds two v_mfma_f32_32x32x16_fp8_fp8 (its low and its high 8 bytes: any grouping of K is a valid
// contraction as long as both operands use the same one).
typedef _Float16 v8hf __attribute__((ext_vector_type(8)));
template <int ADT, typename ACC>
__device__ __forceinline__ ACC mfma_step(v4i a, v4i b, ACC c) {
    if constexpr (ADT == HERO_I8) return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    else if constexpr (ADT == HERO_BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    else if constexpr (ADT == HERO_F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8hf, a), __builtin_bit_cast(v8hf, b), c, 0, 0, 0);
    else {
        const long a0 = (long)(((uint64_t)(uint32_t)a[1] << 32) | (uint32_t)a[0]), a1 = (long)(((uint64_t)(uint32_t)a[3] << 32) | (uint32_t)a[2]);
        const long b0 = (long)(((uint64_t)(uint32_t)b[1] << 32) | (uint32_t)b[0]), b1 = (long)(((uint64_t)(uint32_t)b[3] << 32) | (uint32_t)b[2]);
        c = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a0, b0, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a1, b1, c, 0, 0, 0);
    }
}
// The same on 16 x 16 tiles: one instruction takes a whole 64-byte slab of 16 rows of each operand.  At the clock the power limit allows
// these sustain more than the 32 x 32 ones (half the accumulator traffic per multiply-add; hero_probe_mfma_i8, registers only, random
// bytes: INT8 4.15 against 3.48 POP/s).
template <int ADT> struct Acc4Of { using type = typename std::conditional<ADT == HERO_I8, v4i, v4f>::type; };
template <int ADT, typename ACC>
__device__ __forceinline__ ACC mfma16_step(v4i a, v4i b, ACC c) {
    if constexpr (ADT == HERO_I8) return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
    else if constexpr (ADT == HERO_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8hf, a), __builtin_bit_cast(v8hf, b), c, 0, 0, 0);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), in order
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); static_for<N, I + 1>(f); }
}
template <int ADT> struct AccOf { using type = typename std::conditional<ADT == HERO_I8, v16i, v16f>::type; };

template <int CDT> struct ElemSize { static constexpr int v = CDT == HERO_I32 ? 4 : ((CDT == HERO_I8 || CDT == HERO_F8E4M3) ? 1 : 2); };

// XCD-aware tile order: workgroups go round-robin to the 8 XCDs, so XCD x takes the
// contiguous range [x * per_xcd, (x+1) * per_xcd) of a grouped order in which 64
// consecutive tiles form an 8 x 8 square of panels (operands shared through that XCD's L2).
template <int BM, int BN>
__device__ __forceinline__ void tile_from_seq(const GemmArgs& g, int seq, int& m0, int& n0) {
    const int grp = seq / (GROUP_M * g.ntn), rem = seq % (GROUP_M * g.ntn);
    const int gsize = min(g.ntm - grp * GROUP_M, GROUP_M);
    m0 = (grp * GROUP_M + rem % gsize) * BM;
    n0 = (rem / gsize) * BN;
}
template <int BM, int BN>
__device__ __forceinline__ bool tile_origin(const GemmArgs& g, int& m0, int& n0) {
    const int seq = (blockIdx.x % NUM_XCD) * g.per_xcd + blockIdx.x / NUM_XCD;
    if (seq >= g.ntm * g.ntn) return false;
    tile_from_seq<BM, BN>(g, seq, m0, n0);
    return true;
}

// Per-column epilogue vectors of the tile -> LDS ([3][BN] floats: column scale, bias,
// output scale), issued before the main loop so their latency hides behind it.
template <int BN, int NT, int EPI, bool UNIT = false>
__device__ __forceinline__ void stage_col_vectors(const GemmArgs& g, float* sv, int n0, int tid) {
    if (EPI == HERO_EPI_RAW_I32) return;
    for (int c = tid; c < BN; c += NT) {
        const int n = min(n0 + c, g.N - 1);
        if (!UNIT) sv[c] = g.b_col_scale[n];
        sv[BN + c] = g.bias ? g.bias[n] : 0.0f;
        if (EPI == HERO_EPI_GELU_REQUANT) sv[2 * BN + c] = __fdiv_rn(1.0f, g.out_col_scale[n]);   // 1 / S_a[j]
    }
}

// ---- direct epilogue ---------------------------------------------------------------------------
// No LDS: after the fp32 epilogue a lane holds, for ONE output row, 4-column groups q (columns
// 8q + 4hh .. + 3 of the wave's 32*TN columns).  v_permlane32_swap exchanges the groups q >= NQ/2
// of lanes 0..31 with the groups q < NQ/2 of lanes 32..63, after which lane l < 32 owns the
// row's first 16*TN columns and lane l + 32 the other 16*TN, contiguous in registers: every lane
// writes one contiguous piece of its row (32 B of INT8 codes, 64 B of 16-bit values for TN = 2)
// with 128-bit stores, and the residual of the fused add is read in the same layout.
__device__ __forceinline__ void swap32(uint32_t a, uint32_t b, uint32_t& lo, uint32_t& hi) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);   // r[0] = {a.low, b.low}, r[1] = {a.high, b.high}
    lo = r[0]; hi = r[1];
}
// ND dwords of one row, first column col (ES bytes per element), bounds-checked against N unless `full`
template <int ES, int ND>
__device__ __forceinline__ void store_piece(int8_t* cp, const uint32_t (&d)[ND], int col, int N, bool full, bool al16) {
    constexpr int EPD = 4 / ES;                                     // elements per dword
    if (full) {
        if (al16) {
#pragma unroll
            for (int k = 0; k < ND / 4; ++k) {
                v4i o = {(int)d[4 * k], (int)d[4 * k + 1], (int)d[4 * k + 2], (int)d[4 * k + 3]};
                *reinterpret_cast<v4i*>(cp + 16 * k) = o;
            }
        } else {
#pragma unroll
            for (int k = 0; k < ND; ++k) *reinterpret_cast<uint32_t*>(cp + 4 * k) = d[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const int c = col + k * EPD;
            if (c + EPD <= N) *reinterpret_cast<uint32_t*>(cp + 4 * k) = d[k];
            else if (ES < 4) {
#pragma unroll
                for (int b = 0; b < EPD; ++b)
                    if (c + b < N) {
                        if (ES == 1) cp[4 * k + b] = (int8_t)(d[k] >> (8 * b));
                        else *reinterpret_cast<uint16_t*>(cp + 4 * k + 2 * b) = (uint16_t)(d[k] >> (16 * b));
                    }
            }
        }
    }
}

// ACC is v16i (INT8 operands) or v16f (bf16 operands: UNIT, no scales, y = acc + bias).
template <int BM, int BN, int WM, int WN, int EPI, int CDT, int RDT, bool OS_RAW = false, bool UNIT = false, typename ACC = v16i>
__device__ __forceinline__ void epilogue_direct(const GemmArgs& g, ACC (&acc)[BM / WM / 32][BN / WN / 32],
                                                const float* sv, const float (&rsr)[BM / WM / 32],
                                                int m0, int n0, int tid) {
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32, NQ = TN * 4, H = NQ / 2;
    constexpr bool FUSE_RES = RDT >= 0;
    constexpr int ES = ElemSize<CDT>::v;
    const int lane = tid & 63, wave = tid >> 6, wm = wave / WN, wn = wave % WN;
    const int hh = lane >> 5, ml = lane & 31;
    const bool has_rs = g.a_row_scale != nullptr;
    const int colw = n0 + wn * TN * 32;                            // first column of this wave
    const int col0 = colw + hh * H * 8;                            // first column this lane stores (after the swap)
    const bool al16 = (g.ldc * ES) % 16 == 0;
    const bool full = col0 + H * 8 <= g.N;

    // per-column vectors of this lane's 4-column groups, from LDS into registers once
    v4f cs[NQ], bs[NQ];
    if (EPI != HERO_EPI_RAW_I32) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int nl = wn * TN * 32 + q * 8 + hh * 4;
            if (!UNIT) cs[q] = *reinterpret_cast<const v4f*>(sv + nl);
            bs[q] = *reinterpret_cast<const v4f*>(sv + BN + nl);
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = m0 + wm * TM * 32 + i * 32 + ml;
        const bool rowok = row < g.M;
        const float rs = rsr[i];
        if constexpr (EPI == HERO_EPI_RAW_I32) {                  // 16 bytes per group: stored as they are
            if (rowok) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int j = q >> 2, gq = q & 3, col = colw + q * 8 + hh * 4;
                    uint32_t d[4];                                  // int32 sums, or the bits of fp32 ones
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const auto v = acc[i][j][4 * gq + t];
                        if constexpr (std::is_same<ACC, v16i>::value) d[t] = (uint32_t)v;
                        else d[t] = __float_as_uint(v);
                    }
                    if (col < g.N) store_piece<4, 4>((int8_t*)g.C + ((int64_t)row * g.ldc + col) * 4, d, col, g.N, col + 4 <= g.N, al16);
                }
            }
        } else {
            float y[NQ][4];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int j = q >> 2, gq = q & 3;
                v4f os;                                           // 1 / S_a of the group, re-read per pass (registers)
                if (EPI == HERO_EPI_GELU_REQUANT) {
                    int nl = wn * TN * 32 + q * 8 + hh * 4;
                    asm volatile("" : "+v"(nl));                  // opaque: one load per pass, not one long-lived copy
                    os = *reinterpret_cast<const v4f*>(sv + 2 * BN + nl);
                    if (OS_RAW)                                   // the vector holds S_a itself: hardware reciprocal (1 ulp; +-1 LSB class)
#pragma unroll
                        for (int t = 0; t < 4; ++t) os[t] = __builtin_amdgcn_rcpf(os[t]);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float v = (float)acc[i][j][4 * gq + t];
                    if (UNIT) v = v + bs[q][t];
                    else {
                        if (has_rs) v = v * rs;
                        v = fmaf(v, cs[q][t], bs[q][t]);
                    }
                    if (EPI == HERO_EPI_DEQUANT_GELU || EPI == HERO_EPI_GELU_REQUANT) v = gelu_erf(v);
                    // GELU^quant is in the +-1 LSB class (fp32 GELU vs the definition's fp64), so the
                    // division by S_a[j] is a multiplication by its reciprocal
                    if (EPI == HERO_EPI_GELU_REQUANT) v = v * os[t];
                    y[q][t] = v;
                }
            }
            if constexpr (ES == 1) {
                uint32_t w[NQ], d[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    w[q] = CDT == HERO_F8E4M3 ? fp8x4_sat(y[q][0], y[q][1], y[q][2], y[q][3]) : quant4_sat(y[q][0], y[q][1], y[q][2], y[q][3]);
#pragma unroll
                for (int q = 0; q < H; ++q) swap32(w[q], w[q + H], d[2 * q], d[2 * q + 1]);
                if (rowok && col0 < g.N) store_piece<1, NQ>((int8_t*)g.C + (int64_t)row * g.ldc + col0, d, col0, g.N, full, al16);
            } else if constexpr (!FUSE_RES) {
                uint32_t d[2 * NQ];
#pragma unroll
                for (int q = 0; q < H; ++q) {
                    const uint32_t a0 = pack2_hp<CDT>(y[q][0], y[q][1]), a1 = pack2_hp<CDT>(y[q][2], y[q][3]);
                    const uint32_t b0 = pack2_hp<CDT>(y[q + H][0], y[q + H][1]), b1 = pack2_hp<CDT>(y[q + H][2], y[q + H][3]);
                    swap32(a0, b0, d[4 * q], d[4 * q + 2]);
                    swap32(a1, b1, d[4 * q + 1], d[4 * q + 3]);
                }
                if (rowok && col0 < g.N) store_piece<2, 2 * NQ>((int8_t*)g.C + ((int64_t)row * g.ldc + col0) * 2, d, col0, g.N, full, al16);
            } else {
                // fused residual: the fp32 values change lanes, the residual is read in the stored layout
                uint32_t z[H][8], d[2 * NQ];
#pragma unroll
                for (int q = 0; q < H; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        swap32(__float_as_uint(y[q][t]), __float_as_uint(y[q + H][t]), z[q][t], z[q][4 + t]);
                if (rowok && col0 < g.N) {
                    const uint16_t* rp = (const uint16_t*)g.residual + (int64_t)row * g.ldr + col0;
                    const bool rl16 = (g.ldr * 2) % 16 == 0 && ((uintptr_t)g.residual & 15) == 0;
#pragma unroll
                    for (int q = 0; q < H; ++q) {
                        uint32_t r[4];
                        if (full && rl16) {
                            v4i rv = *reinterpret_cast<const v4i*>(rp + 8 * q);
                            r[0] = rv[0]; r[1] = rv[1]; r[2] = rv[2]; r[3] = rv[3];
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const int c = col0 + 8 * q + 2 * k;
                                const uint32_t e0 = c < g.N ? rp[8 * q + 2 * k] : 0, e1 = c + 1 < g.N ? rp[8 * q + 2 * k + 1] : 0;
                                r[k] = e0 | (e1 << 16);
                            }
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            d[4 * q + k] = pack2_hp<CDT>(__uint_as_float(z[q][2 * k]) + hp_to_f32<RDT>(r[k] & 0xffffu),
                                                         __uint_as_float(z[q][2 * k + 1]) + hp_to_f32<RDT>(r[k] >> 16));
                        }
                    }
                    store_piece<2, 2 * NQ>((int8_t*)g.C + ((int64_t)row * g.ldc + col0) * 2, d, col0, g.N, full, al16);
                }
            }
        }
    }
}

// The epilogue behind 16 x 16 tiles whose weight rows were taken in the order 16 (r / 4) + 4 j + r % 4 (r: row of the instruction, j: its
// tile of the wave's 64 columns): lane l then holds, for ONE output row (l % 16 of each of the TI tiles), the 16 consecutive columns
// 16 (l / 16) .. + 15, column 4 j + t in acc[i][j][t], and nothing has to change lanes.  8-bit results and raw sums.
template <int BM, int BN, int WM, int WN, int EPI, int CDT, bool UNIT, typename ACC, int TI>
__device__ __forceinline__ void epilogue_rows16(const GemmArgs& g, ACC (&acc)[TI][4], const float* sv, const float (&rsr)[TI], int m0, int n0, int tid) {
    static_assert(BN / WN == 64 && BM / WM == 16 * TI, "a wave owns 64 columns");
    constexpr int ES = ElemSize<CDT>::v;
    static_assert(ES != 2, "epilogue_rows16_hp is for 16 bits");
    const int lane = tid & 63, wave = tid >> 6, wm = wave / WN, wn = wave % WN, nl = wn * 64 + (lane >> 4) * 16;
    const int col0 = n0 + nl;
    const bool has_rs = g.a_row_scale != nullptr, al16 = (g.ldc * ES) % 16 == 0, full = col0 + 16 <= g.N;
    v4f cs[4], bs[4];
    if (EPI != HERO_EPI_RAW_I32) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!UNIT) cs[j] = *reinterpret_cast<const v4f*>(sv + nl + 4 * j);
            bs[j] = *reinterpret_cast<const v4f*>(sv + BN + nl + 4 * j);
        }
    }
    v4f os[4];                                                    // 1 / S_a
    if (EPI == HERO_EPI_GELU_REQUANT) {
#pragma unroll
        for (int j = 0; j < 4; ++j) os[j] = *reinterpret_cast<const v4f*>(sv + 2 * BN + nl + 4 * j);
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int row = m0 + wm * TI * 16 + i * 16 + (lane & 15);
        const bool ok = row < g.M && col0 < g.N;
        if constexpr (EPI == HERO_EPI_RAW_I32) {
            uint32_t d[16];                                       // int32 sums, or the bits of fp32 ones
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const auto v = acc[i][e >> 2][e & 3];
                if constexpr (std::is_same<ACC, v4i>::value) d[e] = (uint32_t)v;
                else d[e] = __float_as_uint(v);
            }
            if (ok) store_piece<4, 16>((int8_t*)g.C + ((int64_t)row * g.ldc + col0) * 4, d, col0, g.N, full, al16);
        } else {
            const float rs = rsr[i];
            float y[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v = (float)acc[i][e >> 2][e & 3];
                if (UNIT) v = v + bs[e >> 2][e & 3];
                else {
                    if (has_rs) v = v * rs;
                    v = fmaf(v, cs[e >> 2][e & 3], bs[e >> 2][e & 3]);
                }
                if (EPI == HERO_EPI_GELU_REQUANT) v = gelu_erf(v) * os[e >> 2][e & 3];      // the +-1 LSB class, see epilogue_direct
                y[e] = v;
            }
            uint32_t d[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                d[j] = CDT == HERO_F8E4M3 ? fp8x4_sat(y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]) : quant4_sat(y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]);
            if (ok) store_piece<1, 4>((int8_t*)g.C + (int64_t)row * g.ldc + col0, d, col0, g.N, full, al16);
        }
    }
}

// The same for 16-bit results.  WHOLE: all of the wave's rows and columns exist and its pieces lie on 16 bytes (uniform), so that neither a row nor
// a store asks again and a row's address is the one above it plus a constant: four branches and 64-bit products per row were a tenth of the epilogue.
// us, asked per row -> once, what the lane's number enters worked out per tile (where the kernel still does), GELU of eight values side by side (of the three it is the first that counts: INT8 -> FP16 GELU 16384 x 4096
// x 1024 85.8 before, 84.6 with the other two, 82.7 with all; FP16 16384 x 4096 x 512 74.5, 74.4, 73.3): BERT-large layer 32 x 512 in M1 362.0 -> 358.5, GELU 602 x 16384 x 4096
// 47.5 -> 46.8, GPT prefill 8 x 2048 3112 -> 3101, chunk 2 x 301 unchanged.
// (8-bit results keep the other form: theirs is ahead by 2 to 4 % launched by itself, REQUANT 16384 x 3072 x 1024 50.1 -> 48.3, but the BERT-large layer is
// up to 2 % slower: its clock falls by more than the cycles.)
// A residual off 16-byte boundaries, and that of a piece that N cuts, comes element by element without a test (columns past the last one read the last one and
// are not stored): a test is a branch, and every second element was waited for by itself, row after row of the tile that ends the launch.  us, a test per element
// before this form of the epilogue, with it -> now: off 16 bytes INT8 16384 x 1024 x 1024 (rows 1028 apart) 40.0, 40.4 -> 24.8, BF16 16384 x 3076 x 1024 168.8, 171.3 -> 118.8;
// cut FP16 + GELU 2049 x 2303 x 512 15.6, 16.1 -> 14.6, INT8 -> BF16 3000 x 3000 x 1024 21.4, 21.6 -> 20.3, 7000 x 1500 x 1024 25.1, 25.4 -> 23.6.
template <int BM, int BN, int WM, int WN, int EPI, int CDT, int RDT, bool UNIT, typename ACC, int TI>
__device__ __forceinline__ void epilogue_rows16_hp(const GemmArgs& g, ACC (&acc)[TI][4], const float* sv, const float (&rsr)[TI], int m0, int n0, int wave, int lane) {
    static_assert(BN / WN == 64 && BM / WM == 16 * TI && ElemSize<CDT>::v == 2, "a wave owns 64 columns, 16-bit results");
    const int wm = wave / WN, wn = wave % WN, nl = wn * 64 + (lane >> 4) * 16;
    const int col0 = n0 + nl, mw = m0 + wm * TI * 16;
    const bool al16 = (g.ldc * 2) % 16 == 0, full = col0 + 16 <= g.N;
    const bool rl16 = RDT >= 0 && (g.ldr * 2) % 16 == 0 && ((uintptr_t)g.residual & 15) == 0;
    v4f cs[4], bs[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!UNIT) cs[j] = *reinterpret_cast<const v4f*>(sv + nl + 4 * j);
        bs[j] = *reinterpret_cast<const v4f*>(sv + BN + nl + 4 * j);
    }
    auto rows = [&](auto WHOLE) {
        constexpr bool whole = decltype(WHOLE)::value;
        int8_t* cp = (int8_t*)g.C + ((int64_t)(mw + (lane & 15)) * g.ldc + col0) * 2;
        const uint16_t* rp = RDT >= 0 ? (const uint16_t*)g.residual + (int64_t)(mw + (lane & 15)) * g.ldr + col0 : nullptr;
#pragma unroll
        for (int i = 0; i < TI; ++i, cp += 32 * g.ldc, rp += RDT >= 0 ? 16 * g.ldr : 0) {
            float y[16];
#pragma unroll
            for (int h = 0; h < 16; h += 8) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int j = (h + e) >> 2, t = e & 3;
                    v[e] = (float)acc[i][j][t];
                    if (UNIT) v[e] = v[e] + bs[j][t];
                    else v[e] = fmaf(v[e] * rsr[i], cs[j][t], bs[j][t]);           // (no row scale: 1)
                }
                if (EPI == HERO_EPI_DEQUANT_GELU) gelu_erf8(v);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[h + e] = v[e];
            }
            if (!whole && (mw + i * 16 + (lane & 15) >= g.M || col0 >= g.N)) continue;
            if constexpr (RDT >= 0) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    uint32_t r[4];
                    if (whole || (full && rl16)) {
                        const v4i rv = *reinterpret_cast<const v4i*>(rp + 8 * q);
                        r[0] = rv[0]; r[1] = rv[1]; r[2] = rv[2]; r[3] = rv[3];
                    } else if (full) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) r[k] = rp[8 * q + 2 * k] | ((uint32_t)rp[8 * q + 2 * k + 1] << 16);
                    } else {
                        const int last = g.N - 1 - col0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) r[k] = rp[min(8 * q + 2 * k, last)] | ((uint32_t)rp[min(8 * q + 2 * k + 1, last)] << 16);
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        y[8 * q + 2 * k] += hp_to_f32<RDT>(r[k] & 0xffffu);
                        y[8 * q + 2 * k + 1] += hp_to_f32<RDT>(r[k] >> 16);
                    }
                }
            }
            uint32_t d[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) d[k] = pack2_hp<CDT>(y[2 * k], y[2 * k + 1]);
            store_piece<2, 8>(cp, d, col0, g.N, whole || full, whole || al16);
        }
    };
    // (Not for a plain result of 128 x 128 tiles, where it gains nothing and the loop in front of it comes out slower.  us, without / with: INT8 -> FP16 1500 x 3072 x 4096 29.1 /
    // 29.5, 1500 x 3001 x 4096 29.1 / 29.5, 2049 x 2303 x 4096 29.8 / 30.0, FP16 1500 x 3072 x 2048 28.9 / 29.0.)
    constexpr bool ASK = BM > 128 || RDT >= 0 || EPI == HERO_EPI_DEQUANT_GELU;
    if (ASK && mw + TI * 16 <= g.M && n0 + wn * 64 + 64 <= g.N && al16 && (RDT < 0 || rl16)) rows(std::true_type{});
    else rows(std::false_type{});
}

// s_waitcnt immediate that waits only for vmcnt <= n (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4 and lgkmcnt 11:8 left at their maxima).
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
constexpr int vmcnt_lds_imm(int n) { return vmcnt_imm(n) & ~0x0F00; }        // .. and for every LDS access of this wave

// One direct global->LDS load: 64 lanes x 16 bytes land at LDS address lds_base + lane * 16
// (lds_base is wave-uniform and travels in M0).  Written as inline assembly on purpose: the
// compiler then does not track these loads and does not force vmcnt(0) in front of every LDS
// read; the kernel waits for exactly the slab it is about to read (vmcnt counts them in order).
__device__ __forceinline__ void dma16(const int8_t* gp, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(gp), "s"(lds_base) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) void*)p);
}

__device__ __forceinline__ void dma16s(uint32_t voff, const int8_t* sbase, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory", "m0");
}
__device__ __forceinline__ void dma4s(uint32_t voff, const float* sbase, uint32_t lds_base) {   // lane l -> lds_base + 4 l
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory", "m0");
}

template <typename K>
inline hero_status launch_grid(GemmArgs g, int BM, int BN, int threads, K kernel, hipStream_t st) {
    g.ntm = (g.M + BM - 1) / BM;
    g.ntn = (g.N + BN - 1) / BN;
    const int64_t tiles = (int64_t)g.ntm * g.ntn;
    g.per_xcd = (int)((tiles + NUM_XCD - 1) / NUM_XCD);
    if ((int64_t)g.per_xcd * NUM_XCD > 0x7fffffffLL) return HERO_ERR_SHAPE;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(g.per_xcd * NUM_XCD)), dim3(threads), 0, st, g);
    return hero_launch_status();
}

// ---- the ring kernel's forms (gemm_ring.h): BM x BN tile, number of K groups ---------------------------------
enum RingForm { RING_NONE = -1, RING_32x32_K8, RING_32x32_K4, RING_32x64_K2, RING_32x64_K4, RING_64x32_K4, RING_64x64_K2,
                RING_64x64, RING_128x64_K2, RING_128x64, RING_128x128, RING_128x256 /* K split only */ };

// 32-bit per-lane offsets (256 rows of lda / ldb bytes)
inline bool ring_ok(int64_t lda_bytes, int64_t ldb_bytes) { return lda_bytes < (1 << 24) && ldb_bytes < (1 << 24); }
// Which form, or RING_NONE: a problem for the persistent kernels.  What decides is whether every one of the 256 CUs streams
// its share of the weights: the largest tile that still gives every CU one workgroup, and while there are fewer
// tiles than CUs, K groups inside the workgroup.  (Two workgroups per CU where the form's LDS allows it: 64 x 64 without K
// groups, 128 x 64 without.)  Measured on this kernel over M = 1 .. 16384 and the (N, K) of the three models and of vocabularies,
// every operand type, 16-bit, 8-bit and GELU^quant results, weights resident and cold, 1948 combinations: the choice (persistent
// kernels included) is within 2.2 % of the best of twelve forms on average, 25 % at most.  Some of the figures, us, weights out
// of the caches for the 4096-wide model (register-staged, plain 16-bit or persistent kernels of before -> now):
//   INT8  64 x 12288 x 4096 17.7 -> 15.0, 128 x 12288 x 4096 29.3 -> 19.2, 512 x 4096 x 4096 25.2 -> 16.3,
//         2048 x 1024 x 4096 18.9 -> 14.8, 128 x 768 x 3072 5.5 -> 5.0;  E4M3 64 x 4096 x 4096 13.2 -> 8.6
//   BF16  800 x 768 x 3072 54.6 -> 13.3, 3 x 4096 x 16384 263 -> 37, 700 x 4096 x 16384 213 -> 131
inline RingForm ring_form(int64_t M, int64_t N, int64_t kb, hero_epilogue epi) {
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t slabs = (kb + 2 * BK - 1) / (2 * BK), t32 = tiles(32, 32), t12864 = tiles(128, 64);
    if (M <= 32 && t32 > 256 && tiles(32, 64) <= 256) return slabs >= 64 ? RING_32x64_K4 : RING_32x64_K2;
    if (t32 <= 256) return slabs >= 32 ? RING_32x32_K4 : RING_32x32_K8;       // K8 has a short ring: better while K is short
    if (tiles(64, 32) <= 256) return RING_64x32_K4;
    if (tiles(32, 64) <= 256) return RING_32x64_K4;                           // (651 x 768: 252 of these, 264 of the others)
    if (tiles(64, 64) <= 256) return RING_64x64_K2;
    if (t12864 <= 256 && slabs >= 32) return RING_128x64_K2;
    if (tiles(64, 64) <= 512) return RING_64x64;
    // Few rows and more columns than that (a vocabulary's logits): the weights are all there is to stream, and tall tiles stream
    // them through fewer waves.  us, cold weights, persistent 256 x 256 / this: INT8 1 x 50304 x 4096 57 / 44, 64 rows 58 / 54, BF16
    // 16 rows 108 / 83; 64 x 64 / 32 x 64 with two K groups: 1 x 36864 x 4096 38 / 33, 1 x 50304 x 768 11.9 / 15.7.
    if (M <= 64) return M <= 32 && slabs >= 32 ? (slabs >= 64 ? RING_32x64_K4 : RING_32x64_K2) : RING_64x64;
    // Two rounds or more.  A tile of 64 columns writes half a 128-byte line of an 8-bit result, and GELU leaves the matrix cores
    // idle between two tiles of a workgroup, so only 16-bit and raw results without GELU go on, while K is short (the persistent
    // ring never gets going).  us, 128 x 64 ring / persistent: REQUANT 8192 x 1024 x 1024 19.0 / 15.1, 6000 x 768 x 768 12.0 /
    // 10.1, GELU^quant 2048 x 4096 x 1024 20.0 / 18.2; DEQUANT 8192 x 1024 x 1024 15.7 / 16.5, 2048 x 3072 x 1024 13.2 / 15.0.
    // (the last full round of an 8-bit result: REQUANT 4096 x 1024 x 1024 128 x 64 11.1, 128 x 128 9.3)
    const bool gelu = epi == HERO_EPI_DEQUANT_GELU || epi == HERO_EPI_GELU_REQUANT;
    if (tiles(128, 128) <= 256 && (slabs >= 32 || (epi == HERO_EPI_REQUANT && t12864 > 448))) return RING_128x128;
    if (t12864 <= 512 || (epi != HERO_EPI_REQUANT && !gelu && slabs <= 8 && t12864 <= 1024)) return RING_128x64;
    return RING_NONE;
}
// The weight-streaming kernel of few rows (gemm_skinny.hip): whole 16-column tiles, K in eight equal parts.  Beyond three tiles
// per CU the ring's 64-column tiles stream as well (32-bit-per-lane offsets as there), and below 4 MB of weights a product is
// a launch.  us, cold weights, ring (with the K split where it is one) -> this:
//   INT8 3 x 4096 x 4096 7.3 -> 6.0, 3 x 4096 x 16384 18.6 -> 13.6, 24 rows 18.9 -> 16.1, 3 x 12288 x 4096 11.8 -> 11.2, 24 rows 12.3
//   -> 12.3, 16 x 2560 x 10240 12.7 -> 10.4, 32 x 1024 x 4096 5.6 -> 4.8;  E4M3 24 x 4096 x 4096 8.4 -> 6.9;  BF16 3 x 4096 x 8192 39
//   -> 26, 32 x 2048 x 4096 8.1 -> 6.6;  not taken: INT8 24 x 16384 x 4096 14.4 / 15.0, 3 x 32768 x 1024 8.6 / 10.9
inline bool skinny_ok(int64_t M, int64_t N, int64_t kb, int64_t lda_bytes, int64_t ldb_bytes, int64_t max_n = 12288) {
    return M <= 32 && N % 16 == 0 && N <= max_n && kb % (8 * 2 * BK) == 0 && N * kb >= (4 << 20) && ring_ok(lda_bytes, ldb_bytes);
}
// the persistent kernel (gemm_persistent.h): a tile of `rows` x 256 or, with 128, of 128 x 128; and a K split's planes
template <int ADT, int EPI, int CDT, int RDT> hero_status launch_persistent_tile(const GemmArgs& g, int rows, hipStream_t st);
template <int ADT> hero_status launch_persistent_part(const GemmArgs& g, int rows, hipStream_t st);
hero_status launch_skinny(const GemmArgs& g, hero_dtype adt, hero_epilogue epi, hero_dtype c_dt, hipStream_t st);
template <int ADT, int EPI, int CDT, int RDT, bool HALF> hero_status launch_ring_slabs(const GemmArgs& g, RingForm f, hipStream_t st);
template <int ADT, int EPI, int CDT, int RDT>
hero_status launch_ring(const GemmArgs& g, RingForm f, hipStream_t st) {
    return g.K % (2 * BK) != 0 ? launch_ring_slabs<ADT, EPI, CDT, RDT, true>(g, f, st) : launch_ring_slabs<ADT, EPI, CDT, RDT, false>(g, f, st);
}
// g.ksplit ranges of g.kslabs slabs, raw accumulators into planes of g.C; the forms of the K split
template <int ADT, bool HALF> hero_status launch_ring_part_slabs(GemmArgs g, RingForm f, hipStream_t st);
template <int ADT>
hero_status launch_ring_part(const GemmArgs& g, RingForm f, hipStream_t st) {
    return g.K % (2 * BK) != 0 ? launch_ring_part_slabs<ADT, true>(g, f, st) : launch_ring_part_slabs<ADT, false>(g, f, st);
}

}  // namespace hero_gemm
