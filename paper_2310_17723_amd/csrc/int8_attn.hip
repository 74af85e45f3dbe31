// hero_int8_attn: INT8 attention, QK^T -> Softmax^quant -> PV (paper Sec. 2.2.2, quantized
// attention flow: A = d~ X_q,int8 X_k,int8^T is NOT quantized, S_p P_int8 = Softmax^quant(A)
// with unsigned codes, X_attn,int8 S_attn = S_p S_v P_int8 X_v,int8).
//
// The softmax is normalised before it is quantized, so the row maximum and the row sum
// must be known before the first code is produced.  Four kernels (the rule: attn_entry):
//   * int8_attn_kernel (described here) streams the keys twice (pass 1: QK^T, row max / row sum; pass 2: QK^T
//     again, codes, PV), and in its online variant once;
//   * int8_attn_keep_kernel: up to 512 keys of 64 channels, one pass, the scores kept in registers;
//   * int8_attn_split_kernel: few queries, the keys split over a block's waves;
//   * int8_attn_decode_kernel: one query per sequence, a stream of the cache.
// A and P never leave the chip.
//
// Layout.  A block owns 128 queries of one (batch, head); each of its 4 waves owns 32 of them.
// Scores are computed TRANSPOSED, S^T = K Q^T (v_mfma_i32_32x32x32_i8 with the key
// fragment as first operand), so lane l holds query l % 32 and the keys 8g + 4(l/32) + t
// of a 32-key step in accumulator register 4g + t: a query's row statistics need one
// exchange between lanes l and l^32, and the 16 codes a lane produces are already the
// second-operand fragment of the PV MFMA (O^T = V^T P^T) provided V^T is stored in LDS with
// the same key order, which the V staging does.
// The matrix cores multiply signed bytes; codes are 0..255, so P-128 is fed and
// 128 * colsum(V) is added back, exact in int32.  Masked keys carry code 0 (fed as -128), so
// the column sums run over every staged key and are the same for all queries of the block:
// the four waves take turns adding them up from the V fragments they already hold (v_dot4
// against ones) and exchange them through LDS once, at the end.
// The kernel is bound by the plain-ALU work per score (exp2, conversion, rounding), not by
// the matrix cores, so both passes are written to spend as few vector instructions per score
// as possible (see the comment in front of pass 1).
#include "gemm_common.h"          // direct global -> LDS loads
#include <atomic>
#include <type_traits>

namespace {

constexpr int BQ = 128;   // queries per block
constexpr int BKV = 64;   // keys per LDS tile

struct AttnArgs {
    const int8_t* q; const int8_t* k; const int8_t* v;
    int64_t qs[4], ks[4], vs[4];
    int B, H, Sq, Skv;
    float qk_scale, p_scale;
    const float* qk_scale_h;          // per-head d~ (online variant) or NULL
    int use_buf;                      // K / V of one (batch, head) span < 2 GB with non-negative strides
    const float* out_col_scale; int scale_is_scalar;
    int mask; const int32_t* kv_len;
    void* out; int64_t ldo;
    // decode inside a layer: this call's key / value rows [B][H * DH] (row stride nstride), not yet in the cache; the kernel
    // writes them at position kv_len[b] - 1 (kc / vc: the cache, writable) and attends to them.  NULL: nothing to append
    const int8_t* kn; const int8_t* vn; int64_t nstride; int8_t* kc; int8_t* vc;
};

// the larger of lane l's and lane l ^ 32's value
template <typename T>
__device__ __forceinline__ T pair_max(T x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t lo = r[0], hi = r[1];                      // (a bit cast of the element itself would read r[0] twice)
    return max(__builtin_bit_cast(T, lo), __builtin_bit_cast(T, hi));
}

// the output rows of a block of BQ padded queries: zeros
template <int DH, int ODT>
__device__ __forceinline__ void zero_rows(const AttnArgs& a, int b, int h, int q0, int threads) {
    constexpr int U = DH / 4;                                  // stores of 4 elements, as the kernels' own
    const int rows = min(BQ, a.Sq - q0);
    for (int idx = threadIdx.x; idx < rows * U; idx += threads) {
        const int64_t e = ((int64_t)b * a.Sq + q0 + idx / U) * a.ldo + (int64_t)h * DH + (idx % U) * 4;
        if (ODT == HERO_I8 || ODT == HERO_F8E4M3) *reinterpret_cast<uint32_t*>((int8_t*)a.out + e) = 0u;
        else { v2i z = {0, 0}; *reinterpret_cast<v2i*>((uint16_t*)a.out + e) = z; }
    }
}

// FMT = HERO_F8E4M3: the same flow with E4M3 codes (Sec. 2.1): q, k, v are E4M3 bytes, the scores and the PV sums
// are fp32 accumulators of v_mfma_f32_32x32x64_f8f6f4, the probabilities are quantized to non-negative E4M3 codes
// (saturating at 448 = p / S_p for p = 1 with S_p = 1/448), signed operands need no offset and no column sums.
// Staging, masks, tile order and the two-pass structure are those of the INT8 kernel.
template <int DH, int ODT, bool ONLINE = false, int FMT = HERO_I8>
__global__ __launch_bounds__(256, ONLINE ? (DH == 64 ? 3 : 2) : (DH == 64 ? 4 : 3)) void int8_attn_kernel(AttnArgs a) {
    constexpr bool F8 = FMT == HERO_F8E4M3;
    static_assert(!(F8 && ONLINE), "the online variant is INT8 only");
    using SACC = typename std::conditional<F8, v16f, v16i>::type;     // score / output accumulators
    constexpr int KLD = DH + 16;        // sK row stride (bytes)
    constexpr int VLD = BKV + 16;       // sVt row stride (bytes)
    constexpr int DS = DH / 32;         // 32-wide steps over the head dimension
    __shared__ __attribute__((aligned(16))) int8_t sK[2][BKV * KLD];
    __shared__ __attribute__((aligned(16))) int8_t sVt[2][DH * VLD];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hh = lane >> 5, ql = lane & 31;
    // Workgroups go round-robin to the 8 XCDs; all query blocks of one (batch, head) are sent to
    // the SAME XCD, back to back, so its K / V stream hits that XCD's L2 after the first block, and
    // so are the HG = 128 / DH neighbouring heads whose K / V rows share 128-byte cache lines with it
    // in the packed [token][head][channel] layout (otherwise each XCD would fetch whole lines to use
    // a fraction of them).
    constexpr int HG = DH >= 128 ? 1 : 128 / DH;
    const int nqb = (a.Sq + BQ - 1) / BQ;
    const int slot = blockIdx.x / 8, grp = (slot / (HG * nqb)) * 8 + (blockIdx.x % 8), within = slot % (HG * nqb);
    const int bh = grp * HG + within / nqb;
    if (bh >= a.B * a.H) return;
    // The query blocks of a (batch, head) differ in length (causal: block j sees j + 1 blocks of keys; padding: the
    // blocks past the sequence's end leave at once), and the hardware places workgroups on the compute units in
    // launch order, round and round: with the same order inside every group a compute unit is handed the same kind
    // of block every time, the long ones always go to the same few, and the launch waits for those.  The order
    // inside a group therefore rotates with a hash of the group's number.
    const uint32_t rot = ((uint32_t)(slot / (HG * nqb)) * 2654435761u) >> 20;
    const int qb = (int)((within % nqb + rot) % (uint32_t)nqb);
    const int b = bh / a.H, h = bh % a.H, q0 = qb * BQ;
    const int len = a.kv_len ? min(max(a.kv_len[b], 0), a.Skv) : a.Skv;
    const int shift = len - a.Sq;                       // causal: key k visible iff k <= i + shift
    // Which 32 queries of the block a wave owns rotates with the block: with the padding mask the last sub-blocks
    // of a sequence's last block are idle, and the busy waves of co-resident blocks should not share a SIMD.
    const int wq = (wave + slot) & 3;
    const int qi = q0 + wq * 32 + ql;                   // this lane's query
    int nvis = len;
    if (a.mask == HERO_MASK_CAUSAL) nvis = min(len, qi + shift + 1);
    nvis = max(nvis, 0);
    // keys any query of the block can see -> number of key tiles
    int kmax = len;
    if (a.mask == HERO_MASK_CAUSAL) kmax = min(len, min(q0 + BQ, a.Sq) + shift);
    const int ntiles = (max(kmax, 0) + BKV - 1) / BKV;
    // PADDING mask in self-attention: the positions >= len are padding as queries too and their output rows are
    // zeros.  A block with no real query writes them and leaves; a wave with no real query keeps staging K / V
    // and meeting the barriers (and adds its share of the column sums) but computes no score.
    const int qlim = (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) ? len : a.Sq;
    if (q0 >= qlim) { zero_rows<DH, ODT>(a, b, h, q0, 256); return; }
    const bool wact = __builtin_amdgcn_readfirstlane(q0 + wq * 32) < qlim;     // wave-uniform

    // ---- Q fragments (second MFMA operand), kept in registers -----------------------------
    v4i qf[DS];
    {
        const int8_t* qp = a.q + (int64_t)b * a.qs[0] + (int64_t)min(qi, a.Sq - 1) * a.qs[1] + (int64_t)h * a.qs[2];
#pragma unroll
        for (int d = 0; d < DS; ++d) qf[d] = *reinterpret_cast<const v4i*>(qp + d * 32 + hh * 16);
        // The fragments pass through an empty asm statement so that they count as arrived from here on:
        // otherwise the first MFMA of every tile waits for ALL outstanding global loads (vmcnt(0)),
        // the just-issued prefetch of the next tile included.
#pragma unroll
        for (int d = 0; d < DS; ++d) asm volatile("" : "+v"(qf[d]));
    }
    const int8_t* kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2];
    const int8_t* vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2];

    // K / V tiles: global -> registers (next tile, in flight during the current tile's math) -> LDS
    // (double buffered, one barrier per tile).  V is written transposed, keys permuted so that the
    // PV operand fragment is one 128-bit read: key row 32kb + 8g + 4h + t -> position 32kb + 16h + 4g + t.
    constexpr int UNITS = BKV * (DH / 16) / 256;
    constexpr int VUNITS = (BKV / 4) * (DH / 4) / 256;     // V: units of 4 keys x 4 channels (one dword per key)
    v4i rk[UNITS];
    int rv[VUNITS][4];
    // K / V tiles that lie wholly inside the key range are fetched through buffer descriptors when the
    // host found that a (batch, head) operand spans less than 2 GB: the address is a wave-uniform base
    // plus a 32-bit lane offset (one add per load and tile instead of a 64-bit multiply per load).  A
    // ragged last tile, and operands beyond 2 GB, take clamped 64-bit addresses.
    __amdgpu_buffer_rsrc_t krs, vrs;
    uint32_t koff[UNITS], voff[VUNITS];
    if (a.use_buf) {
        krs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(kbase), 0, (int)((int64_t)(a.Skv - 1) * a.ks[1] + DH), 0x00020000);
        vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(vbase), 0, (int)((int64_t)(a.Skv - 1) * a.vs[1] + DH), 0x00020000);
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int idx = tid + u * 256, row = idx / (DH / 16), ch = idx % (DH / 16);
            koff[u] = (uint32_t)row * (uint32_t)a.ks[1] + ch * 16;
        }
#pragma unroll
        for (int u = 0; u < VUNITS; ++u) {
            const int idx = tid + u * 256, kg = (idx >> 2) % (BKV / 4), cg = (idx & 3) + 4 * (idx / BKV);
            voff[u] = (uint32_t)(kg * 4) * (uint32_t)a.vs[1] + cg * 4;
        }
    }
    auto load_k = [&](int tile) {
        if (a.use_buf && (tile + 1) * BKV <= a.Skv) {
            const uint32_t tb = (uint32_t)tile * (uint32_t)(BKV * (uint32_t)a.ks[1]);
#pragma unroll
            for (int u = 0; u < UNITS; ++u)
                rk[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(krs, koff[u] + tb, 0, 0));
            return;
        }
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            int idx = tid + u * 256, row = idx / (DH / 16), ch = idx % (DH / 16);
            int key = min(tile * BKV + row, a.Skv - 1);
            rk[u] = *reinterpret_cast<const v4i*>(kbase + (int64_t)key * a.ks[1] + ch * 16);
        }
    };
    // V unit: key group kg (4 consecutive keys) x channel group cg (4 channels).  Four consecutive lanes
    // read 16 contiguous bytes of one key row; the 64 transposed dword stores of a wave (rows 4cg + j,
    // 16 key-group positions each) fall into 64 different banks.
    auto load_v = [&](int tile) {
        if (a.use_buf && (tile + 1) * BKV <= a.Skv) {
            const uint32_t tb = (uint32_t)tile * (uint32_t)(BKV * (uint32_t)a.vs[1]);
#pragma unroll
            for (int u = 0; u < VUNITS; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    rv[u][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(vrs, voff[u] + tb + (uint32_t)i * (uint32_t)a.vs[1], 0, 0);
            return;
        }
#pragma unroll
        for (int u = 0; u < VUNITS; ++u) {
            const int idx = tid + u * 256, kg = (idx >> 2) % (BKV / 4), cg = (idx & 3) + 4 * (idx / BKV);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int key = min(tile * BKV + kg * 4 + i, a.Skv - 1);
                rv[u][i] = *reinterpret_cast<const int*>(vbase + (int64_t)key * a.vs[1] + cg * 4);
            }
        }
    };
    auto store_k = [&](int buf) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            int idx = tid + u * 256, row = idx / (DH / 16), ch = idx % (DH / 16);
            *reinterpret_cast<v4i*>(&sK[buf][row * KLD + ch * 16]) = rk[u];
        }
    };
    auto store_v = [&](int buf) {
#pragma unroll
        for (int u = 0; u < VUNITS; ++u) {
            const int idx = tid + u * 256, kg = (idx >> 2) % (BKV / 4), cg = (idx & 3) + 4 * (idx / BKV);
            // 4 x 4 byte transpose in registers: dword j of the result = channel 4cg + j of keys 4kg .. 4kg + 3
            const uint32_t d0 = rv[u][0], d1 = rv[u][1], d2 = rv[u][2], d3 = rv[u][3];
            const uint32_t lo01 = __builtin_amdgcn_perm(d1, d0, 0x05010400u), hi01 = __builtin_amdgcn_perm(d1, d0, 0x07030602u);
            const uint32_t lo23 = __builtin_amdgcn_perm(d3, d2, 0x05010400u), hi23 = __builtin_amdgcn_perm(d3, d2, 0x07030602u);
            const uint32_t t[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                   __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
            // keys 4kg .. 4kg+3 sit at positions pos .. pos+3 of the permuted key order (see above)
            const int pos = ((kg * 4) & 32) + (kg & 1) * 16 + ((kg & 7) >> 1) * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<uint32_t*>(&sVt[buf][(cg * 4 + j) * VLD + pos]) = t[j];
        }
    };
    // S^T for the 32-key step s of the staged tile
    auto scores = [&](int buf, int s) {
        SACC acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0;
        if constexpr (F8) {
#pragma unroll
            for (int d = 0; d < DS; d += 2) {
                const v4i k0 = *reinterpret_cast<const v4i*>(&sK[buf][(s * 32 + ql) * KLD + d * 32 + hh * 16]);
                const v4i k1 = *reinterpret_cast<const v4i*>(&sK[buf][(s * 32 + ql) * KLD + (d + 1) * 32 + hh * 16]);
                acc = mfma_wide_f8(k0, k1, qf[d], qf[d + 1], acc);
            }
        } else {
#pragma unroll
            for (int d = 0; d < DS; ++d) {
                v4i kf = *reinterpret_cast<const v4i*>(&sK[buf][(s * 32 + ql) * KLD + d * 32 + hh * 16]);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf, qf[d], acc, 0, 0, 0);
            }
        }
        return acc;
    };

    // Both passes work in the log2 domain on the raw integer scores: p = 2^(acc * c2 - m2) with
    // c2 = d~ * log2(e).  The row maximum is taken on the integers (the scale is positive), masked
    // keys are replaced by a very negative integer (only in tiles that contain one), and in pass 2
    // the normaliser and 1/S_p are folded into the exponent, so a code costs one int->float
    // conversion, one fma, one exp2 and one saturating round-to-u8.
    const float c2 = (a.qk_scale_h ? a.qk_scale_h[h] : a.qk_scale) * 1.44269504088896340736f;
    constexpr int MASKED = -0x40000000;
    // first tile in which some key is hidden from some query of this wave (wave-uniform)
    int nvis_min = nvis;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nvis_min = min(nvis_min, __shfl_xor(nvis_min, o));

    // ---- the online variant: ONE sweep.  The codes of a 64-key tile are taken against the running row
    // maximum m (so the largest weight seen so far has code 255) and stay un-normalised; the integer sums
    // of a run of tiles with an unchanged maximum are kept in int32 (oi, li); only when some query of the
    // wave raises its maximum are they folded into the fp32 accumulators (of, lf) and everything gathered
    // so far is rescaled by 2^(m_old - m_new); the division by the sum of the weights happens once, at the end.  The matrix cores take
    // signed bytes: the fragment holds 127 - code (one XOR) and a second MFMA against the constant -127
    // removes the offset, so oi = -sum_k code_k v_k exactly, with no column sums and no extra vector work.
    if constexpr (ONLINE) {
        constexpr float L255 = 7.99435343685885793770f;           // log2(255)
        v16i oi[DS];
        v16f of[DS];
        uint32_t li = 0;
        float lf = 0.0f, m2 = -INFINITY;
#pragma unroll
        for (int c = 0; c < DS; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) { oi[c][r] = 0; of[c][r] = 0.0f; }
        const v4i cm127 = {(int)0x81818181u, (int)0x81818181u, (int)0x81818181u, (int)0x81818181u};
        if (ntiles > 0) { load_k(0); load_v(0); store_k(0); store_v(0); }
        __syncthreads();
        for (int tile = 0; tile < ntiles; ++tile) {
            const int buf = tile & 1;
            if (tile + 1 < ntiles) { load_k(tile + 1); load_v(tile + 1); }
            const bool edge = (tile + 1) * BKV > nvis_min;
            auto online_tile = [&](auto EDGE) {
                // the tile's maximum first; the scores are computed again for the codes (a second QK^T on
                // the idle matrix cores costs less than keeping 32 more registers alive)
                int imax = MASKED;
                auto tile_scores = [&](int s) {
                    v16i acc = scores(buf, s);
                    if constexpr (decltype(EDGE)::value) {
                        const int lim = nvis - (tile * BKV + s * 32 + hh * 4);  // key visible iff 8g + t < lim
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = ((r >> 2) * 8 + (r & 3)) < lim ? acc[r] : MASKED;
                    }
                    return acc;
                };
#pragma unroll
                for (int s = 0; s < BKV / 32; ++s) {
                    const v16i acc = tile_scores(s);
#pragma unroll
                    for (int r = 0; r < 16; ++r) imax = max(imax, acc[r]);
                }
                imax = max(imax, __shfl_xor(imax, 32));
                const float mn = imax > MASKED ? fmaxf(m2, (float)imax * c2) : m2;
                if (__builtin_amdgcn_ballot_w64(mn != m2) != 0) {                // wave-uniform
                    const float alpha = mn == m2 ? 1.0f : __builtin_amdgcn_exp2f(m2 - mn);
#pragma unroll
                    for (int c = 0; c < DS; ++c)
#pragma unroll
                        for (int r = 0; r < 16; ++r) { of[c][r] = (of[c][r] + (float)oi[c][r]) * alpha; oi[c][r] = 0; }
                    lf = (lf + (float)li) * alpha;
                    li = 0;
                    m2 = mn;
                }
                {
                    const float off = L255 - m2;
#pragma unroll
                    for (int s = 0; s < BKV / 32; ++s) {
                        const v16i acc = scores(buf, s);
                        const int lim = nvis - (tile * BKV + s * 32 + hh * 4);
                        v4i pf;
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            uint32_t w = 0;
#pragma unroll
                            for (int t = 0; t < 4; ++t) {
                                float e = __builtin_amdgcn_exp2f(fmaf((float)acc[4 * g + t], c2, off));
                                if constexpr (decltype(EDGE)::value) e = (g * 8 + t) < lim ? e : 0.0f;
                                w = __builtin_amdgcn_cvt_pk_u8_f32(e, t, w);
                            }
                            li = __builtin_amdgcn_sad_u8(w, 0u, li);             // + the four codes
                            pf[g] = (int)(w ^ 0x7f7f7f7fu);                      // 127 - code as signed bytes
                        }
#pragma unroll
                        for (int c = 0; c < DS; ++c) {
                            v4i vf = *reinterpret_cast<const v4i*>(&sVt[buf][(c * 32 + ql) * VLD + s * 32 + hh * 16]);
                            oi[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, pf, oi[c], 0, 0, 0);
                            oi[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, cm127, oi[c], 0, 0, 0);
                        }
                    }
                }
            };
            if (!wact) {} else if (edge) online_tile(std::true_type{}); else online_tile(std::false_type{});
            if (tile + 1 < ntiles) { store_k(buf ^ 1); store_v(buf ^ 1); }
            __syncthreads();
        }
        if (qi >= a.Sq) return;
        float l = lf + (float)li;
        l += __shfl_xor(l, 32);
        // oi / of hold MINUS the weighted sums; y = O / L * c[j] / S_p
        const float inv = l > 0.0f ? __fdiv_rn(-1.0f, l * a.p_scale) : 0.0f;
        const int64_t orow = ((int64_t)b * a.Sq + qi) * a.ldo + (int64_t)h * DH;
#pragma unroll
        for (int c = 0; c < DS; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int e0 = c * 32 + g * 8 + hh * 4;
                float y[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float sc = a.scale_is_scalar ? a.out_col_scale[0] : a.out_col_scale[h * DH + e0 + t];
                    y[t] = (of[c][4 * g + t] + (float)oi[c][4 * g + t]) * inv * sc;
                    if (qi >= qlim) y[t] = 0.0f;              // padded query: zeros
                }
                if (ODT == HERO_I8) {
                    *reinterpret_cast<uint32_t*>((int8_t*)a.out + orow + e0) = quant4_sat(y[0], y[1], y[2], y[3]);
                } else {
                    v2i w = {(int)pack2_hp<ODT>(y[0], y[1]), (int)pack2_hp<ODT>(y[2], y[3])};
                    *reinterpret_cast<v2i*>((uint16_t*)a.out + orow + e0) = w;
                }
            }
        return;
    }

    // ---- pass 1: row max and row sum ------------------------------------------------------------
    // One maximum per tile, or per 32 keys in tiles that hide some (a block that is hidden altogether is left out); the two lanes of a query exchange
    // theirs by v_permlane32_swap.  us, an exchange through LDS every 32 keys -> this: 8 x 32 x 2048 x 128 causal 394 -> 387, E4M3 332 -> 324, 2 x 32 x 2048
    // without a mask 178 -> 174, 150 -> 145, 8 x 32 x 200 behind 1300 keys 76 -> 74, 62.6 -> 59.9, 8 x 16 x 1000 x 64 64 -> 63, 58.2 -> 56.5, 3 x 32 x 290 causal 20.6 -> 20.2.
    // (64 keys to a maximum in every tile: 21.2 there, 17 x 32 x 92 16.8 -> 17.6.  Maxima of a lane's own keys, joined behind the last tile: another 2 %, but their
    // factors' errors showed where all probabilities are equal.)
    float m2 = -INFINITY, l = 0.0f;           // running max (log2 domain) and sum of 2^(a2 - m2), this lane's keys
    constexpr float FMASKED = -3.0e38f;       // E4M3 scores are floats: the mask value of that variant
    if (ntiles > 0) { load_k(0); store_k(0); }
    __syncthreads();
    for (int tile = 0; tile < ntiles; ++tile) {
        const int buf = tile & 1;
        if (tile + 1 < ntiles) load_k(tile + 1);
        const bool edge = (tile + 1) * BKV > nvis_min;
        auto pass1_tile = [&](auto EDGE) {
            const int lim = nvis - (tile * BKV + hh * 4);                       // key visible iff 32s + 8g + t < lim
            constexpr int G = decltype(EDGE)::value ? 1 : BKV / 32;             // 32-key blocks to a maximum
#pragma unroll
            for (int s0 = 0; s0 < BKV / 32; s0 += G) {
                SACC acc[G];
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    acc[s] = scores(buf, s0 + s);
                    if constexpr (decltype(EDGE)::value)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            if constexpr (F8) acc[s][r] = s0 * 32 + (r >> 2) * 8 + (r & 3) < lim ? acc[s][r] : FMASKED;
                            else acc[s][r] = s0 * 32 + (r >> 2) * 8 + (r & 3) < lim ? acc[s][r] : MASKED;
                        }
                }
                auto smax = acc[0][0];
#pragma unroll
                for (int s = 0; s < G; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r) smax = max(smax, acc[s][r]);
                smax = pair_max(smax);
                if (F8 ? (float)smax > FMASKED : (int)smax > MASKED) {          // same decision in both lanes of a query
                    const float mn = fmaxf(m2, (float)smax * c2);
                    float sum = 0.0f;
#pragma unroll
                    for (int s = 0; s < G; ++s) {
                        float part = 0.0f;
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            float e = __builtin_amdgcn_exp2f(fmaf((float)acc[s][r], c2, -mn));
                            // (a hidden key counts for nothing at any scale of the scores, also where c2 brings the mask's value back into range)
                            if constexpr (decltype(EDGE)::value) e = s0 * 32 + (r >> 2) * 8 + (r & 3) < lim ? e : 0.0f;
                            part += e;
                        }
                        sum += part;
                    }
                    l = fmaf(l, __builtin_amdgcn_exp2f(m2 - mn), sum);
                    m2 = mn;
                }
            }
        };
        if (!wact) {} else if (edge) pass1_tile(std::true_type{}); else pass1_tile(std::false_type{});
        if (tile + 1 < ntiles) store_k(buf ^ 1);
        __syncthreads();
    }
    l += __shfl_xor(l, 32);
    // exponent offset of pass 2: 2^(acc*c2 - m2) / l / S_p = 2^(acc*c2 + off); a row that saw no key gets codes 0
    const float off = l > 0.0f ? -m2 - __log2f(l * a.p_scale) : -INFINITY;

    // ---- pass 2: codes and PV --------------------------------------------------------------------
    SACC o[DS];
    int csum[DS];                                         // this wave's share of colsum(V): channel 32c + ql, keys of half hh
#pragma unroll
    for (int c = 0; c < DS; ++c) {
        csum[c] = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) o[c][r] = 0;
    }
    if (ntiles > 0) { load_k(0); load_v(0); store_k(0); store_v(0); }
    __syncthreads();
    for (int tile = 0; tile < ntiles; ++tile) {
        const int buf = tile & 1;
        if (tile + 1 < ntiles) { load_k(tile + 1); load_v(tile + 1); }
        const bool edge = (tile + 1) * BKV > nvis_min;
        auto pass2_tile = [&](auto EDGE) {
            if constexpr (F8) {
                // codes of the whole 64-key tile first (two 32-key steps), then ONE K = 64 matrix instruction per
                // 32 channels: e4m3(min(2^(acc*c2 + off), 448)), two codes per conversion instruction
                v4i pf[BKV / 32];
#pragma unroll
                for (int s = 0; s < BKV / 32; ++s) {
                    const v16f acc = scores(buf, s);
                    const int lim = nvis - (tile * BKV + s * 32 + hh * 4);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float e[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            e[t] = fminf(__builtin_amdgcn_exp2f(fmaf(acc[4 * g + t], c2, off)), 448.0f);
                            if constexpr (decltype(EDGE)::value) e[t] = (g * 8 + t) < lim ? e[t] : 0.0f;
                        }
                        int w = __builtin_amdgcn_cvt_pk_fp8_f32(e[0], e[1], 0, false);
                        pf[s][g] = __builtin_amdgcn_cvt_pk_fp8_f32(e[2], e[3], w, true);
                    }
                }
#pragma unroll
                for (int c = 0; c < DS; ++c) {
                    const v4i v0 = *reinterpret_cast<const v4i*>(&sVt[buf][(c * 32 + ql) * VLD + hh * 16]);
                    const v4i v1 = *reinterpret_cast<const v4i*>(&sVt[buf][(c * 32 + ql) * VLD + 32 + hh * 16]);
                    o[c] = mfma_wide_f8(v0, v1, pf[0], pf[1], o[c]);
                }
            } else {
#pragma unroll
            for (int s = 0; s < BKV / 32; ++s) {
                v16i acc = scores(buf, s);
                const int lim = nvis - (tile * BKV + s * 32 + hh * 4);          // key visible iff 8g + t < lim
                v4i pf;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint32_t w = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float e = __builtin_amdgcn_exp2f(fmaf((float)acc[4 * g + t], c2, off));
                        if constexpr (decltype(EDGE)::value) e = (g * 8 + t) < lim ? e : 0.0f;
                        w = __builtin_amdgcn_cvt_pk_u8_f32(e, t, w);     // sat_[0,255](rne(.)) into byte t
                    }
                    pf[g] = (int)(w ^ 0x80808080u);                         // codes - 128 as signed bytes
                }
#pragma unroll
                for (int c = 0; c < DS; ++c) {
                    v4i vf = *reinterpret_cast<const v4i*>(&sVt[buf][(c * 32 + ql) * VLD + s * 32 + hh * 16]);
                    o[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, pf, o[c], 0, 0, 0);
                    if (((tile * (BKV / 32) + s) & 3) == wave) {         // wave-uniform: one wave per 32-key step
#pragma unroll
                        for (int w = 0; w < 4; ++w) csum[c] = __builtin_amdgcn_sdot4(vf[w], 0x01010101, csum[c], false);
                    }
                }
            }
            }
        };
        if (!wact) {
            if constexpr (!F8) {                              // only the wave's share of the column sums
#pragma unroll
                for (int s = 0; s < BKV / 32; ++s)
                    if (((tile * (BKV / 32) + s) & 3) == wave) {
#pragma unroll
                        for (int c = 0; c < DS; ++c) {
                            const v4i vf = *reinterpret_cast<const v4i*>(&sVt[buf][(c * 32 + ql) * VLD + s * 32 + hh * 16]);
#pragma unroll
                            for (int w = 0; w < 4; ++w) csum[c] = __builtin_amdgcn_sdot4(vf[w], 0x01010101, csum[c], false);
                        }
                    }
            }
        } else if (edge) pass2_tile(std::true_type{}); else pass2_tile(std::false_type{});
        if (tile + 1 < ntiles) { store_k(buf ^ 1); store_v(buf ^ 1); }
        __syncthreads();
    }

    // ---- colsum(V) of the block: every wave adds its share per channel (the loop's last barrier has
    // released the K buffers, which now hold the sums)
    int* const colsum = reinterpret_cast<int*>(&sK[0][0]);
    if constexpr (!F8) {
        for (int c = tid; c < DH; c += 256) colsum[c] = 0;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < DS; ++c) atomicAdd(&colsum[c * 32 + ql], csum[c]);
        __syncthreads();
    }

    // ---- output: lane holds query ql, channels 32c + 8g + 4hh + t -----------------------------------
    if (qi >= a.Sq) return;
    const int64_t orow = ((int64_t)b * a.Sq + qi) * a.ldo + (int64_t)h * DH;
#pragma unroll
    for (int c = 0; c < DS; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e0 = c * 32 + g * 8 + hh * 4;
            float y[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float sc = a.scale_is_scalar ? a.out_col_scale[0] : a.out_col_scale[h * DH + e0 + t];
                if constexpr (F8) y[t] = o[c][4 * g + t] * sc;
                else y[t] = (float)(o[c][4 * g + t] + 128 * colsum[e0 + t]) * sc;
                if (qi >= qlim) y[t] = 0.0f;                  // padded query: zeros
            }
            if (ODT == HERO_I8) {
                *reinterpret_cast<uint32_t*>((int8_t*)a.out + orow + e0) = quant4_sat(y[0], y[1], y[2], y[3]);
            } else if (ODT == HERO_F8E4M3) {
                *reinterpret_cast<uint32_t*>((int8_t*)a.out + orow + e0) = fp8x4_sat(y[0], y[1], y[2], y[3]);
            } else {
                v2i w = {(int)pack2_hp<ODT>(y[0], y[1]), (int)pack2_hp<ODT>(y[2], y[3])};
                *reinterpret_cast<v2i*>((uint16_t*)a.out + orow + e0) = w;
            }
        }
}

// ------------------------------------------------------------------------------------------
// Up to 512 keys of 64 channels (the encoders): one pass.  The core of the two-pass kernel above takes 15 vector slots per score, 8 of
// them the two quarter-rate exp2, because a block's scores do not survive until the row sum is known.  Here they do: a wave takes 16 queries
// at a time (v_mfma_*_16x16x64: lane l holds, for query l % 16, the keys 16 s + 4 (l / 16) + t of every 16-key step s), so that the
// scores of up to 256 keys, later their exponentials, stay in 16 registers per 64 keys, and a code is one multiplication and one
// packing conversion away: 10 slots per score (conversion, half a maximum, fma, exp2 (4), sum, product, packing conversion; counted with
// staging, masks and results 13.4 instructions or 16.4 slots per score, the two-pass kernel 15.0 or 21).  The
// codes of a 64-key tile are the PV operand as they stand, V being staged transposed with its keys in the same order.
// A block owns 128 queries of one (batch, head), in four groups of 32 (two sets of 16 each), and stages all of K (direct to LDS) and
// V once.  KW waves share a group's keys: one up to 256 keys, then no barrier follows; two beyond (all scores of 512 keys in one wave's
// registers leave two waves per SIMD, and 32 x 16 x 512 took 73 us, the two-pass kernel 69): the halves' maxima and sums meet in LDS,
// and each wave ends with half of the channels.  A hidden key is left out by the size of its masked score alone, which asks for a scale of
// KEEP_MIN_QK or more; the two-pass kernel serves the others (selecting the exponentials here made the 256- and 512-key forms spill).
// The offset of the unsigned codes is removed by a second matrix instruction as in the online variant, so o = -sum code * v.  The vector
// ALU is the largest term (32 x 16 x 512 padded: 58 % of the cycles with exp2 weighted, the matrix pipe 11 %); four waves per SIMD.
// ------------------------------------------------------------------------------------------
// (2^30 - 2^20) * 2^-23 * log2(e) = 184: with the largest score, 64 * 128 * 128, on either side of the mask's value a hidden key's
// exponential, below 2^-149, is 0 (E4M3: 3e38 beside 64 * 448 * 448)
constexpr float KEEP_MIN_QK = 0x1p-23f;

template <int ODT, int FMT, int NT, int KW>
__global__ __launch_bounds__(256 * KW, 4) void int8_attn_keep_kernel(AttnArgs a) {
    constexpr bool F8 = FMT == HERO_F8E4M3;
    using V4 = typename std::conditional<F8, v4f, v4i>::type;
    constexpr int DH = 64, NC = DH / 16, VLD = NT * 64, HG = 2, NW = 4 * KW, NH = NT / KW;       // NH: tiles of a wave
    static_assert((NT == 2 || NT == 4 || NT == 8) && NH <= 4, "score registers");
    __shared__ __attribute__((aligned(1024))) int8_t sK[NT * 64 * DH];       // 16-byte chunk c of key k at c ^ ((k >> 2) & 3)
    // V transposed: key 64 i + 16 t + 4 g + j of a channel is byte 4 t + j of its 16-byte chunk 4 i + g, and chunk c of channel h lies at
    // c ^ ((h ^ (h >> 4 << 2)) & 15): 16 channels' reads, and the transposed stores, fall into different banks
    constexpr int VX = NT * 4 < 16 ? NT * 4 - 1 : 15;
    __shared__ __attribute__((aligned(1024))) int8_t sVt[DH * VLD];
    __shared__ __attribute__((aligned(16))) float scale[DH];
    __shared__ float stat[KW == 1 ? 1 : 4 * KW * 32];                        // [group][half]: row maximum and row sum of 16 queries
    __shared__ __attribute__((aligned(16))) V4 xch[KW == 1 ? 1 : 4 * 2 * 64];     // [group][2 channel groups][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave & 3, kh = wave >> 2;
    const int ql = lane & 15, gq = lane >> 4;
    // blocks: order, rotation and the padding rule are those of the two-pass kernel
    const int nqb = (a.Sq + BQ - 1) / BQ;
    const int slot = blockIdx.x / 8, grp = (slot / (HG * nqb)) * 8 + (blockIdx.x % 8), within = slot % (HG * nqb);
    const int bh = grp * HG + within / nqb;
    if (bh >= a.B * a.H) return;
    const uint32_t rot = ((uint32_t)(slot / (HG * nqb)) * 2654435761u) >> 20;
    const int qb = (int)((within % nqb + rot) % (uint32_t)nqb);
    const int b = bh / a.H, h = bh % a.H, q0 = qb * BQ;
    const int len = a.kv_len ? min(max(a.kv_len[b], 0), a.Skv) : a.Skv;
    const int shift = len - a.Sq;
    const bool causal = a.mask == HERO_MASK_CAUSAL;
    const int qlim = (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) ? len : a.Sq;
    const int kmax = max(causal ? min(len, min(q0 + BQ, a.Sq) + shift) : len, 0);
    if (q0 >= qlim) { zero_rows<DH, ODT>(a, b, h, q0, 256 * KW); return; }       // (before any barrier: the whole block leaves)
    const int ntiles = (kmax + 63) / 64;
    const int w0 = q0 + ((group + slot) & 3) * 32;                           // this wave's queries
    v4i qf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
        qf[s] = *reinterpret_cast<const v4i*>(a.q + (int64_t)b * a.qs[0] + (int64_t)min(w0 + s * 16 + ql, a.Sq - 1) * a.qs[1] + (int64_t)h * a.qs[2] + gq * 16);
    const int8_t* const kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2];
    const int8_t* const vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2];
    {
        // K: a load is 16 rows; lane l brings the chunk that belongs at position l % 4 of row l / 4.  V: wave w takes the tiles w, w + NW;
        // a lane holds 16 channels of four keys.  Rows past the last key repeat it (masked below).
        const int kr = lane >> 2, kc = ((lane & 3) ^ ((kr >> 2) & 3)) * 16;
        const uint32_t kdst = __builtin_amdgcn_readfirstlane(hero_gemm::lds_offset(sK));
        for (int u = wave; u < ntiles * 4; u += NW)
            hero_gemm::dma16(kbase + (int64_t)min(u * 16 + kr, a.Skv - 1) * a.ks[1] + kc, kdst + u * 16 * DH);
        constexpr int VU = (NT + NW - 1) / NW;
        v4i rv[VU][4];
        const int kg = lane >> 2, c4 = lane & 3;                             // four-key group of the tile, 16-channel group
#pragma unroll
        for (int u = 0; u < VU; ++u)
            if (u * NW + wave < ntiles)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    rv[u][i] = *reinterpret_cast<const v4i*>(vbase + (int64_t)min((u * NW + wave) * 64 + kg * 4 + i, a.Skv - 1) * a.vs[1] + c4 * 16);
#pragma unroll
        for (int u = 0; u < VU; ++u)
            if (u * NW + wave < ntiles) {
                const int chunk = (u * NW + wave) * 4 + (kg & 3);
#pragma unroll
                for (int w = 0; w < 4; ++w) {                                // 4 x 4 byte transposes
                    const uint32_t d0 = rv[u][0][w], d1 = rv[u][1][w], d2 = rv[u][2][w], d3 = rv[u][3][w];
                    const uint32_t lo01 = __builtin_amdgcn_perm(d1, d0, 0x05010400u), hi01 = __builtin_amdgcn_perm(d1, d0, 0x07030602u);
                    const uint32_t lo23 = __builtin_amdgcn_perm(d3, d2, 0x05010400u), hi23 = __builtin_amdgcn_perm(d3, d2, 0x07030602u);
                    const uint32_t tr[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                            __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<uint32_t*>(sVt + (c4 * 16 + w * 4 + j) * VLD + ((chunk ^ ((w * 4 + j) ^ (c4 << 2))) & VX) * 16 +
                                                     (chunk & ~VX) * 16 + (kg >> 2) * 4) = tr[j];
                }
            }
        if (tid < DH) scale[tid] = a.out_col_scale[a.scale_is_scalar ? 0 : h * DH + tid];
        __builtin_amdgcn_s_waitcnt(hero_gemm::vmcnt_imm(0));                 // the direct loads are not the compiler's to wait for
        __syncthreads();
    }
    const float c2 = a.qk_scale * 1.44269504088896340736f;
    constexpr int MASKED = -0x40000000;
    constexpr float FMASKED = -3.0e38f;
    constexpr typename std::conditional<F8, float, int>::type HIDDEN = (typename std::conditional<F8, float, int>::type)(F8 ? FMASKED : (float)MASKED);
    auto mfma = [](v4i x, v4i y, V4 c) {
        if constexpr (F8) {                                                  // the upper half of K is zeros
            const v8i x8 = {x[0], x[1], x[2], x[3], 0, 0, 0, 0}, y8 = {y[0], y[1], y[2], y[3], 0, 0, 0, 0};
            return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x8, y8, c, 0, 0, 0, 0, 0, 0);
        } else return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, c, 0, 0, 0);
    };
    // a wave's i-th tile is KW i + kh.  Chunk 4 t + gq of channel 16 c + ql is at (gq ^ ql) ^ 4 (t ^ c) within its 16 (8): one of four (two)
    // addresses per lane
    constexpr int VK = VX == 15 ? 4 : 2;
    const int8_t* const kf = sK + (kh * 64 + ql) * DH + ((gq ^ ((ql >> 2) & 3)) << 4);       // + 16 DH per step
    int va[VK];
#pragma unroll
    for (int k = 0; k < VK; ++k) va[k] = ql * VLD + (((gq ^ ql ^ ((k ^ kh) << 2)) & VX) << 4);
#pragma nounroll
    for (int set = 0; set < 2; ++set) {
        const v4i qs = set ? qf[1] : qf[0];
        const int qfirst = w0 + set * 16, qi = qfirst + ql;
        if (KW == 1 && qfirst >= a.Sq) break;                                    // (two halves meet at barriers: all sets run)
        const int64_t orow = ((int64_t)b * a.Sq + qi) * a.ldo + (int64_t)h * DH;
        const int nvis = max(causal ? min(len, qi + shift + 1) : len, 0);
        // tiles this set sees, and the first of them that hides a key from one of its queries (both uniform)
        const int last = max(causal ? min(len, min(qfirst + 16, a.Sq) + shift) : len, 0);
        const int nt = qfirst < qlim ? (last + 63) / 64 : 0, edge = (max(causal ? min(len, qfirst + shift + 1) : len, 0)) / 64;
        const int n = KW == 1 ? nt : (nt + 1 - kh) / 2;                          // this wave's tiles
        V4 o[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) o[c] = V4{0, 0, 0, 0};
        // `meet` turns this wave's maximum (log2 domain) and sum into the factor of its exponentials
        auto meet = [&](float m2, float l) -> float {
            if constexpr (KW == 1) return l > 0.0f ? __fdiv_rn(1.0f, l * a.p_scale) : 0.0f;       // a row that saw no key gets codes 0
            else {
                float* const st = stat + group * (KW * 32);
                if (gq == 0) { st[kh * 32 + ql] = m2; st[kh * 32 + 16 + ql] = l; }
                __syncthreads();
                const float mo = st[(kh ^ 1) * 32 + ql], lo = st[(kh ^ 1) * 32 + 16 + ql], m = fmaxf(m2, mo);
                if (!(m > -INFINITY)) return 0.0f;
                const float f = __builtin_amdgcn_exp2f(m2 - m);
                const float sum = kh == 0 ? fmaf(l, f, lo * __builtin_amdgcn_exp2f(mo - m)) : fmaf(lo, __builtin_amdgcn_exp2f(mo - m), l * f);
                return sum > 0.0f ? __fdiv_rn(f, sum * a.p_scale) : 0.0f;       // (E4M3: a row with a NaN among its scores, as one wave's)
            }
        };
        auto run = [&](auto NTILE) {
            constexpr int N = decltype(NTILE)::value;
            V4 sc[N][4];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int t = KW * i + kh;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    sc[i][s] = mfma(*reinterpret_cast<const v4i*>(kf + (KW * i * 4 + s) * 16 * DH), qs, V4{0, 0, 0, 0});
                if (t >= edge) {
                    const int lim = nvis - t * 64 - gq * 4;                      // key visible iff 16 s + j < lim
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int j = 0; j < 4; ++j) sc[i][s][j] = 16 * s + j < lim ? sc[i][s][j] : HIDDEN;
                }
            }
            auto smax = sc[0][0][0];
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int s = 0; s < 4; ++s) smax = max(max(max(max(smax, sc[i][s][0]), sc[i][s][1]), sc[i][s][2]), sc[i][s][3]);
            smax = max(smax, __shfl_xor(smax, 16));
            smax = max(smax, __shfl_xor(smax, 32));
            const bool any = F8 ? (float)smax > FMASKED : (int)smax > MASKED;    // the same in all lanes of a query
            const float m2 = any ? (float)smax * c2 : 0.0f;                      // (nothing visible: every exponential is 0)
            float l = 0.0f;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float lt = 0.0f;
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float e = __builtin_amdgcn_exp2f(fmaf((float)sc[i][s][j], c2, -m2));
                        if constexpr (F8) sc[i][s][j] = e; else sc[i][s][j] = __float_as_int(e);
                        lt += e;
                    }
                l += lt;
            }
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const float r = meet(any ? m2 : -INFINITY, any ? l : 0.0f);
            auto ev = [&](int i, int s, int j) { if constexpr (F8) return sc[i][s][j]; else return __int_as_float(sc[i][s][j]); };
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v4i pf;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if constexpr (F8) {
                        const int w = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(ev(i, s, 0) * r, 448.0f), fminf(ev(i, s, 1) * r, 448.0f), 0, false);
                        pf[s] = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(ev(i, s, 2) * r, 448.0f), fminf(ev(i, s, 3) * r, 448.0f), w, true);
                    } else {
                        uint32_t w = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) w = __builtin_amdgcn_cvt_pk_u8_f32(ev(i, s, j) * r, j, w);
                        pf[s] = (int)(w ^ 0x7f7f7f7fu);                          // 127 - code as signed bytes
                    }
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const v4i v = *reinterpret_cast<const v4i*>(sVt + va[(c ^ (KW * i)) & (VK - 1)] + c * 16 * VLD + (KW * i / VK) * VK * 64);
                    o[c] = mfma(v, pf, o[c]);
                    if constexpr (!F8) o[c] = mfma(v, v4i{(int)0x81818181u, (int)0x81818181u, (int)0x81818181u, (int)0x81818181u}, o[c]);    // * -127
                }
            }
        };
        if (n == 1) run(std::integral_constant<int, 1>{});
        else if (n == 2) run(std::integral_constant<int, 2>{});
        else if (NH > 2 && n == 3) run(std::integral_constant<int, (NH > 2 ? 3 : 1)>{});
        else if (NH > 2 && n == 4) run(std::integral_constant<int, (NH > 2 ? 4 : 1)>{});
        else meet(-INFINITY, 0.0f);
        if constexpr (KW == 2) {
            // halves of the keys -> halves of the channels
            V4* const x = xch + group * 128 + lane;
            if (kh == 1) { x[0] = o[0]; x[64] = o[1]; }
            __syncthreads();
            if (kh == 0) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const V4 p = x[c * 64];
#pragma unroll
                    for (int t = 0; t < 4; ++t) o[c][t] += p[t];
                    x[c * 64] = o[2 + c];
                }
            }
            __syncthreads();
            if (kh == 1) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const V4 p = x[c * 64];
#pragma unroll
                    for (int t = 0; t < 4; ++t) o[c][t] = p[t] + o[2 + c][t];
                }
            }
        }
        if (qi >= a.Sq) continue;
#pragma unroll
        for (int c = 0; c < NC / KW; ++c) {
            const int e0 = (kh * 2 + c) * 16 + gq * 4;
            const v4f scl = *reinterpret_cast<const v4f*>(scale + e0);
            float y[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                y[t] = (F8 ? (float)o[c][t] : (float)-o[c][t]) * scl[t];
                if (qi >= qlim) y[t] = 0.0f;                                     // padded query: zeros
            }
            if (ODT == HERO_I8) *reinterpret_cast<uint32_t*>((int8_t*)a.out + orow + e0) = quant4_sat(y[0], y[1], y[2], y[3]);
            else if (ODT == HERO_F8E4M3) *reinterpret_cast<uint32_t*>((int8_t*)a.out + orow + e0) = fp8x4_sat(y[0], y[1], y[2], y[3]);
            else *reinterpret_cast<v2i*>((uint16_t*)a.out + orow + e0) = v2i{(int)pack2_hp<ODT>(y[0], y[1]), (int)pack2_hp<ODT>(y[2], y[3])};
        }
    }
}

// ------------------------------------------------------------------------------------------
// Few query blocks (a short sentence, a prompt chunk of few users): the kernel above runs as one serial chain of two
// passes over the keys per block of 128 queries, on as many CUs as there are blocks.  Here a block owns 32 queries and its
// NW waves split the KEYS: wave w takes the 32-key steps w, w + NW, .., with K fragments straight from memory, V transposed
// through LDS of its own and no barrier inside a pass.  The waves' row maxima and sums meet in LDS between the passes, their
// PV sums (exact integers; E4M3: fp32, added in the order of the waves) at the end.  Four times the K / V reads from the
// L2 for a quarter of the chain; bound by latency.  Same codes by the same formulas as above; the offset of the unsigned codes is
// removed by a second matrix instruction as in the online variant, so o = -sum code * v.
// ------------------------------------------------------------------------------------------
template <int DH, int ODT, int FMT, int NW, int CW>
__global__ __launch_bounds__(64 * NW) void int8_attn_split_kernel(AttnArgs a) {
    constexpr bool F8 = FMT == HERO_F8E4M3;
    using SACC = typename std::conditional<F8, v16f, v16i>::type;
    using ST = typename std::conditional<F8, float, int>::type;
    using V4 = typename std::conditional<F8, v4f, v4i>::type;
    constexpr int SQ = 32, SK = 32, VLD = SK + 16, DS = DH / 32, TLD = 36;
    // V: a unit is 4 keys x CW channels; with 16 of them a load is 128 bits, and every 16 channels lie 32 bytes further on (the stores of eight
    // units' same channel fall into different banks that way; GPT layer, 2 x 301 tokens behind 900 keys, 253.3 -> 251.2 us; launch_split has the rule).
    static_assert(CW == 4 || (CW == 16 && DH >= 128), "64 channels have half as many units of 16 as a wave has lanes");
    constexpr int VU = (SK / 4) * (DH / CW) / 64, VPAD = CW == 16 ? 32 : 0, VT = DH * VLD + DH / 16 * VPAD;
    __shared__ __attribute__((aligned(16))) int8_t pool[NW * VT > NW * SQ * TLD * 4 ? NW * VT : NW * SQ * TLD * 4];
    __shared__ float sm[NW][SQ], sl[NW][SQ];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hh = lane >> 5, ql = lane & 31;
    constexpr int HG = DH >= 128 ? 1 : 128 / DH;                 // block order: as above, per 32 queries
    const int nqb = (a.Sq + SQ - 1) / SQ;
    const int slot = blockIdx.x / 8, grp = (slot / (HG * nqb)) * 8 + (blockIdx.x % 8), within = slot % (HG * nqb);
    const int bh = grp * HG + within / nqb;
    if (bh >= a.B * a.H) return;
    const int b = bh / a.H, h = bh % a.H, q0 = (within % nqb) * SQ;
    const int len = a.kv_len ? min(max(a.kv_len[b], 0), a.Skv) : a.Skv;
    const int shift = len - a.Sq, qi = q0 + ql;
    int nvis = len, kmax = len;
    if (a.mask == HERO_MASK_CAUSAL) {
        nvis = min(len, qi + shift + 1);
        kmax = min(len, min(q0 + SQ, a.Sq) + shift);
    }
    nvis = max(nvis, 0);
    const int qlim = (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) ? len : a.Sq;      // padded positions ask nothing
    const int nsteps = q0 >= qlim ? 0 : (max(kmax, 0) + SK - 1) / SK;                  // block-uniform
    v4i qf[DS];
    {
        const int8_t* qp = a.q + (int64_t)b * a.qs[0] + (int64_t)min(qi, a.Sq - 1) * a.qs[1] + (int64_t)h * a.qs[2];
#pragma unroll
        for (int d = 0; d < DS; ++d) qf[d] = *reinterpret_cast<const v4i*>(qp + d * 32 + hh * 16);
    }
    const int8_t* const kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2] + hh * 16;
    const int8_t* const vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2];
    int8_t* const sv = pool + wave * VT;
    v4i k0[DS], k1[DS];                                          // two steps in flight in pass 1
    int rv[VU][4][CW / 4];
    auto load_k = [&](v4i (&kf)[DS], int step) {                                // lane: key row ql of the step, its 16-byte pieces of half hh
        const int8_t* p = kbase + (int64_t)min(step * SK + ql, a.Skv - 1) * a.ks[1];
#pragma unroll
        for (int d = 0; d < DS; ++d) kf[d] = *reinterpret_cast<const v4i*>(p + d * 32);
    };
    // eight consecutive lanes read 128 (32) contiguous bytes of one key row
    auto load_v = [&](int step) {
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int kg = (lane >> 3) & 7, cg = (lane & 7) + 8 * u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int8_t* p = vbase + (int64_t)min(step * SK + kg * 4 + i, a.Skv - 1) * a.vs[1] + cg * CW;
                if constexpr (CW == 16) {
                    const v4i w = *reinterpret_cast<const v4i*>(p);
#pragma unroll
                    for (int c = 0; c < 4; ++c) rv[u][i][c] = w[c];
                } else rv[u][i][0] = *reinterpret_cast<const int*>(p);
            }
        }
    };
    auto store_v = [&]() {
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int kg = (lane >> 3) & 7, cg = (lane & 7) + 8 * u;
            const int pos = (kg & 1) * 16 + (kg >> 1) * 4;       // the key order of the PV fragment (see the kernel above)
#pragma unroll
            for (int c = 0; c < CW / 4; ++c) {
                const uint32_t d0 = rv[u][0][c], d1 = rv[u][1][c], d2 = rv[u][2][c], d3 = rv[u][3][c];
                const uint32_t lo01 = __builtin_amdgcn_perm(d1, d0, 0x05010400u), hi01 = __builtin_amdgcn_perm(d1, d0, 0x07030602u);
                const uint32_t lo23 = __builtin_amdgcn_perm(d3, d2, 0x05010400u), hi23 = __builtin_amdgcn_perm(d3, d2, 0x07030602u);
                const uint32_t t[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                       __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<uint32_t*>(&sv[(cg * CW + c * 4 + j) * VLD + (VPAD ? cg * VPAD : 0) + pos]) = t[j];
            }
        }
    };
    auto scores = [&](const v4i (&kf)[DS]) {
        SACC acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0;
        if constexpr (F8) {
#pragma unroll
            for (int d = 0; d < DS; d += 2) acc = mfma_wide_f8(kf[d], kf[d + 1], qf[d], qf[d + 1], acc);
        } else {
#pragma unroll
            for (int d = 0; d < DS; ++d) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[d], qf[d], acc, 0, 0, 0);
        }
        return acc;
    };
    const float c2 = a.qk_scale * 1.44269504088896340736f;
    constexpr int MASKED = -0x40000000;
    constexpr float FMASKED = -3.0e38f;

    int nvis_min = nvis;                                         // the first step with a key hidden from some query
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) nvis_min = min(nvis_min, __shfl_xor(nvis_min, o));

    // ---- pass 1: this wave's row maxima and sums
    float m2 = -INFINITY, l = 0.0f;
    auto stats = [&](v4i (&kf)[DS], int step) {
        SACC acc = scores(kf);
        if (step + 2 * NW < nsteps) load_k(kf, step + 2 * NW);
        const bool edge = (step + 1) * SK > nvis_min;
        const int lim = nvis - (step * SK + hh * 4);             // key visible iff 8g + t < lim
        if (edge) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if constexpr (F8) acc[r] = ((r >> 2) * 8 + (r & 3)) < lim ? acc[r] : FMASKED;
                else acc[r] = ((r >> 2) * 8 + (r & 3)) < lim ? acc[r] : MASKED;
            }
        }
        auto smax = acc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) smax = max(smax, acc[r]);
        smax = pair_max(smax);
        if (F8 ? (float)smax > FMASKED : (int)smax > MASKED) {
            const float mn = fmaxf(m2, (float)smax * c2);
            float e[16], sum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(fmaf((float)acc[r], c2, -mn));
            if (edge) {                                          // (as above: a hidden key counts for nothing)
#pragma unroll
                for (int r = 0; r < 16; ++r) e[r] = ((r >> 2) * 8 + (r & 3)) < lim ? e[r] : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += e[r];
            l = fmaf(l, __builtin_amdgcn_exp2f(m2 - mn), sum);
            m2 = mn;
        }
    };
    if (wave < nsteps) load_k(k0, wave);
    if (wave + NW < nsteps) load_k(k1, wave + NW);
    for (int step = wave; step < nsteps; step += 2 * NW) {
        stats(k0, step);
        if (step + NW < nsteps) stats(k1, step + NW);
    }
    if (wave < nsteps) { load_k(k0, wave); load_v(wave); }       // in flight while the waves meet
    l += __shfl_xor(l, 32);
    if (hh == 0) { sm[wave][ql] = m2; sl[wave][ql] = l; }
    __syncthreads();
    float M = sm[0][ql];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm[w][ql]);
    float L = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { const float lw = sl[w][ql]; if (lw > 0.0f) L = fmaf(lw, __builtin_amdgcn_exp2f(sm[w][ql] - M), L); }
    const float off = L > 0.0f ? -M - __log2f(L * a.p_scale) : -INFINITY;

    // ---- pass 2: codes and PV
    SACC o[DS];
#pragma unroll
    for (int c = 0; c < DS; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[c][r] = 0;
    const v4i cm127 = {(int)0x81818181u, (int)0x81818181u, (int)0x81818181u, (int)0x81818181u}, zero = {0, 0, 0, 0};
    for (int step = wave; step < nsteps; step += NW) {
        store_v();
        const SACC acc = scores(k0);
        if (step + NW < nsteps) { load_k(k0, step + NW); load_v(step + NW); }
        v4i pf;
        auto codes = [&](auto EDGE) {
            const int lim = nvis - (step * SK + hh * 4);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float e[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    e[t] = __builtin_amdgcn_exp2f(fmaf((float)acc[4 * g + t], c2, off));
                    if constexpr (decltype(EDGE)::value) e[t] = (g * 8 + t) < lim ? e[t] : 0.0f;
                }
                if constexpr (F8) {
                    const int w = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(e[0], 448.0f), fminf(e[1], 448.0f), 0, false);
                    pf[g] = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(e[2], 448.0f), fminf(e[3], 448.0f), w, true);
                } else {
                    uint32_t w = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) w = __builtin_amdgcn_cvt_pk_u8_f32(e[t], t, w);
                    pf[g] = (int)(w ^ 0x7f7f7f7fu);              // 127 - code as signed bytes
                }
            }
        };
        if ((step + 1) * SK > nvis_min) codes(std::true_type{}); else codes(std::false_type{});
        // the wave reads what its own lanes wrote: LDS operations of one wave keep their order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < DS; ++c) {
            const v4i vf = *reinterpret_cast<const v4i*>(&sv[(c * 32 + ql) * VLD + (c * 2 + (ql >> 4)) * VPAD + hh * 16]);
            if constexpr (F8) o[c] = mfma_wide_f8(vf, zero, pf, zero, o[c]);
            else {
                o[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, pf, o[c], 0, 0, 0);
                o[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, cm127, o[c], 0, 0, 0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // ---- the waves' sums, 32 channels at a time: [wave][query][channel] in LDS, 4 channels of a query per thread
    ST* const tile = reinterpret_cast<ST*>(pool);
#pragma unroll
    for (int c = 0; c < DS; ++c) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<V4*>(tile + (wave * SQ + ql) * TLD + g * 8 + hh * 4) = V4{o[c][4 * g], o[c][4 * g + 1], o[c][4 * g + 2], o[c][4 * g + 3]};
        __syncthreads();
        if (tid < SQ * 8) {
            const int q = tid >> 3, e0 = c * 32 + (tid & 7) * 4;
            V4 tot = {0, 0, 0, 0};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const V4 p = *reinterpret_cast<const V4*>(tile + (w * SQ + q) * TLD + (tid & 7) * 4);
#pragma unroll
                for (int t = 0; t < 4; ++t) tot[t] += p[t];
            }
            if (q0 + q < a.Sq) {
                float y[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float sc = a.scale_is_scalar ? a.out_col_scale[0] : a.out_col_scale[h * DH + e0 + t];
                    y[t] = (F8 ? (float)tot[t] : (float)(-tot[t])) * sc;
                    if (q0 + q >= qlim) y[t] = 0.0f;             // padded query: zeros
                }
                const int64_t oi = ((int64_t)b * a.Sq + q0 + q) * a.ldo + (int64_t)h * DH + e0;
                if (ODT == HERO_I8) *reinterpret_cast<uint32_t*>((int8_t*)a.out + oi) = quant4_sat(y[0], y[1], y[2], y[3]);
                else if (ODT == HERO_F8E4M3) *reinterpret_cast<uint32_t*>((int8_t*)a.out + oi) = fp8x4_sat(y[0], y[1], y[2], y[3]);
                else *reinterpret_cast<v2i*>((uint16_t*)a.out + oi) = v2i{(int)pack2_hp<ODT>(y[0], y[1]), (int)pack2_hp<ODT>(y[2], y[3])};
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Decode (one query per sequence): HBM-bound on the K and V cache, so no matrix cores; K and
// V are each read exactly once.  One block per (batch, head); Dh / 16 lanes share a key (16 bytes of
// the row each, so a wave-level load covers whole rows = 1 KB of consecutive cache).
//   phase 1: integer scores q.k (v_dot4) for every key -> LDS
//   phase 2: row max / sum in the log2 domain (block reduction), codes 0..255 -> LDS
//   phase 3: acc[e] = sum_k P[k] * v[k][e] in int32, reduced over the key groups through LDS
// What bounds the stream is the bytes in flight: UNR loads per lane, NT lanes.  With many blocks, 256 threads (several
// blocks per CU, their phases overlap: 64 x 32 heads x 2049 keys 189 us, 5.7 TB/s); with at most one block per CU, 512 threads
// and the first V loads out during the softmax (the rule and its figures: attn_entry).  A short cache is bound by the chain
// of reductions: those go through data-parallel moves, not LDS.
// In a layer, the block also appends this call's K / V row to its cache: no other block reads that row, and the two
// 4-5 us launches of a step that copied it are gone.
// ------------------------------------------------------------------------------------------
constexpr int DEC_MAX_KEYS = 16384;

// The value of lane ^ O by data-parallel moves, without a trip through LDS.  O = 4 is a rotation within 16 lanes: only where lanes
// that agree in their three lowest bits hold the same already (a butterfly from the top down).
template <int O, typename T>
__device__ __forceinline__ T lane_xor(T x) {
    const uint32_t b = __builtin_bit_cast(uint32_t, x);
    if constexpr (O == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
        return __builtin_bit_cast(T, (threadIdx.x & 32) ? r[0] : r[1]);
    } else if constexpr (O == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(b, b, false, false);
        return __builtin_bit_cast(T, (threadIdx.x & 16) ? r[0] : r[1]);
    } else {
        constexpr int ctrl = O == 8 ? 0x128 : (O == 4 ? 0x124 : (O == 2 ? 0x4E : 0xB1));      // row_ror:8, row_ror:4, quad_perm
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xF, 0xF, true));
    }
}
template <typename T, typename F>
__device__ __forceinline__ T wave_butterfly(T x, F op) {                 // 32 down to 1: every lane ends with the wave's value
    x = op(x, lane_xor<32>(x)); x = op(x, lane_xor<16>(x)); x = op(x, lane_xor<8>(x));
    x = op(x, lane_xor<4>(x)); x = op(x, lane_xor<2>(x)); return op(x, lane_xor<1>(x));
}

// FMT = HERO_F8E4M3: E4M3 operands: the bytes are decoded two at a time (v_cvt_pk_f32_fp8), scores and PV sums are
// fp32, the probability code is e4m3(min(p / S_p, 448)) and its decoded value is what PV multiplies.
template <int DH, int ODT, int FMT, int NT>
__global__ __launch_bounds__(NT) void int8_attn_decode_kernel(AttnArgs a) {
    constexpr bool F8 = FMT == HERO_F8E4M3;
    using ST = typename std::conditional<F8, float, int>::type;      // score / accumulator element
    constexpr int LPK = DH / 16;                 // lanes per key
    constexpr int KPI = NT / LPK;                // keys per block iteration
    constexpr int NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) int smem_dec[];
    ST* sc = reinterpret_cast<ST*>(smem_dec);                      // [len] scores, later codes (F8: their decoded values)
    using V4 = typename std::conditional<F8, v4f, v4i>::type;
    __shared__ float red[2 * NW];
    __shared__ __attribute__((aligned(16))) ST racc[NW][DH + 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.y, h = blockIdx.x;
    const int kvl = a.kv_len ? a.kv_len[b] : a.Skv;
    const int len = min(max(kvl, 0), a.Skv);     // one query: it sees every valid key
    const int sub = tid % LPK, kg = tid / LPK;
    const int8_t* kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2] + sub * 16;
    const int8_t* vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2] + sub * 16;
    const v4i qv = *reinterpret_cast<const v4i*>(a.q + (int64_t)b * a.qs[0] + (int64_t)h * a.qs[2] + sub * 16);
    // the appended row: position len - 1, kept in the registers of every key group (group 0 uses it)
    const bool app = a.kn && kvl >= 1 && kvl <= a.Skv;               // block-uniform
    const int hist = app ? len - 1 : len;                            // keys that are read from the cache
    v4i kn = {0, 0, 0, 0}, vn = {0, 0, 0, 0};
    if (app) {
        const int64_t src = (int64_t)b * a.nstride + (int64_t)h * DH + sub * 16;
        kn = *reinterpret_cast<const v4i*>(a.kn + src);
        vn = *reinterpret_cast<const v4i*>(a.vn + src);
    }
    // 16 E4M3 bytes -> 16 floats
    auto decode16 = [](const v4i& w, float (&f)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], true);
            f[4 * i] = lo[0]; f[4 * i + 1] = lo[1]; f[4 * i + 2] = hi[0]; f[4 * i + 3] = hi[1];
        }
    };
    float qf[16];
    if constexpr (F8) decode16(qv, qf);

    // ---- phase 1: scores ---------------------------------------------------------------------
    constexpr float FMASKED = -3.0e38f;
    ST lmax = F8 ? (ST)FMASKED : (ST)-0x40000000;
    auto score = [&](const v4i& kv) {
        ST d = 0;
        if constexpr (F8) {
            float kf[16];
            decode16(kv, kf);
#pragma unroll
            for (int e = 0; e < 16; ++e) d = fmaf(kf[e], qf[e], d);
        } else {
#pragma unroll
            for (int w = 0; w < 4; ++w) d = __builtin_amdgcn_sdot4(kv[w], qv[w], d, false);
        }
        d += lane_xor<1>(d);
        d += lane_xor<2>(d);
        if constexpr (LPK == 8)                                           // the other quad of the eight lanes (both are uniform by now)
            d += __builtin_bit_cast(ST, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, d), 0x141, 0xF, 0xF, true));     // row_half_mirror
        return d;
    };
    // the stream is bound by the bytes in flight: UNR loads per lane are issued before the first is used.  Unit u of a round is
    // KPI keys, KPW of them this wave's; in the last, partial round a wave leaves out the units in which it has no key (all but
    // a few of them where the cache is short)
    constexpr int UNR = 8, KPW = 64 / LPK, ROUND = UNR * KPI;
    const int full = hist / ROUND * ROUND;
    const int rest = (max(hist - full - __builtin_amdgcn_readfirstlane(wave) * KPW, 0) + KPI - 1) / KPI;      // units of this wave
    auto load_full = [&](v4i (&r)[UNR], const int8_t* base, int64_t stride, int k0) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) r[u] = *reinterpret_cast<const v4i*>(base + (int64_t)(k0 + u * KPI + kg) * stride);
    };
    auto load_rest = [&](v4i (&r)[UNR], const int8_t* base, int64_t stride) {
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (u < rest) r[u] = *reinterpret_cast<const v4i*>(base + (int64_t)min(full + u * KPI + kg, hist - 1) * stride);
    };
    auto take = [&](int key, ST d) {
        if (sub == 0 && key < hist) { sc[key] = d; lmax = max(lmax, d); }
    };
    v4i kv[UNR];
    for (int k0 = 0; k0 < full; k0 += ROUND) {
        load_full(kv, kbase, a.ks[1], k0);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const ST d = score(kv[u]);
            if (sub == 0) sc[k0 + u * KPI + kg] = d;
            lmax = max(lmax, d);
        }
    }
    load_rest(kv, kbase, a.ks[1]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) if (u < rest) take(full + u * KPI + kg, score(kv[u]));
    if (app) {
        const ST d = score(kn);
        if (tid == 0) sc[hist] = d;
        lmax = max(lmax, d);
        if (kg == 0) {
            const int64_t dst = (int64_t)hist * a.ks[1], vst = (int64_t)hist * a.vs[1];
            *reinterpret_cast<v4i*>(a.kc + (kbase - a.k) + dst) = kn;
            *reinterpret_cast<v4i*>(a.vc + (vbase - a.v) + vst) = vn;
        }
    }
    // one block per CU: the first V loads are in flight during the softmax (several overlap anyway, and need the registers)
    constexpr bool EARLY_V = NT > 256;
    v4i vv[UNR];
    if (!EARLY_V) {} else if (full > 0) load_full(vv, vbase, a.vs[1], 0); else load_rest(vv, vbase, a.vs[1]);
    // block max
    lmax = wave_butterfly(lmax, [](ST x, ST y) { return max(x, y); });
    if (lane == 0) red[wave] = F8 ? (float)lmax : __int_as_float((int)lmax);
    __syncthreads();
    const float c2 = a.qk_scale * 1.44269504088896340736f;
    float m2;
    if constexpr (F8) {
        float m = red[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, red[w]);
        m2 = m * c2;
    } else {
        int m = __float_as_int(red[0]);
#pragma unroll
        for (int w = 1; w < NW; ++w) m = max(m, __float_as_int(red[w]));
        m2 = (float)m * c2;
    }
    // ---- phase 2: sum, then codes --------------------------------------------------------------
    float lsum = 0.0f;
    for (int k = tid; k < len; k += NT) lsum += __builtin_amdgcn_exp2f(fmaf((float)sc[k], c2, -m2));
    lsum = wave_butterfly(lsum, [](float x, float y) { return x + y; });
    if (lane == 0) red[NW + wave] = lsum;
    __syncthreads();
    float l = red[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) l += red[NW + w];
    const float off = l > 0.0f ? -m2 - __log2f(l * a.p_scale) : -INFINITY;
    for (int k = tid; k < len; k += NT) {
        const float e = __builtin_amdgcn_exp2f(fmaf((float)sc[k], c2, off));
        if constexpr (F8) sc[k] = __builtin_amdgcn_cvt_f32_fp8(__builtin_amdgcn_cvt_pk_fp8_f32(fminf(e, 448.0f), 0.0f, 0, false), 0);
        else sc[k] = (int)__builtin_amdgcn_cvt_pk_u8_f32(e, 0, 0u);
    }
    __syncthreads();
    // ---- phase 3: PV ------------------------------------------------------------------------------
    ST acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0;
    auto pv = [&](const v4i& w, const ST p) {
        if constexpr (F8) {
            float vf[16];
            decode16(w, vf);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] += p * (int)(int8_t)(w[e >> 2] >> (8 * (e & 3)));
        }
    };
    for (int k0 = 0; k0 < full; k0 += ROUND) {
        if (!EARLY_V || k0 > 0) load_full(vv, vbase, a.vs[1], k0);
#pragma unroll
        for (int u = 0; u < UNR; ++u) pv(vv[u], sc[k0 + u * KPI + kg]);
    }
    if (!EARLY_V || full > 0) load_rest(vv, vbase, a.vs[1]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
        const int key = full + u * KPI + kg;
        if (u < rest) pv(vv[u], key < hist ? sc[key] : (ST)0);
    }
    if (app && kg == 0) pv(vn, sc[hist]);
    // sum over the key groups: across a wave's lanes first, then through LDS in the fixed order of the waves.  The halves and the
    // rows of 16 lanes exchange elements while they add (v_permlane32_swap, v_permlane16_swap), so a lane of row r is left with
    // the elements 8 (r / 2) + 4 (r % 2) + 0 .. 3 of its 16, for the key groups of its row, which rotations add.  (Sixteen
    // butterflies through LDS cost a block of 1024 threads 2 us.)
    auto bits = [](ST x) { return __builtin_bit_cast(uint32_t, x); };
    auto val = [](uint32_t x) { return __builtin_bit_cast(ST, x); };
    ST half[8], quad[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const auto r = __builtin_amdgcn_permlane32_swap(bits(acc[e]), bits(acc[e + 8]), false, false);
        half[e] = val(r[0]) + val(r[1]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto r = __builtin_amdgcn_permlane16_swap(bits(half[e]), bits(half[e + 4]), false, false);
        quad[e] = val(r[0]) + val(r[1]);
        quad[e] += val((uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits(quad[e]), 0x128, 0xF, 0xF, true));              // row_ror:8
        if (LPK == 4) quad[e] += val((uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits(quad[e]), 0x124, 0xF, 0xF, true));  // row_ror:4
    }
    if ((lane & 15) < LPK) {
        const int row = lane >> 4;
        *reinterpret_cast<V4*>(&racc[wave][sub * 16 + 8 * (row >> 1) + 4 * (row & 1)]) = V4{quad[0], quad[1], quad[2], quad[3]};
    }
    __syncthreads();
    if (tid < DH) {
        ST tot = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) tot += racc[w][tid];
        const float scl = a.scale_is_scalar ? a.out_col_scale[0] : a.out_col_scale[h * DH + tid];
        const float y = (float)tot * scl;
        const int64_t oidx = (int64_t)b * a.ldo + (int64_t)h * DH + tid;
        if (ODT == HERO_I8) ((int8_t*)a.out)[oidx] = (int8_t)(rne_low_byte(__builtin_amdgcn_fmed3f(y, -127.0f, 127.0f)) & 0xff);
        else if (ODT == HERO_F8E4M3) ((uint8_t*)a.out)[oidx] = (uint8_t)(fp8x4_sat(y, 0.0f, 0.0f, 0.0f) & 0xffu);
        else ((uint16_t*)a.out)[oidx] = (uint16_t)f32_to_hp<ODT>(y);
    }
}

__global__ void zero_rows_kernel(int8_t* out, int64_t bytes) {
    int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 16;
    if (i < bytes) *reinterpret_cast<v4i*>(out + i) = v4i{0, 0, 0, 0};
}

// The decode kernel keeps one score per key in dynamic LDS; beyond 32 KB a kernel must be told once (per device) how
// much it may ask for.  The attribute is raised to the kernel's maximum the first time a launch needs more than the
// default, not on every call.
template <int DH, int ODT, int FMT, int NT>
bool decode_lds_ready(size_t lds) {
    static std::atomic<bool> raised[64];
    if (lds <= 32768) return true;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    if (raised[dev].load(std::memory_order_acquire)) return true;
    if (hipFuncSetAttribute((const void*)int8_attn_decode_kernel<DH, ODT, FMT, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            DEC_MAX_KEYS * (int)sizeof(int)) != hipSuccess) return false;
    raised[dev].store(true, std::memory_order_release);
    return true;
}

template <int DH, bool ONLINE = false, int FMT = HERO_I8>
hero_status launch(const AttnArgs& a, hero_dtype out_dt, hipStream_t st) {
    constexpr int HG = DH >= 128 ? 1 : 128 / DH;               // heads per workgroup group (see the kernel)
    const int64_t nqb = (a.Sq + BQ - 1) / BQ, hgroups = ((int64_t)a.B * a.H + HG - 1) / HG, rounds = (hgroups + 7) / 8;
    if (rounds * 8 * HG * nqb > 0x7fffffffLL) return HERO_ERR_SHAPE;
    dim3 grid((unsigned)(rounds * 8 * HG * nqb)), block(256);
    if (out_dt == HERO_BF16) hipLaunchKernelGGL((int8_attn_kernel<DH, HERO_BF16, ONLINE, FMT>), grid, block, 0, st, a);
    else if (out_dt == HERO_F16) hipLaunchKernelGGL((int8_attn_kernel<DH, HERO_F16, ONLINE, FMT>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((int8_attn_kernel<DH, FMT, ONLINE, FMT>), grid, block, 0, st, a);      // 8-bit output in the operands' format
    return hero_launch_status();
}

template <int FMT>
hero_status launch_keep(const AttnArgs& a, hero_dtype out_dt, hipStream_t st) {
    const int64_t nqb = (a.Sq + BQ - 1) / BQ, hgroups = ((int64_t)a.B * a.H + 1) / 2, rounds = (hgroups + 7) / 8;
    if (rounds * 16 * nqb > 0x7fffffffLL) return HERO_ERR_SHAPE;
    auto go = [&](auto NT, auto KW) -> hero_status {
        constexpr int nt = decltype(NT)::value, kw = decltype(KW)::value;
        dim3 grid((unsigned)(rounds * 16 * nqb)), block(256 * kw);
        if (out_dt == HERO_BF16) hipLaunchKernelGGL((int8_attn_keep_kernel<HERO_BF16, FMT, nt, kw>), grid, block, 0, st, a);
        else if (out_dt == HERO_F16) hipLaunchKernelGGL((int8_attn_keep_kernel<HERO_F16, FMT, nt, kw>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((int8_attn_keep_kernel<FMT, FMT, nt, kw>), grid, block, 0, st, a);
        return hero_launch_status();
    };
    constexpr std::integral_constant<int, 1> one;
    if (a.Skv <= 128) return go(std::integral_constant<int, 2>{}, one);
    if (a.Skv <= 256) return go(std::integral_constant<int, 4>{}, one);
    return go(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
}

template <int DH, int FMT, int NW>
hero_status launch_split(const AttnArgs& a, hero_dtype out_dt, hipStream_t st) {
    constexpr int HG = DH >= 128 ? 1 : 128 / DH;
    const int64_t nqb = (a.Sq + 31) / 32, hgroups = ((int64_t)a.B * a.H + HG - 1) / HG, rounds = (hgroups + 7) / 8;
    if (rounds * 8 * HG * nqb > 0x7fffffffLL) return HERO_ERR_SHAPE;
    dim3 grid((unsigned)(rounds * 8 * HG * nqb)), block(64 * NW);
    auto go = [&](auto W) {
        constexpr int CW = decltype(W)::value;
        if (out_dt == HERO_BF16) hipLaunchKernelGGL((int8_attn_split_kernel<DH, HERO_BF16, FMT, NW, CW>), grid, block, 0, st, a);
        else if (out_dt == HERO_F16) hipLaunchKernelGGL((int8_attn_split_kernel<DH, HERO_F16, FMT, NW, CW>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((int8_attn_split_kernel<DH, FMT, FMT, NW, CW>), grid, block, 0, st, a);
    };
    // V in 128-bit loads (128 channels), but not for E4M3 with at most one block per CU and 1024 keys or more, whose steps, shorter by a matrix instruction, wait
    // longer for four such loads than for sixteen of 32 bits.  us, 32 / 128 bits: E4M3 32 blocks x 2165 keys 23.3 / 24.5, 112 x 1553 19.5 / 20.2, 224 x 1694 21.8 /
    // 22.2, 128 x 820 12.4 / 12.6, but padded 64 x 831 11.7 / 11.4, 128 x 498 9.8 / 9.6, 384 x 1837 26.6 / 24.8, 640 x 1338 38.0 / 36.3;  INT8 64 x 1969 17.6 / 17.4, 320 x 859 20.0 / 18.9.
    if constexpr (DH >= 128) {
        if (FMT != HERO_F8E4M3 || (int64_t)a.B * a.H * nqb > 256 || a.Skv < 1024) {
            go(std::integral_constant<int, 16>{});
            return hero_launch_status();
        }
    }
    if constexpr (DH < 128 || FMT == HERO_F8E4M3) go(std::integral_constant<int, 4>{});
    return hero_launch_status();
}

// argument checks and dispatch shared by the two entry points (online: the single-sweep variant)
hero_status attn_entry(const int8_t* q, const int64_t q_strides[4],
                       const int8_t* k, const int64_t k_strides[4],
                       const int8_t* v, const int64_t v_strides[4],
                       int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh,
                       float qk_scale, const float* qk_scale_h, bool online, bool fp8,
                       float p_scale, const float* out_col_scale, int out_scale_is_scalar,
                       hero_mask mask, const int32_t* kv_len,
                       void* out, hero_dtype out_dt, int64_t ldo, void* stream,
                       const int8_t* kn = nullptr, const int8_t* vn = nullptr, int64_t nstride = 0) {
    if (B < 0 || H < 0 || Sq < 0 || Skv < 0) return HERO_ERR_SHAPE;
    if (Dh != 64 && Dh != 128) return HERO_ERR_UNSUPPORTED;
    const hero_dtype dt8 = fp8 ? HERO_F8E4M3 : HERO_I8;                  // the 8-bit output format is the operands'
    if (out_dt != dt8 && out_dt != HERO_BF16 && out_dt != HERO_F16) return HERO_ERR_UNSUPPORTED;
    if (mask != HERO_MASK_NONE && mask != HERO_MASK_PADDING && mask != HERO_MASK_CAUSAL) return HERO_ERR_UNSUPPORTED;
    if (B == 0 || H == 0 || Sq == 0) return HERO_OK;
    if (!out || !out_col_scale || !q_strides || !k_strides || !v_strides) return HERO_ERR_NULL;
    if (Skv > 0 && (!q || !k || !v)) return HERO_ERR_NULL;
    if (mask == HERO_MASK_PADDING && !kv_len) return HERO_ERR_NULL;
    if (online && !qk_scale_h) return HERO_ERR_NULL;
    if (out_dt != dt8 && !out_scale_is_scalar) return HERO_ERR_UNSUPPORTED;
    if (!(p_scale > 0.0f)) return HERO_ERR_SHAPE;
    if (ldo < H * Dh) return HERO_ERR_SHAPE;
    if (B > 65535 || H > 65535 || Sq > 0x7fffffffLL || Skv > 0x7fffffffLL) return HERO_ERR_SHAPE;
    const int64_t* ss[3] = {q_strides, k_strides, v_strides};
    for (int t = 0; t < 3; ++t) {
        if (ss[t][3] != 1) return HERO_ERR_UNSUPPORTED;
        if (ss[t][0] % 16 || ss[t][1] % 16 || ss[t][2] % 16) return HERO_ERR_ALIGN;
    }
    const int64_t o_elem = out_dt == dt8 ? 1 : 2;
    if ((ldo * o_elem) % 16 != 0 || !hero_aligned16(out) || !hero_aligned16(q) || !hero_aligned16(k) || !hero_aligned16(v))
        return HERO_ERR_ALIGN;
    AttnArgs a;
    a.q = q; a.k = k; a.v = v;
    for (int t = 0; t < 4; ++t) { a.qs[t] = q_strides[t]; a.ks[t] = k_strides[t]; a.vs[t] = v_strides[t]; }
    a.B = (int)B; a.H = (int)H; a.Sq = (int)Sq; a.Skv = (int)Skv;
    a.qk_scale = qk_scale; a.qk_scale_h = qk_scale_h; a.p_scale = p_scale; a.out_col_scale = out_col_scale; a.scale_is_scalar = out_scale_is_scalar;
    a.mask = (int)mask; a.kv_len = kv_len; a.out = out; a.ldo = ldo;
    a.kn = kn; a.vn = vn; a.nstride = nstride; a.kc = const_cast<int8_t*>(k); a.vc = const_cast<int8_t*>(v);
    a.use_buf = Skv > 0 && k_strides[1] >= 0 && v_strides[1] >= 0 &&
                (Skv + BKV) * k_strides[1] + Dh < (1LL << 31) && (Skv + BKV) * v_strides[1] + Dh < (1LL << 31);
    hipStream_t st = (hipStream_t)stream;
    if (Skv == 0) {     // no keys at all: every query outputs 0
        const int64_t bytes = B * Sq * ldo * o_elem;                 // a multiple of 16 (ldo rule)
        const int64_t blocks = (bytes / 16 + 255) / 256;
        if (blocks > 0x7fffffffLL) return HERO_ERR_SHAPE;
        hipLaunchKernelGGL(zero_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (int8_t*)out, bytes);
        return hero_launch_status();
    }
    if (online) return Dh == 64 ? launch<64, true>(a, out_dt, st) : launch<128, true>(a, out_dt, st);
    if (Sq == 1 && Skv <= DEC_MAX_KEYS) {          // decode: the cache-streaming kernel
        // One block per CU or fewer: 512 threads.  Measured, us, 256 / 512 / 1024 threads: 96 blocks (Dh 128) x 1 key 3.3 / 3.5 /
        // 4.1, x 128 4.6 / 4.5 / 4.8, x 512 8.1 / 6.9 / 7.0, x 2048 23.6 / 18.6 / 19.1; 256 blocks x 1000 16.5 / 14.5 / 16.6.  From two
        // blocks on a CU narrow ones are ahead: 288 x 1000 18.9 / 20.3 / 23.6, 768 x 1 3.8 / 5.5 / 9.6.
        const int nt = B * H <= 256 ? 512 : 256;
        dim3 grid((unsigned)H, (unsigned)B), block(nt);
        const size_t lds = (size_t)Skv * sizeof(int);
#define HERO_DEC_NT(DH_, ODT_, FMT_, NT_) do { \
            if (!decode_lds_ready<DH_, ODT_, FMT_, NT_>(lds)) return HERO_ERR_LAUNCH; \
            hipLaunchKernelGGL((int8_attn_decode_kernel<DH_, ODT_, FMT_, NT_>), grid, block, lds, st, a); } while (0)
#define HERO_DEC(DH_, ODT_, FMT_) do { if (nt == 512) HERO_DEC_NT(DH_, ODT_, FMT_, 512); else HERO_DEC_NT(DH_, ODT_, FMT_, 256); } while (0)
#define HERO_DEC_DT(DH_, FMT_) do { \
            if (out_dt == HERO_BF16) HERO_DEC(DH_, HERO_BF16, FMT_); else if (out_dt == HERO_F16) HERO_DEC(DH_, HERO_F16, FMT_); \
            else HERO_DEC(DH_, FMT_, FMT_); } while (0)
        if (fp8) { if (Dh == 64) HERO_DEC_DT(64, HERO_F8E4M3); else HERO_DEC_DT(128, HERO_F8E4M3); }
        else { if (Dh == 64) HERO_DEC_DT(64, HERO_I8); else HERO_DEC_DT(128, HERO_I8); }
#undef HERO_DEC_DT
#undef HERO_DEC
#undef HERO_DEC_NT
        return hero_launch_status();
    }
    // At most one 128-query block per CU, or a single 32-query piece: the keys are split over the waves.  Measured, us, 128-query
    // kernel -> split: 1 x 12 heads x 128 8.8 -> 5.3, 2 x 16 x 512 18.5 -> 10.8, 2 x 32 x 301 behind 900 keys 47.6 -> 37.2,
    // 8 x 32 x 8 behind 2000 keys 78.7 -> 31.0, 256 blocks of 1 x 32 x 1024 causal 43 -> 37; beyond (512 blocks of 8 x 16 x 512)
    // 23.5 -> 26.0: there the chip is full and reading K / V four times as often costs more than the shorter chain gives.  With
    // Dh = 128 a CU holds fewer of its blocks, and it is full from three pieces of 32 queries on: 2 x 32 x 301 (640 pieces) above,
    // but 8 x 32 x 128 (1024) 12.3 -> 14.1, E4M3 4 x 32 x 200 (896) 13.9 -> 14.8.
    // Up to 512 keys of 64 channels the one-pass kernel takes over from three quarters of the CUs on, and beyond from the two-pass
    // kernel altogether: split -> one pass 128 blocks (8 x 16 x 100) 5.7 -> 6.3, 192 (12 x 16 x 128) 7.0 -> 6.6, 256 (4 x 16 x 512)
    // 15.0 -> 10.7, (8 x 16 x 256) 10.5 -> 8.4; two passes -> one 32 x 16 x 512 padded 65 -> 56.5, 11 x 16 x 347 19.7 -> 14.4, 16 x 16 x 256
    // 14.9 -> 10.4, 32 x 12 x 128 10.1 -> 7.6; E4M3 11 x 16 x 347 18.0 -> 14.2, 16 x 16 x 256 14.0 -> 10.9.  Up to one block per CU it
    // stays with the split kernel where the blocks are little more than half full (192 blocks of 129 padded keys 6.0 / 7.2, of 160
    // 6.7 / 7.5; but of 192, three quarters full, 8.2 / 7.4), and where an XCD is handed more of the 512-key form's blocks than it has CUs (252
    // blocks, 36 on some XCDs: 300 keys 12.1 / 12.8; 216 blocks, 30: 12.0 / 9.2).
    const int64_t nqb = (Sq + BQ - 1) / BQ, blocks = B * H * nqb, pieces = B * H * ((Sq + 31) / 32), on_xcd = (B * H + 15) / 16 * 2 * nqb;
    // E4M3 of more than 256 keys, from six blocks of the two-pass kernel per CU on: its wide matrix instruction takes 64 keys where the one-pass
    // kernel's is half filled, and with many blocks that shows; padding, which ends its blocks early, adds to it.  Two passes / one, padded:
    // 2064 blocks 260 keys 31.3 / 32.3, 320 36.0 / 37.2, 448 43.1 / 44.4, 480 47.8 / 48.7, 512 55.4 / 54.4, 3072 blocks 320 48.4 / 53.1, 512
    // 71.3 / 72.2, but 1392 blocks 320 27.3 / 26.8;  full: 2064 blocks 320 43.3 / 46.5, 347 52.6 / 52.0, 448 54.1 / 51.1, 512 62.0 / 57.1.
    // Heads of few queries, whose blocks are short and take both of a CU's places in one pass, cross earlier (full, 64 queries: 504
    // blocks 400 keys 0.87 of the two-pass time, 516 blocks 1.12, 1032 1.28; 96 queries: 768 blocks 0.94, 1032 1.06).
    const bool many_f8 = fp8 && Skv > 256 && ((blocks >= 1536 && Skv <= (mask == HERO_MASK_PADDING ? 480 : 352)) ||
                                              (Sq <= 64 && blocks > 512) || (Sq <= 96 && blocks > 1024));
    const bool few = blocks <= 191 || (blocks <= 256 && (2 * pieces <= 5 * blocks || (Skv > 256 && on_xcd > 32)));
    const bool keep = Dh == 64 && Skv <= 512 && qk_scale >= KEEP_MIN_QK && !many_f8;
    if (((keep ? few : blocks <= 256) && (Dh == 64 || pieces <= 768)) || Sq <= 32) {
        if (fp8) return Dh == 64 ? launch_split<64, HERO_F8E4M3, 4>(a, out_dt, st) : launch_split<128, HERO_F8E4M3, 4>(a, out_dt, st);
        return Dh == 64 ? launch_split<64, HERO_I8, 4>(a, out_dt, st) : launch_split<128, HERO_I8, 4>(a, out_dt, st);
    }
    if (keep) return fp8 ? launch_keep<HERO_F8E4M3>(a, out_dt, st) : launch_keep<HERO_I8>(a, out_dt, st);
    if (fp8) return Dh == 64 ? launch<64, false, HERO_F8E4M3>(a, out_dt, st) : launch<128, false, HERO_F8E4M3>(a, out_dt, st);
    return Dh == 64 ? launch<64>(a, out_dt, st) : launch<128>(a, out_dt, st);
}

}  // namespace

// One decode step of a layer: hero_int8_attn / hero_fp8_attn over the cache, with this call's K / V rows (row stride nstride)
// written to their place in it by the same kernel.  HERO_ERR_UNSUPPORTED: not a case of that kernel (the caller appends and
// attends in two launches).  Not part of the C ABI.
hero_status hero_attn_decode_append(const int8_t* q, const int64_t q_strides[4], const int8_t* kn, const int8_t* vn, int64_t nstride,
                                    int8_t* kc, int8_t* vc, const int64_t c_strides[4], int64_t B, int64_t H, int64_t Smax, int64_t Dh,
                                    float qk_scale, float p_scale, const float* out_col_scale, int out_scale_is_scalar, hero_mask mask,
                                    const int32_t* kv_len, void* out, hero_dtype out_dt, int64_t ldo, bool fp8, void* stream) {
    if (Smax <= 0 || Smax > DEC_MAX_KEYS) return HERO_ERR_UNSUPPORTED;
    return attn_entry(q, q_strides, kc, c_strides, vc, c_strides, B, H, 1, Smax, Dh, qk_scale, nullptr, false, fp8, p_scale,
                      out_col_scale, out_scale_is_scalar, mask, kv_len, out, out_dt, ldo, stream, kn, vn, nstride);
}

extern "C" hero_status hero_int8_attn(const int8_t* q, const int64_t q_strides[4],
                                      const int8_t* k, const int64_t k_strides[4],
                                      const int8_t* v, const int64_t v_strides[4],
                                      int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh,
                                      float qk_scale, float p_scale, const float* out_col_scale, int out_scale_is_scalar,
                                      hero_mask mask, const int32_t* kv_len,
                                      void* out, hero_dtype out_dt, int64_t ldo, void* stream) {
    return attn_entry(q, q_strides, k, k_strides, v, v_strides, B, H, Sq, Skv, Dh, qk_scale, nullptr, false, false, p_scale,
                      out_col_scale, out_scale_is_scalar, mask, kv_len, out, out_dt, ldo, stream);
}

extern "C" hero_status hero_int8_attn_online(const int8_t* q, const int64_t q_strides[4],
                                             const int8_t* k, const int64_t k_strides[4],
                                             const int8_t* v, const int64_t v_strides[4],
                                             int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh,
                                             const float* qk_scale_h, float p_scale, const float* out_col_scale,
                                             int out_scale_is_scalar, hero_mask mask, const int32_t* kv_len,
                                             void* out, hero_dtype out_dt, int64_t ldo, void* stream) {
    return attn_entry(q, q_strides, k, k_strides, v, v_strides, B, H, Sq, Skv, Dh, 0.0f, qk_scale_h, true, false, p_scale,
                      out_col_scale, out_scale_is_scalar, mask, kv_len, out, out_dt, ldo, stream);
}

extern "C" hero_status hero_fp8_attn(const void* q, const int64_t q_strides[4],
                                     const void* k, const int64_t k_strides[4],
                                     const void* v, const int64_t v_strides[4],
                                     int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh,
                                     float qk_scale, float p_scale, const float* out_col_scale, int out_scale_is_scalar,
                                     hero_mask mask, const int32_t* kv_len,
                                     void* out, hero_dtype out_dt, int64_t ldo, void* stream) {
    return attn_entry((const int8_t*)q, q_strides, (const int8_t*)k, k_strides, (const int8_t*)v, v_strides, B, H, Sq, Skv, Dh,
                      qk_scale, nullptr, false, true, p_scale, out_col_scale, out_scale_is_scalar, mask, kv_len, out, out_dt, ldo, stream);
}
