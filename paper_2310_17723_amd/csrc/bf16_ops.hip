// 16-bit side of a switched module (paper Sec. 2.3, Table 1: a module marked with a cross runs
// in FP16 / BF16): hero_hp_attn (and its BF16-only name hero_bf16_attn); hero_hp_gemm is in int8_gemm.hip.
// bf16 or fp16 operands, fp32 accumulation on the matrix cores (v_mfma_f32_32x32x16_bf16 / _f16), results in
// the operands' type.
#include "hero_common.h"

namespace {

typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// one 32x32x16 matrix instruction on 8 + 8 16-bit values per lane; DT = HERO_BF16 or HERO_F16
template <int DT>
__device__ __forceinline__ v16f mfma_hp(v4i a, v4i b, v16f c) {
    if constexpr (DT == HERO_BF16) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}

// s + the two 16-bit values of pk (v_dot2_f32_bf16 / _f16 against ones)
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
template <int DT>
__device__ __forceinline__ float add_pair(uint32_t pk, float s) {
    if constexpr (DT == HERO_BF16) return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, pk), __builtin_bit_cast(v2bf, 0x3f803f80u), s, false);
    else return __builtin_amdgcn_fdot2(__builtin_bit_cast(v2h, pk), v2h{(_Float16)1.0f, (_Float16)1.0f}, s, false);
}

// ------------------------------------------------------------------------------------------
// Attention core softmax(q k^T * scale) v, single pass with an online softmax (nothing is
// quantized here, so the running rescale is legitimate).  Scores are computed transposed
// (S^T = K Q^T): lane l owns query l % 32, so the running max / sum and the rescale of the
// output accumulators are per-lane scalars.
// Bound by the vector ALU and the latency of a tile's chain (scores, maximum, exponentials, PV): per score half a maximum, the fma that
// scales and subtracts, exp2 (four slots), half a packing conversion and half a v_dot2 that sums the packed values.  Keys are compared with
// the limit only in tiles that hide one, a wave leaves out tiles of which it sees nothing.  us, with a multiplication, a comparison and a
// select per score and sums of unpacked values -> this: 8 x 16 x 512 padded 24.5 -> 21.5, 16 x 16 x 300 causal 19.9 -> 17.2, 4 x 32 x 1024 x 128
// causal 120 -> 107 (FP16 126 -> 113), 8 x 32 x 256 behind 2048 keys 156 -> 130;  BERT-large layer 32 x 512 in M1 385 -> 379.  (The maximum raised once
// per 64 keys: another 2-5 %, but an error larger by 0.1 .. 0.6 %, since fewer probabilities are exactly 1.)
// ------------------------------------------------------------------------------------------
constexpr int ABQ = 128, ABKV = 64;

struct BAttnArgs {
    const uint16_t* q; const uint16_t* k; const uint16_t* v;
    int64_t qs[4], ks[4], vs[4];
    int B, H, Sq, Skv; float scale; int mask; const int32_t* kv_len;
    uint16_t* out; int64_t ldo;
};

template <int DH, int DT>
__global__ __launch_bounds__(256) void bf16_attn_kernel(BAttnArgs a) {
    constexpr int KLD = DH * 2 + 16;       // sK row stride, bytes
    constexpr int VLD = ABKV * 2 + 16;     // sVt row stride, bytes (64 keys of bf16)
    constexpr int DS = DH / 16;            // 16-wide MFMA k-steps over the head dimension
    constexpr int CT = DH / 32;            // 32-channel output tiles
    __shared__ __attribute__((aligned(16))) int8_t sK[ABKV * KLD];
    __shared__ __attribute__((aligned(16))) int8_t sVt[DH * VLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5, ql = lane & 31;
    // Workgroups go round-robin to the 8 XCDs: all query blocks of one (batch, head) are sent to the same XCD, back to
    // back, so its K / V stream hits that XCD's L2 after the first block; their order inside the head rotates with a
    // hash of the head's number (the blocks of a causal or padded head differ in length, and the hardware places
    // workgroups on the compute units in launch order: a fixed order hands a unit the same kind of block every time).
    const int nqb = (a.Sq + ABQ - 1) / ABQ;
    const int slot = blockIdx.x / 8, bh = (slot / nqb) * 8 + (int)(blockIdx.x % 8);
    if (bh >= a.B * a.H) return;
    const uint32_t rot = ((uint32_t)(slot / nqb) * 2654435761u) >> 20;
    const int b = bh / a.H, h = bh % a.H, q0 = (int)((slot % nqb + rot) % (uint32_t)nqb) * ABQ;
    const int len = a.kv_len ? min(max(a.kv_len[b], 0), a.Skv) : a.Skv;
    const int shift = len - a.Sq;
    const int qi = q0 + wave * 32 + ql;
    int nvis = len;
    if (a.mask == HERO_MASK_CAUSAL) nvis = min(len, qi + shift + 1);
    nvis = max(nvis, 0);
    int kmax = len;
    if (a.mask == HERO_MASK_CAUSAL) kmax = min(len, min(q0 + ABQ, a.Sq) + shift);
    // PADDING mask in self-attention: the positions >= len are padding as queries too; they see no key (output 0)
    if (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) {
        if (qi >= len) nvis = 0;
        if (q0 >= len) kmax = 0;
    }
    const int ntiles = (max(kmax, 0) + ABKV - 1) / ABKV;

    v4i qf[DS];
    {
        const uint16_t* qp = a.q + (int64_t)b * a.qs[0] + (int64_t)min(qi, a.Sq - 1) * a.qs[1] + (int64_t)h * a.qs[2];
#pragma unroll
        for (int d = 0; d < DS; ++d) qf[d] = *reinterpret_cast<const v4i*>(qp + d * 16 + hh * 8);
    }
    const uint16_t* kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2];
    const uint16_t* vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2];
    const float c2 = a.scale * 1.44269504088896340736f;
    // the scale goes into the exponent's fma, the maximum is taken of the sums themselves; any other scale is multiplied in first
    const bool fold = c2 > 0.0f && c2 < 1e30f;
    const float cf = fold ? c2 : 1.0f;
    // of this wave's 32 queries (uniform): tiles before `edge` hide no key from any of them, tiles from `wvis` on all
    const int w0 = __builtin_amdgcn_readfirstlane(q0 + wave * 32);
    int nmin = len, nmax = len;
    if (a.mask == HERO_MASK_CAUSAL) {
        nmin = min(len, w0 + shift + 1);
        nmax = min(len, w0 + 32 + shift);
    }
    if (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) {
        if (w0 + 32 > len) nmin = 0;
        if (w0 >= len) nmax = 0;
    }
    const int edge = max(nmin, 0) / ABKV, wvis = (max(nmax, 0) + ABKV - 1) / ABKV;
    float m2 = -INFINITY, l = 0.0f;
    v16f o[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[c][r] = 0.0f;

    // K / V tiles: global -> registers (the next tile's loads are in flight during the current tile's math) -> LDS.
    // A thread's unit is one 16-byte chunk (8 channels) of TWO neighbouring key rows 2r, 2r + 1: V is stored transposed
    // and the two keys sit side by side there, so a channel's pair of values goes out as one 32-bit store.
    constexpr int CPRW = DH / 8;                           // 16-byte chunks per K/V row
    constexpr int PAIRS = (ABKV / 2) * CPRW / 256;         // units per thread and tile
    v4i rk[PAIRS][2], rv[PAIRS][2];
    auto fetch = [&](int tile) {
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            const int idx = tid + u * 256, rp = idx / CPRW, ch = idx % CPRW;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int key = min(tile * ABKV + 2 * rp + j, a.Skv - 1);
                rk[u][j] = *reinterpret_cast<const v4i*>(kbase + (int64_t)key * a.ks[1] + ch * 8);
                rv[u][j] = *reinterpret_cast<const v4i*>(vbase + (int64_t)key * a.vs[1] + ch * 8);
            }
        }
    };
    if (ntiles > 0) fetch(0);
    for (int tile = 0; tile < ntiles; ++tile) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            const int idx = tid + u * 256, rp = idx / CPRW, ch = idx % CPRW, row = 2 * rp;
            *reinterpret_cast<v4i*>(&sK[row * KLD + ch * 16]) = rk[u][0];
            *reinterpret_cast<v4i*>(&sK[(row + 1) * KLD + ch * 16]) = rk[u][1];
            // key row 32kb + 8g + 4h' + t of the tile -> position 32kb + 16(g>>1) + 8h' + 4(g&1) + t:
            // within each 16-key MFMA step, half h' holds its 8 keys (g&1, t) contiguously; rows 2r and 2r + 1
            // differ in the lowest bit of t only
            const int r32 = row & 31, g4 = r32 >> 3, hp = (r32 >> 2) & 1, t = r32 & 3;
            const int pos = (row & 32) + (g4 >> 1) * 16 + hp * 8 + (g4 & 1) * 4 + t;
#pragma unroll
            for (int j = 0; j < 4; ++j) {                   // channels 2j, 2j + 1 of both keys
                const uint32_t w0 = (uint32_t)rv[u][0][j], w1 = (uint32_t)rv[u][1][j];
                *reinterpret_cast<uint32_t*>(&sVt[(ch * 8 + 2 * j) * VLD + pos * 2]) = __builtin_amdgcn_perm(w1, w0, 0x05040100u);
                *reinterpret_cast<uint32_t*>(&sVt[(ch * 8 + 2 * j + 1) * VLD + pos * 2]) = __builtin_amdgcn_perm(w1, w0, 0x07060302u);
            }
        }
        __syncthreads();
        if (tile + 1 < ntiles) fetch(tile + 1);
        if (tile >= wvis) continue;
        v16f acc[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][r] = 0.0f;
#pragma unroll
            for (int d = 0; d < DS; ++d) {
                const v4i kf = *reinterpret_cast<const v4i*>(&sK[(s * 32 + ql) * KLD + d * 32 + hh * 16]);
                acc[s] = mfma_hp<DT>(kf, qf[d], acc[s]);
            }
        }
        if (!fold)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[s][r] *= c2;
        if (tile >= edge) {
            const int lim = nvis - tile * ABKV - hh * 4;
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[s][r] = s * 32 + (r >> 2) * 8 + (r & 3) < lim ? acc[s][r] : -INFINITY;
        }
        // (the maximum is raised every 32 keys: the key that raises it has a probability of 1, which 16 bits hold without an error)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float tmax = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, acc[s][r]);
            const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
            tmax = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
            const float mn = fmaxf(m2, tmax * cf), ms = mn > -INFINITY ? mn : 0.0f;      // (no key seen yet: every exponential is 0)
            const float resc = __builtin_amdgcn_exp2f(m2 - ms);
            uint32_t pb[8];
            float sum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const uint32_t pk = pack2_hp<DT>(__builtin_amdgcn_exp2f(fmaf(acc[s][r], cf, -ms)), __builtin_amdgcn_exp2f(fmaf(acc[s][r + 1], cf, -ms)));
                sum = add_pair<DT>(pk, sum);                                        // the sum of what PV really multiplies
                pb[r >> 1] = pk;
            }
            l = fmaf(l, resc, sum);
            // the accumulators are rescaled only in steps where some query of the wave raises its maximum
            // (otherwise every factor is exactly 1)
            if (__builtin_amdgcn_ballot_w64(mn != m2) != 0) {
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[c][r] *= resc;
            }
            m2 = mn;
            // registers 0..7 (g = 0,1) feed the first 16-key MFMA step, 8..15 (g = 2,3) the second
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const v4i pf = {(int)pb[4 * st], (int)pb[4 * st + 1], (int)pb[4 * st + 2], (int)pb[4 * st + 3]};
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const v4i vf = *reinterpret_cast<const v4i*>(&sVt[(c * 32 + ql) * VLD + (s * 32 + st * 16 + hh * 8) * 2]);
                    o[c] = mfma_hp<DT>(vf, pf, o[c]);
                }
            }
        }
    }
    l += __shfl_xor(l, 32);
    if (qi >= a.Sq) return;
    // (a score beyond fp32: the fma's exponent is -inf where the product alone, minus the maximum, was NaN)
    const float inv_l = m2 == INFINITY ? __builtin_nanf("") : (l > 0.0f ? 1.0f / l : 0.0f);
    const int64_t orow = ((int64_t)b * a.Sq + qi) * a.ldo + (int64_t)h * DH;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e0 = c * 32 + g * 8 + hh * 4;
            v2i w = {(int)pack2_hp<DT>(o[c][4 * g] * inv_l, o[c][4 * g + 1] * inv_l),
                     (int)pack2_hp<DT>(o[c][4 * g + 2] * inv_l, o[c][4 * g + 3] * inv_l)};
            *reinterpret_cast<v2i*>(a.out + orow + e0) = w;
        }
}

// ------------------------------------------------------------------------------------------
// Few query blocks: a block owns 32 queries and its NW waves split the keys (wave w: the 32-key steps w, w + NW, ..), each
// with K fragments straight from memory, V transposed through LDS of its own, and an online softmax of its own; the waves'
// (maximum, sum, output) meet in LDS at the end, added in the order of the waves.  The kernel above runs such a launch as one
// serial chain per block on as many CUs as there are blocks of 128 queries.  Bound by latency.
// ------------------------------------------------------------------------------------------
template <int DH, int DT, int NW>
__global__ __launch_bounds__(64 * NW) void bf16_attn_split_kernel(BAttnArgs a) {
    constexpr int SQ = 32, SK = 32, VLD = SK * 2 + 16, DS = DH / 16, CT = DH / 32, CPRW = DH / 8, VU = (SK / 2) * CPRW / 64, TLD = 36;
    __shared__ __attribute__((aligned(16))) int8_t pool[NW * DH * VLD > NW * SQ * TLD * 4 ? NW * DH * VLD : NW * SQ * TLD * 4];
    __shared__ float sm[NW][SQ], sl[NW][SQ];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hh = lane >> 5, ql = lane & 31;
    const int nqb = (a.Sq + SQ - 1) / SQ;                        // all query blocks of one (batch, head) on one XCD, as above
    const int slot = blockIdx.x / 8, bh = (slot / nqb) * 8 + (int)(blockIdx.x % 8);
    if (bh >= a.B * a.H) return;
    const int b = bh / a.H, h = bh % a.H, q0 = (slot % nqb) * SQ;
    const int len = a.kv_len ? min(max(a.kv_len[b], 0), a.Skv) : a.Skv;
    const int shift = len - a.Sq, qi = q0 + ql;
    int nvis = len, kmax = len;
    if (a.mask == HERO_MASK_CAUSAL) {
        nvis = min(len, qi + shift + 1);
        kmax = min(len, min(q0 + SQ, a.Sq) + shift);
    }
    nvis = max(nvis, 0);
    if (a.mask == HERO_MASK_PADDING && a.Sq == a.Skv) {          // padded positions ask nothing
        if (qi >= len) nvis = 0;
        if (q0 >= len) kmax = 0;
    }
    const int nsteps = (max(kmax, 0) + SK - 1) / SK;
    v4i qf[DS];
    {
        const uint16_t* qp = a.q + (int64_t)b * a.qs[0] + (int64_t)min(qi, a.Sq - 1) * a.qs[1] + (int64_t)h * a.qs[2];
#pragma unroll
        for (int d = 0; d < DS; ++d) qf[d] = *reinterpret_cast<const v4i*>(qp + d * 16 + hh * 8);
    }
    const uint16_t* const kbase = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[2] + hh * 8;
    const uint16_t* const vbase = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[2];
    int8_t* const sv = pool + wave * DH * VLD;
    v4i kf[DS], rv[VU][2];
    auto load_k = [&](int step) {
        const uint16_t* p = kbase + (int64_t)min(step * SK + ql, a.Skv - 1) * a.ks[1];
#pragma unroll
        for (int d = 0; d < DS; ++d) kf[d] = *reinterpret_cast<const v4i*>(p + d * 16);
    };
    auto load_v = [&](int step) {                                // unit: 8 channels of two neighbouring keys
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int idx = lane + u * 64, rp = idx / CPRW, ch = idx % CPRW;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                rv[u][j] = *reinterpret_cast<const v4i*>(vbase + (int64_t)min(step * SK + 2 * rp + j, a.Skv - 1) * a.vs[1] + ch * 8);
        }
    };
    auto store_v = [&]() {
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int idx = lane + u * 64, rp = idx / CPRW, ch = idx % CPRW, row = 2 * rp;
            const int g4 = row >> 3, hp = (row >> 2) & 1, t = row & 3;      // the key order of the PV fragment (see above)
            const int pos = (g4 >> 1) * 16 + hp * 8 + (g4 & 1) * 4 + t;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t w0 = (uint32_t)rv[u][0][j], w1 = (uint32_t)rv[u][1][j];
                *reinterpret_cast<uint32_t*>(&sv[(ch * 8 + 2 * j) * VLD + pos * 2]) = __builtin_amdgcn_perm(w1, w0, 0x05040100u);
                *reinterpret_cast<uint32_t*>(&sv[(ch * 8 + 2 * j + 1) * VLD + pos * 2]) = __builtin_amdgcn_perm(w1, w0, 0x07060302u);
            }
        }
    };
    const float c2 = a.scale * 1.44269504088896340736f;
    float m2 = -INFINITY, l = 0.0f;
    v16f o[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[c][r] = 0.0f;
    if (wave < nsteps) { load_k(wave); load_v(wave); }
    for (int step = wave; step < nsteps; step += NW) {
        store_v();
        v16f acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int d = 0; d < DS; ++d) acc = mfma_hp<DT>(kf[d], qf[d], acc);
        if (step + NW < nsteps) { load_k(step + NW); load_v(step + NW); }
        float tmax = -INFINITY;
        const int lim = nvis - (step * SK + hh * 4);             // key visible iff 8g + t < lim
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[r] = ((r >> 2) * 8 + (r & 3)) < lim ? acc[r] * c2 : -INFINITY;
            tmax = fmaxf(tmax, acc[r]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        uint32_t pb[8];
        if (tmax > -INFINITY) {
            const float mn = fmaxf(m2, tmax), resc = __builtin_amdgcn_exp2f(m2 - mn);
            float sum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float e0 = __builtin_amdgcn_exp2f(acc[r] - mn), e1 = __builtin_amdgcn_exp2f(acc[r + 1] - mn);
                const uint32_t pk = pack2_hp<DT>(e0, e1);
                sum += hp_to_f32<DT>(pk & 0xffffu) + hp_to_f32<DT>(pk >> 16);           // the sum of what PV really multiplies
                pb[r >> 1] = pk;
            }
            l = fmaf(l, resc, sum);
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[c][r] *= resc;
            m2 = mn;
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) pb[r] = 0;
        }
        // the wave reads what its own lanes wrote: LDS operations of one wave keep their order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < 2; ++s) {                            // registers 0..7 feed the first 16-key step, 8..15 the second
            const v4i pf = {(int)pb[4 * s], (int)pb[4 * s + 1], (int)pb[4 * s + 2], (int)pb[4 * s + 3]};
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const v4i vf = *reinterpret_cast<const v4i*>(&sv[(c * 32 + ql) * VLD + (s * 16 + hh * 8) * 2]);
                o[c] = mfma_hp<DT>(vf, pf, o[c]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    l += __shfl_xor(l, 32);
    if (hh == 0) { sm[wave][ql] = m2; sl[wave][ql] = l; }
    __syncthreads();
    float M = sm[0][ql];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm[w][ql]);
    float L = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { const float lw = sl[w][ql]; if (lw > 0.0f) L = fmaf(lw, __builtin_amdgcn_exp2f(sm[w][ql] - M), L); }
    const float f = l > 0.0f ? __builtin_amdgcn_exp2f(m2 - M) * (1.0f / L) : 0.0f;      // this wave's share, normalised
    float* const tile = reinterpret_cast<float*>(pool);
#pragma unroll
    for (int c = 0; c < CT; ++c) {                               // 32 channels at a time: [wave][query][channel]
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<v4f*>(tile + (wave * SQ + ql) * TLD + g * 8 + hh * 4) =
                v4f{o[c][4 * g] * f, o[c][4 * g + 1] * f, o[c][4 * g + 2] * f, o[c][4 * g + 3] * f};
        __syncthreads();
        if (tid < SQ * 8) {
            const int q = tid >> 3, e0 = c * 32 + (tid & 7) * 4;
            v4f tot = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const v4f p = *reinterpret_cast<const v4f*>(tile + (w * SQ + q) * TLD + (tid & 7) * 4);
#pragma unroll
                for (int t = 0; t < 4; ++t) tot[t] += p[t];
            }
            if (q0 + q < a.Sq)
                *reinterpret_cast<v2i*>(a.out + ((int64_t)b * a.Sq + q0 + q) * a.ldo + (int64_t)h * DH + e0) =
                    v2i{(int)pack2_hp<DT>(tot[0], tot[1]), (int)pack2_hp<DT>(tot[2], tot[3])};
        }
    }
}

__global__ void zero_bf16_kernel(uint16_t* out, int64_t rows, int64_t cols, int64_t ld) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows * cols) out[(i / cols) * ld + i % cols] = 0;
}

}  // namespace

extern "C" hero_status hero_bf16_attn(const void* q, const int64_t q_strides[4],
                                      const void* k, const int64_t k_strides[4],
                                      const void* v, const int64_t v_strides[4],
                                      int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh, float scale,
                                      hero_mask mask, const int32_t* kv_len, void* out, int64_t ldo, void* stream) {
    return hero_hp_attn(q, q_strides, k, k_strides, v, v_strides, B, H, Sq, Skv, Dh, scale, mask, kv_len, out, ldo, HERO_BF16, stream);
}

extern "C" hero_status hero_hp_attn(const void* q, const int64_t q_strides[4],
                                    const void* k, const int64_t k_strides[4],
                                    const void* v, const int64_t v_strides[4],
                                    int64_t B, int64_t H, int64_t Sq, int64_t Skv, int64_t Dh, float scale,
                                    hero_mask mask, const int32_t* kv_len, void* out, int64_t ldo, hero_dtype dt, void* stream) {
    if (dt != HERO_BF16 && dt != HERO_F16) return HERO_ERR_UNSUPPORTED;
    if (B < 0 || H < 0 || Sq < 0 || Skv < 0) return HERO_ERR_SHAPE;
    if (Dh != 64 && Dh != 128) return HERO_ERR_UNSUPPORTED;
    if (mask != HERO_MASK_NONE && mask != HERO_MASK_PADDING && mask != HERO_MASK_CAUSAL) return HERO_ERR_UNSUPPORTED;
    if (B == 0 || H == 0 || Sq == 0) return HERO_OK;
    if (!out || !q_strides || !k_strides || !v_strides) return HERO_ERR_NULL;
    if (Skv > 0 && (!q || !k || !v)) return HERO_ERR_NULL;
    if (mask == HERO_MASK_PADDING && !kv_len) return HERO_ERR_NULL;
    if (ldo < H * Dh) return HERO_ERR_SHAPE;
    if (B > 65535 || H > 65535 || Sq > 0x7fffffffLL || Skv > 0x7fffffffLL) return HERO_ERR_SHAPE;
    const int64_t* ss[3] = {q_strides, k_strides, v_strides};
    for (int t = 0; t < 3; ++t) {
        if (ss[t][3] != 1) return HERO_ERR_UNSUPPORTED;
        if (ss[t][0] % 8 || ss[t][1] % 8 || ss[t][2] % 8) return HERO_ERR_ALIGN;
    }
    if (ldo % 4 || !hero_aligned16(out) || !hero_aligned16(q) || !hero_aligned16(k) || !hero_aligned16(v)) return HERO_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    if (Skv == 0) {
        const int64_t n = B * Sq * H * Dh;
        hipLaunchKernelGGL(zero_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint16_t*)out, B * Sq, H * Dh, ldo);
        return hero_launch_status();
    }
    BAttnArgs a;
    a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
    for (int t = 0; t < 4; ++t) { a.qs[t] = q_strides[t]; a.ks[t] = k_strides[t]; a.vs[t] = v_strides[t]; }
    a.B = (int)B; a.H = (int)H; a.Sq = (int)Sq; a.Skv = (int)Skv; a.scale = scale; a.mask = (int)mask; a.kv_len = kv_len;
    a.out = (uint16_t*)out; a.ldo = ldo;
    // At most one 128-query block per two CUs, or a single 32-query piece: the keys are split over the waves.  Measured, us, block of
    // 128 queries -> split: 7 x 12 heads x 93 7.3 -> 5.7, 2 x 16 x 512 17.4 -> 11.6, 1 x 32 x 400 causal 21.8 -> 18.2; with 192 or 256
    // blocks 33.8 -> 40.9 (1 x 32 x 700), 8.4 -> 10.0 (16 x 16 x 128).  Dh = 128 with two 32-query pieces per CU: only over more than
    // 384 keys (1 x 32 x 512 25.7 -> 23.2, 4 x 32 x 128 10.0 -> 10.5); a single piece of at most 128 keys, Dh = 64: up to three per CU
    // (768 x 32 keys 5.4 -> 5.0, 1024 6.1 -> 6.8).  Against 64 bits the split's own output is the
    // closer one by 2-4 % (behind a layer's codes the two cannot be told apart).
    const int64_t pieces = B * H * ((Sq + 31) / 32);
    const bool split = Sq <= 32 ? Dh == 128 || pieces <= 768 || Skv > 128
                                : B * H * ((Sq + ABQ - 1) / ABQ) <= 128 && (Dh == 64 || pieces <= 448 || (pieces <= 512 && Skv > 384));
    if (split) {
        const int64_t nb = ((B * H + 7) / 8) * 8 * ((Sq + 31) / 32);
        if (nb > 0x7fffffffLL) return HERO_ERR_SHAPE;
        const dim3 sgrid((unsigned)nb), sblock(256);
        if (dt == HERO_BF16) {
            if (Dh == 64) hipLaunchKernelGGL((bf16_attn_split_kernel<64, HERO_BF16, 4>), sgrid, sblock, 0, st, a);
            else hipLaunchKernelGGL((bf16_attn_split_kernel<128, HERO_BF16, 4>), sgrid, sblock, 0, st, a);
        } else {
            if (Dh == 64) hipLaunchKernelGGL((bf16_attn_split_kernel<64, HERO_F16, 4>), sgrid, sblock, 0, st, a);
            else hipLaunchKernelGGL((bf16_attn_split_kernel<128, HERO_F16, 4>), sgrid, sblock, 0, st, a);
        }
        return hero_launch_status();
    }
    const int64_t nblocks = ((B * H + 7) / 8) * 8 * ((Sq + ABQ - 1) / ABQ);   // whole rounds of 8 heads, one per XCD
    if (nblocks > 0x7fffffffLL) return HERO_ERR_SHAPE;
    dim3 grid((unsigned)nblocks);
    if (dt == HERO_BF16) {
        if (Dh == 64) hipLaunchKernelGGL((bf16_attn_kernel<64, HERO_BF16>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((bf16_attn_kernel<128, HERO_BF16>), grid, dim3(256), 0, st, a);
    } else {
        if (Dh == 64) hipLaunchKernelGGL((bf16_attn_kernel<64, HERO_F16>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((bf16_attn_kernel<128, HERO_F16>), grid, dim3(256), 0, st, a);
    }
    return hero_launch_status();
}
