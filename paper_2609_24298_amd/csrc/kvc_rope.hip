// RoPE-aware decode attention over the packed cache on CDNA4 (gfx950): the partials kernel of
// kvc_decode_attn_rope (Sec. 5: keys are compressed before RoPE).
//
// A model with rotary embeddings scores the rotated query q' against each reconstructed key rotated at its
// own position; that depends on the position and cannot be folded into a rank-space query, so the keys are
// rebuilt. One wavefront per (unit, context chunk) walks the chunk in 64-token tiles; in the block of
// token st (the tokens 4 col + st, col = 0..15), position t = t0 + st + 4 col:
//  1. K^T (128 features x 16 tokens) = P_K^T Z^T on v_mfma_f32_16x16x32_f16, the centred codes straight from
//     the packed fields in registers (k_pairs), P_K^T in LDS, shared by the block's wavefronts. Lane
//     (col, kq) holds features 16 rb + 4 kq + v of token 4 col + st, so both members of every rotation pair
//     (j, j + 64) sit in the same lane;
//  2. the rotation splits: the lane rotates its key by 4 col positions (factors constant over the whole
//     chunk, in LDS) and the query side takes the rest, R_-(t0 + st) q', as an operand formed once per tile:
//     row 4 h + st of the A operand is head h for block st, so that the block's logits of head h land in
//     element st of lane row h, which is the layout of the rank-space decode's softmax. R_-st q' is
//     tabulated (fp32) once per block and rotated by the tile's own angle (one fp64 product and one sine
//     and cosine per pair and tile, one lane each);
//  3. the logits on the same matrix instruction, query and key each split into fp16 hi + lo
//     (hi hi + hi lo + lo hi; the query first scaled by a power of two to the middle of the fp16 range, so
//     that its lo parts stay normal), the three products in accumulators of their own.
// Then the online softmax and the rank-space PV products as in the rank-space partials kernel, writing the
// same partials, which its combine kernel merges.
//
// Bound by VALU work per tile (unpacking, 64 rotation and 64 split operations per block) at two wavefronts
// per SIMD: 2048 units x 32k, 2 bpd, have the VALU busy 59 % of the time, the matrix cores 27 %, LDS 7 %; 256 units x
// 128k, 0.5 bpd, 73, 30 and 8 %.
#ifndef KVC_DECODE_PARTIALS_UNIT
#define KVC_DECODE_PARTIALS_UNIT
#endif
#include "kvc_decode.hip"

#include "kvc_codes.h"

namespace kvc {

template <int G> struct RopeShape {
    static constexpr int LM = Shape<G>::LM;
    static constexpr int W = 2;   // wavefronts per SIMD the register budget is cut for
    // Wavefronts per block at most (they share P_K^T and the query table): two blocks of four per CU, or one
    // of eight for G = 8, whose query table leaves room for two blocks only up to four wavefronts (rope_waves).
    static constexpr int kWaves = G == 8 ? 8 : 4;
    static constexpr int kPt = kBtBytes;                             // P_K^T
    static constexpr int kKey = 4 * 64 * 8 * 4;                      // cos, sin of 4 col positions: [rb][2][lane] float4
    static constexpr int kQry = LM * 8 * 64 * 16;                    // R_-st q': [lm][8][lane] float4
    static constexpr int kShared = kPt + kKey + kQry + 64 * 8 + 64;  // + frequencies (fp64), per-head logit scales
    static constexpr int kWave = 16 * LM * kPRowBytes + 64 * 8;      // probability limbs, the tile's cos, sin (+ staged K-step)
};

// K-steps of a k_mode, and the one that holds the tail group (2: none).
__host__ __device__ constexpr int k_steps(int km) { return km < 2 ? 2 : 1; }
__host__ __device__ constexpr int k_tail(int km) { return km == 1 ? 1 : (km == 3 ? 0 : 2); }

// hi + lo fp16 halves of x in element e of two operand fragments. m1 is -1 in a register the compiler does
// not know: x - hi stays one mixed-precision multiply-add that reads the half, not a conversion and a
// subtraction.
__device__ __forceinline__ void split_h(float x, float m1, rc_h8& hi, rc_h8& lo, int e) {
    const _Float16 h = (_Float16)x;
    hi[e] = h;
    lo[e] = (_Float16)fmaf((float)h, m1, x);
}

// Logits of a tile: s[lm][st] (log2 domain, plus off) of the lane's tokens 4 col + st and head 4 lm + grp.
// kb: the tile's K fields (NK K-steps).
template <int G, int B, int KM>
__device__ __forceinline__ void rope_logits(const uint32_t (&kb)[k_steps(KM) * 2 * B], const uint8_t* __restrict__ stage, uint32_t xb,
                                            uint32_t xs, const rc_h8 (&ah)[Shape<G>::LM][4], const rc_h8 (&al)[Shape<G>::LM][4],
                                            float m1, uint32_t e512, const float (&qs)[Shape<G>::LM], const float (&off)[Shape<G>::LM],
                                            float (&s)[Shape<G>::LM][4], int lane) {
    constexpr int NK = k_steps(KM), ks_t = k_tail(KM);
    constexpr int LM = Shape<G>::LM, W0 = k_step_words(B);
    const int col = lane & 15, grp = lane >> 4;
    // K^T of block st
    auto rebuild = [&](int st, rc_f4 (&Cr)[8]) {
        // Opaque LDS offset: the operands are the same for every block, and read again for each they take
        // no registers in between.
        int po = bt_lane(col, grp);
        asm volatile("" : "+v"(po));
        const uint8_t* pt = kvc_dsm + po;
#pragma unroll
        for (int rb = 0; rb < 8; ++rb) Cr[rb] = rc_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            rc_h8 z[2];
            Fld f[3];
            if (ks == ks_t) {
                k_fields_staged<B>(stage, xb + st * xs, f);
                k_pairs<B>(f, false, e512, z);
            } else {
                k_fields_direct<B>(kb + ks * W0, st, f);
                k_pairs<B>(f, (st & 1) != 0, e512, z);
            }
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int rb = 0; rb < 8; ++rb)
                    Cr[rb] = mfma_h(*reinterpret_cast<const rc_h8*>(pt + bt_block(rb, 2 * ks + m)), z[m], Cr[rb]);
        }
    };
    // rotation of block st by 4 col positions, the split, and the logits, two rotation pair groups at a time
    // (matrix step ks takes features 32 ks + ..: pair groups rb = 2 ks, 2 ks + 1 and their partners)
    auto score = [&](int st, const rc_f4 (&Cr)[8]) {
        int ko = RopeShape<G>::kPt + 16 * lane;
        asm volatile("" : "+v"(ko));
        const uint8_t* kc = kvc_dsm + ko;
        constexpr int NS = LM == 1 ? 3 : 1;  // one accumulator per product, or one in all (registers)
        rc_f4 S[LM][NS];
#pragma unroll
        for (int lm = 0; lm < LM; ++lm)
#pragma unroll
            for (int t = 0; t < NS; ++t) S[lm][t] = rc_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            rc_h8 xh, xl, yh, yl;  // features below and above d / 2
#pragma unroll
            for (int r2 = 0; r2 < 2; ++r2) {
                const float4 c0 = *reinterpret_cast<const float4*>(kc + ((2 * ks + r2) * 2) * 1024);
                const float4 c1 = *reinterpret_cast<const float4*>(kc + ((2 * ks + r2) * 2 + 1) * 1024);
                const float cc[4] = {c0.x, c0.z, c1.x, c1.z}, ss[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float a = Cr[2 * ks + r2][v], b = Cr[2 * ks + r2 + 4][v];
                    split_h(fmaf(a, cc[v], -b * ss[v]), m1, xh, xl, 4 * r2 + v);
                    split_h(fmaf(a, ss[v], b * cc[v]), m1, yh, yl, 4 * r2 + v);
                }
            }
#pragma unroll
            for (int lm = 0; lm < LM; ++lm) {
                S[lm][0] = mfma_h(ah[lm][ks], xh, S[lm][0]);
                S[lm][1 % NS] = mfma_h(ah[lm][ks], xl, S[lm][1 % NS]);
                S[lm][2 % NS] = mfma_h(al[lm][ks], xh, S[lm][2 % NS]);
                S[lm][0] = mfma_h(ah[lm][ks + 2], yh, S[lm][0]);
                S[lm][1 % NS] = mfma_h(ah[lm][ks + 2], yl, S[lm][1 % NS]);
                S[lm][2 % NS] = mfma_h(al[lm][ks + 2], yh, S[lm][2 % NS]);
            }
        }
#pragma unroll
        for (int lm = 0; lm < LM; ++lm)
            s[lm][st] = fmaf(NS == 3 ? S[lm][0][st] + (S[lm][1 % NS][st] + S[lm][2 % NS][st]) : S[lm][0][st], qs[lm], off[lm]);
    };
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        rc_f4 Cr[8];
        rebuild(st, Cr);
        score(st, Cr);
    }
}

// Runs CALL with B_ = the value width and NV_ = 4 or 8 value N-tiles (four for ranks <= 64 at up to 4 bits).
#define KVC_ROPE_V(bv, nv4, CALL)                                     \
    if (nv4) {                                                        \
        constexpr int NV_ = 4;                                        \
        switch (bv) {                                                 \
            case 1: { constexpr int B_ = 1; CALL; } break;            \
            case 2: { constexpr int B_ = 2; CALL; } break;            \
            case 3: { constexpr int B_ = 3; CALL; } break;            \
            default: { constexpr int B_ = 4; CALL; } break;           \
        }                                                             \
    } else {                                                          \
        constexpr int NV_ = 8;                                        \
        KVC_SWITCH_B(bv, CALL);                                       \
    }

template <int G, int B, int KM>
__device__ __attribute__((always_inline)) void rope_item(const DevSide& K, const DevSide& V, const uint8_t* __restrict__ sm,
                                                         uint8_t* __restrict__ wl, int u, int rk, int start, int end, int k_cap_tiles,
                                                         int v_cap_tiles, float* __restrict__ out, int lane) {
    using R = RopeShape<G>;
    constexpr int NK = k_steps(KM), ks_t = k_tail(KM);
    constexpr int LM = R::LM, W0 = k_step_words(B);
    float m1 = -1.f;
    asm volatile("" : "+s"(m1));
    const uint32_t e512 = exp512();
    constexpr bool kEarly = NK * W0 <= 16;  // the next tile's K fields have registers of their own
    const float4* qry = reinterpret_cast<const float4*>(sm + R::kPt + R::kKey);
    const double* om = reinterpret_cast<const double*>(sm + R::kPt + R::kKey + R::kQry);
    const float* qsc = reinterpret_cast<const float*>(sm + R::kPt + R::kKey + R::kQry + 64 * 8);
    uint8_t* pmat = wl;
    float2* tcs = reinterpret_cast<float2*>(wl + 16 * LM * kPRowBytes);  // [64 pairs] cos, sin of the tile's start
    uint8_t* stage = wl + R::kWave;
    const int col = lane & 15, grp = lane >> 4;
    const int rv = uni(V.r[u]), bv = uni(V.b[u]), hv = bv == 8 ? 0 : (1 << (bv - 1));
    const bool nv4 = rv <= 64 && bv <= 4;
    const int g16 = rk >> 4, rho = rk & 15;
    const int ktb = 8 * rk * B, vtb = 8 * rv * bv;
    const int tile0 = start / kTile, tile_last = (end - 1) / kTile;
    const uint8_t* kstream = uni(K.codes + K.code_off[u]);
    const uint8_t* vstream = uni(V.codes + V.code_off[u]);
    auto k_rs = [&](int t) {  // tile t of the stream (bounds: the stream's end); none past the chunk
        return __builtin_amdgcn_make_buffer_rsrc((void*)(kstream + (int64_t)t * ktb), (short)0,
                                                 t <= tile_last ? (k_cap_tiles - t) * ktb : 0, kRsrcWord3);
    };
    auto v_rs = [&](int t) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(vstream + (int64_t)t * vtb), (short)0,
                                                 t <= tile_last ? (v_cap_tiles - t) * vtb : 0, kRsrcWord3);
    };
    uint32_t LK[NK];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        const int cg = 4 * ks + grp;
        LK[ks] = ks == ks_t ? (uint32_t)(512 * ks + 8 * lane) : (cg < g16 ? (uint32_t)(128 * cg + 8 * col) : kLaneOOB);
    }
    uint32_t XB = 0, XS = 0;  // staged token fields start at plane-width units XB + st XS
    {
        const int nf = g16 - 4 * (ks_t < 2 ? ks_t : 0);
        if (grp < nf) { XB = (uint32_t)((64 * grp + 4 * col) * 16); XS = 16; }
        else if (grp == nf) { XB = (uint32_t)(nf * 1024 + 4 * col * rho); XS = (uint32_t)rho; }
    }
    const uint32_t LV = (uint32_t)(4 * col + grp), VA = v_lane_adj(rv, col, grp);
    const double om_lane = om[lane];
    float qs[LM], bias[LM], mrun[LM], mb[LM];
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) {
        qs[lm] = 4 * lm + grp < G ? qsc[4 * lm + grp] : 0.f;
        bias[lm] = 0.f;
        mrun[lm] = -INFINITY;
        mb[lm] = 0.f;
    }
    v4i C[LM][9];
#pragma unroll
    for (int pm = 0; pm < LM; ++pm)
#pragma unroll
        for (int nt = 0; nt < 9; ++nt) C[pm][nt] = v4i{0, 0, 0, 0};
    const uint32_t one = col == 0 ? 0x01010101u : 0u;
    const v4i ones = v4i{(int)one, (int)one, (int)one, (int)one};
    uint32_t kb[NK * W0], vb[kVBufWords];
    auto k_load = [&](uint32_t (&w)[NK * W0], int t) {
        const auto rs = k_rs(t);
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) k_load_direct<B>(rs, rk, LK[ks], w + ks * W0);
    };
    k_load(kb, tile0);
#pragma unroll
    for (int k = 0; k < kVBufWords; ++k) vb[k] = 0u;
    {
        const auto vrs = v_rs(tile0);
        KVC_ROPE_V(bv, nv4, (v_prefetch<B_, NV_>(vb, vrs, rv, LV, VA)));
    }
#pragma unroll 1
    for (int tile = tile0; tile <= tile_last; ++tile) {
        const int tok0 = tile * kTile;
        const bool first = tile == tile0;
        uint32_t kn[NK * W0];
        if constexpr (kEarly) k_load(kn, tile + 1);
        {  // cos, sin of the tile's first position for pair `lane` (turns reduced in fp64)
            const double t = (double)tok0 * om_lane;
            float c, sn;
            sincospif(2.f * (float)(t - rint(t)), &sn, &c);
            tcs[lane] = float2{c, sn};
        }
        if constexpr (ks_t < 2) k_write_stage<B>(kb + ks_t * W0, stage, lane);
        wave_lds_sync();
        // R_-(t0 + st) q' as fp16 hi + lo operands (rows 4 h + st)
        rc_h8 ah[LM][4], al[LM][4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const float4* t4 = reinterpret_cast<const float4*>(tcs + 16 * rb + 4 * grp);
            const float4 c0 = t4[0], c1 = t4[1];
            const float tc[4] = {c0.x, c0.z, c1.x, c1.z}, ts[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
            for (int lm = 0; lm < LM; ++lm) {
                const float4 qa4 = qry[(lm * 8 + rb) * 64 + lane], qb4 = qry[(lm * 8 + 4 + rb) * 64 + lane];
                const float qa[4] = {qa4.x, qa4.y, qa4.z, qa4.w}, qb[4] = {qb4.x, qb4.y, qb4.z, qb4.w};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    split_h(fmaf(qa[v], tc[v], qb[v] * ts[v]), m1, ah[lm][rb >> 1], al[lm][rb >> 1], 4 * (rb & 1) + v);
                    split_h(fmaf(qb[v], tc[v], -qa[v] * ts[v]), m1, ah[lm][2 + (rb >> 1)], al[lm][2 + (rb >> 1)], 4 * (rb & 1) + v);
                }
            }
        }
        float s[LM][4];
        rope_logits<G, B, KM>(kb, stage, XB, XS, ah, al, m1, e512, qs, mb, s, lane);
        if constexpr (kEarly) {
#pragma unroll
            for (int k = 0; k < NK * W0; ++k) kb[k] = kn[k];
        } else {
            k_load(kb, tile + 1);
        }

        // ---- online softmax, as in the rank-space decode
        bool raise = first;
        if (tok0 + kTile > end) {
#pragma unroll
            for (int lm = 0; lm < LM; ++lm)
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    if (tok0 + 4 * col + st >= end) s[lm][st] = -INFINITY;
        }
        if constexpr (G % 4 != 0) {  // rows of heads past G
#pragma unroll
            for (int lm = 0; lm < LM; ++lm)
                if (4 * lm + grp >= G) s[lm][0] = s[lm][1] = s[lm][2] = s[lm][3] = -INFINITY;
        }
        float ml[LM];
#pragma unroll
        for (int lm = 0; lm < LM; ++lm) {
            ml[lm] = fmaxf(fmaxf(s[lm][0], s[lm][1]), fmaxf(s[lm][2], s[lm][3]));
            raise = raise || ml[lm] > kLazy;
        }
        if (__any(raise)) raise_max<LM>(first, ml, bias, s, mrun, mb, C);
        write_limbs<LM>(s, pmat, col, grp);
        wave_lds_sync();
        v4i ap[LM];
#pragma unroll
        for (int pm = 0; pm < LM; ++pm)
            ap[pm] = *reinterpret_cast<const v4i*>(pmat + (16 * pm + col) * kPRowBytes + 16 * grp);
        {
            // opaque copies: the offsets of every width are recomputed here, not kept live across the loop
            uint32_t LVt = LV, VAt = VA;
            int rvt = rv;
            asm volatile("" : "+v"(LVt), "+v"(VAt));
            asm volatile("" : "+s"(rvt));
            const auto vrs = v_rs(tile), vrs_n = v_rs(tile + 1);
            KVC_ROPE_V(bv, nv4, (v_tile<B_, LM, NV_>(vb, vrs, vrs_n, rvt, LVt, VAt, ap, C)));
        }
#pragma unroll
        for (int pm = 0; pm < LM; ++pm) C[pm][8] = mfma_i8(ap[pm], ones, C[pm][8]);
        wave_lds_sync();  // pmat, the tile's angles and the staged K-step are rewritten by the next tile
    }
    write_partial<G>(C, mrun, rv, hv, out, lane);
}

// Block (chunks blockIdx.x nw .., unit, heads blockIdx.z G .. of the unit's Gq): one wavefront per chunk, nw of them.
template <int G>
__global__ __launch_bounds__(64 * RopeShape<G>::kWaves) __attribute__((amdgpu_waves_per_eu(RopeShape<G>::W, RopeShape<G>::W)))
void decode_rope_kernel(DevSide K, DevSide V, const uint16_t* __restrict__ q, int Gq, const int32_t* __restrict__ seq_len, int max_seq,
                        int chunk, int n_chunks, int k_cap_tiles, int v_cap_tiles, double log2_base, int wave_lds,
                        float* __restrict__ part) {
    using R = RopeShape<G>;
    constexpr int LM = R::LM;
    const int nw = G == 8 ? uni((int)(blockDim.x >> 6)) : R::kWaves, T = 64 * nw;
    const int u = blockIdx.y, tid = threadIdx.x, wv = uni(tid >> 6), lane = tid & 63, col = lane & 15, grp = lane >> 4;
    const int rk = uni(K.r[u]), bk = uni(K.b[u]);
    uint8_t* sm = kvc_dsm;
    float* key_cs = reinterpret_cast<float*>(sm + R::kPt);
    float4* qry = reinterpret_cast<float4*>(sm + R::kPt + R::kKey);
    double* om = reinterpret_cast<double*>(sm + R::kPt + R::kKey + R::kQry);
    float* qsc = reinterpret_cast<float*>(sm + R::kPt + R::kKey + R::kQry + 64 * 8);
    if (tid < 64) om[tid] = exp2(-(double)tid / 64.0 * log2_base) * 0.15915494309189535;  // turns per position of pair tid
    stage_basis_t<KVC_SIDE_K>(sm, K.basis + K.basis_off[u], rk, tid, T);
    __syncthreads();
    // cos, sin of n positions of pair j (turns reduced in fp64)
    auto turn = [&](int n, int j, float& c, float& sn) {
        const double t = (double)n * om[j];
        sincospif(2.f * (float)(t - rint(t)), &sn, &c);
    };
    for (int e = tid; e < 64 * 16; e += T) {  // pair j = 16 rb + 4 kq + v of lane (col, kq)
        const int j = e >> 4, cc = e & 15, rb = j >> 4, kq = (j >> 2) & 3, v = j & 3;
        float c, sn;
        turn(4 * cc, j, c, sn);
        float* dst = key_cs + ((rb * 2 + (v >> 1)) * 64 + 16 * kq + cc) * 4 + (v & 1) * 2;
        dst[0] = c;
        dst[1] = sn;
    }
    for (int lm = wv; lm < LM; lm += nw) {  // row 4 h + st of the query operand: lane (col, grp), head 4 lm + col / 4
        const int hd = 4 * lm + (col >> 2), st = col & 3;
        float a[4][4], b[4][4], m = 0.f;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint16_t* qh = q + ((int64_t)u * Gq + G * blockIdx.z + (hd < G ? hd : 0)) * kD + 16 * rb + 4 * grp + v;
                a[rb][v] = hd < G ? h2f(qh[0]) : 0.f;
                b[rb][v] = hd < G ? h2f(qh[64]) : 0.f;
                m = fmaxf(m, fmaxf(fabsf(a[rb][v]), fabsf(b[rb][v])));
            }
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
        // largest entry to [2^8, 2^9): |rotated| < 2^10, and hi + lo keep 22 bits of it
        const int ex = m > 0.f ? 9 - __builtin_amdgcn_frexp_expf(m) : 0;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            float4 x, y;
            float* xp = &x.x;
            float* yp = &y.x;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float c, sn;
                turn(st, 16 * rb + 4 * grp + v, c, sn);
                const float av = ldexpf(a[rb][v], ex), bv = ldexpf(b[rb][v], ex);
                xp[v] = fmaf(av, c, bv * sn);
                yp[v] = fmaf(bv, c, -av * sn);
            }
            qry[(lm * 8 + rb) * 64 + lane] = x;
            qry[(lm * 8 + 4 + rb) * 64 + lane] = y;
        }
        // step_K log2(e) / sqrt(128), less the scaling of q'
        if (hd < G && st == 0 && grp == 0) qsc[hd] = ldexpf(K.delta[u] * 1.4426950408889634f * 0.08838834764831845f, -ex);
    }
    __syncthreads();
    const int c = blockIdx.x * nw + wv;
    if (c >= n_chunks) return;  // no block-wide barrier follows
    int Tn = uni(seq_len[u]);
    Tn = Tn < 0 ? 0 : (Tn > max_seq ? max_seq : Tn);
    const int start = uni(c * chunk), end = uni(min(Tn, start + chunk));
    float* __restrict__ out = part + (((int64_t)u * n_chunks + c) * Gq + G * blockIdx.z) * kPartStride;
    if (start >= end) {
        if (lane < G) { out[lane * kPartStride] = -INFINITY; out[lane * kPartStride + 1] = 0.f; }
        return;
    }
    uint8_t* wl = sm + R::kShared + wv * wave_lds;
    switch (k_mode(rk)) {
        case 0: KVC_SWITCH_B(bk, (rope_item<G, B_, 0>(K, V, sm, wl, u, rk, start, end, k_cap_tiles, v_cap_tiles, out, lane))); break;
        case 1: KVC_SWITCH_B(bk, (rope_item<G, B_, 1>(K, V, sm, wl, u, rk, start, end, k_cap_tiles, v_cap_tiles, out, lane))); break;
        case 2: KVC_SWITCH_B(bk, (rope_item<G, B_, 2>(K, V, sm, wl, u, rk, start, end, k_cap_tiles, v_cap_tiles, out, lane))); break;
        default: KVC_SWITCH_B(bk, (rope_item<G, B_, 3>(K, V, sm, wl, u, rk, start, end, k_cap_tiles, v_cap_tiles, out, lane))); break;
    }
}

#ifndef KVC_ROPE_UNIT
extern template __global__ void decode_rope_kernel<4>(DevSide, DevSide, const uint16_t*, int, const int32_t*, int, int, int, int,
                                                      int, double, int, float*);
extern template __global__ void decode_rope_kernel<8>(DevSide, DevSide, const uint16_t*, int, const int32_t*, int, int, int, int,
                                                      int, double, int, float*);

namespace {

constexpr int kLdsPerCu = 160 * 1024;

// Wavefronts per block for n_chunks chunks per unit. With G = 8 and few chunks the wavefronts of a block of eight
// past the last chunk would idle while its LDS keeps a second block off the CU: up to four chunks take blocks
// of four wavefronts (three where the widest staged K-step needs it), two per CU. 2048 units x 300 tokens,
// 2 bpd: 398 -> 238 us, sixteen heads 776 -> 452 (780 in one item of sixteen heads); 256 units x 8192 tokens,
// 3 bpd, sixteen heads (four chunks): 648 -> 428 (618). Five chunks and more fill most of a block of eight.
template <int G>
int rope_waves(int n_chunks, int wave_lds) {
    using R = RopeShape<G>;
    if (G != 8 || n_chunks > 4) return R::kWaves;
    int nw = 4;
    while (nw > 1 && 2 * (R::kShared + nw * wave_lds) > kLdsPerCu) --nw;
    return nw;
}

// Gq query heads per unit, G of them per item.
template <int G>
int launch_rope_g(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q, int Gq, const int32_t* seq_len, int32_t max_seq_len,
                  double log2_base, int stage_bytes, float* part, int* n_chunks, hipStream_t st) {
    using R = RopeShape<G>;
    const int U = k->n_units, tpu = (max_seq_len + kTile - 1) / kTile;
    const int kct = (k->capacity + kTile - 1) / kTile, vct = (v->capacity + kTile - 1) / kTile;
    const int wave_lds = R::kWave + (stage_bytes + 15) / 16 * 16;
    const size_t smem = (size_t)R::kShared + (size_t)R::kWaves * wave_lds;  // of the largest block
    if (smem > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)decode_rope_kernel<G>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return set_error(KVC_EDEVICE, "hipFuncSetAttribute: %s", hipGetErrorString(e));
    }
    // Chunks per unit (at most what the workspace holds): the count that minimises rounds of resident
    // wavefronts x (tiles per item + the block's set-up and an item's ends, about two tiles).
    const int64_t slots = (int64_t)device_cus() * 4 * R::W;
    int best_n = *n_chunks, best_c = (tpu + best_n - 1) / best_n;
    double best = -1.0;
    for (int n = 1; n <= *n_chunks; ++n) {
        const int c = (tpu + n - 1) / n;
        if ((tpu + c - 1) / c != n || c > kMaxChunkTiles) continue;
        const int64_t items = (int64_t)U * (Gq / G) * ((n + R::kWaves - 1) / R::kWaves) * R::kWaves;
        const double cost = (double)((items + slots - 1) / slots) * (c + 2.0) + 0.1 * c;
        if (best < 0.0 || cost < best) { best = cost; best_n = n; best_c = c; }
    }
    *n_chunks = best_n;
    const int nw = rope_waves<G>(best_n, wave_lds);
    hipLaunchKernelGGL(decode_rope_kernel<G>, dim3((best_n + nw - 1) / nw, U, Gq / G), dim3(64 * nw),
                       (size_t)R::kShared + (size_t)nw * wave_lds, st, dev_side(k), dev_side(v), q, Gq, seq_len, max_seq_len, best_c * kTile, best_n, kct, vct, log2_base, wave_lds, part);
    return check_launch("kvc_decode_attn_rope");
}

}  // namespace

int launch_rope_partials(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q, int32_t G, const int32_t* seq_len,
                         int32_t max_seq_len, double log2_base, int stage_bytes, float* part, int* n_chunks, hipStream_t st) {
    switch (G) {
        case 1: return launch_rope_g<1>(k, v, q, G, seq_len, max_seq_len, log2_base, stage_bytes, part, n_chunks, st);
        case 2: return launch_rope_g<2>(k, v, q, G, seq_len, max_seq_len, log2_base, stage_bytes, part, n_chunks, st);
        case 4: return launch_rope_g<4>(k, v, q, G, seq_len, max_seq_len, log2_base, stage_bytes, part, n_chunks, st);
        // sixteen heads as two items of eight, which rebuild the keys twice: at 16 the accumulators and query
        // operands take one wavefront per SIMD and spill (64 units x 16k, 2 bpd: 391 us in one, 199 us in two)
        default: return launch_rope_g<8>(k, v, q, G, seq_len, max_seq_len, log2_base, stage_bytes, part, n_chunks, st);
    }
}
#endif  // KVC_ROPE_UNIT

}  // namespace kvc
