// Decode attention over the packed KV-COBRA cache on CDNA4 (gfx950): kernels
// and the kvc_decode_attn launcher (table step 8; App. I, "Wall-clock at the
// primitive level").
//
// The logits and the probability-weighted sum of values are dense contractions
// in the rank space: S = Qt (G x r_K) . C_K^T (r_K x tokens) and
// A = P (G x tokens) . C_V (tokens x r_V). Both run on int8 matrix cores
// (v_mfma_i32_16x16x64_i8) with exact int32 accumulation:
//  * codes enter as int8 (raw codes for b <= 7; c - 128 for b = 8);
//  * the rank-space query q~ = P_K q is split into three balanced base-254
//    int8 limbs with a per-query scale (relative error ~1e-7 of max|q~|);
//  * the softmax weights p in [0, 2^6] (relative to the chunk's running max) are
//    quantised to P < 2^31 - 2^24 and split into four byte limbs,
//    P = S0 + 2^8 S1 + 2^16 S2 + 2^24 S3 (S0..S2 signed, S3 in [0, 127]). The
//    quantum is 2^-25 of the running max, so a chunk of n tokens loses at most
//    n 2^-26 of its mass to rounding (<= 2^-12 at the longest chunk, 2^14
//    tokens), whatever the shape of the attention;
//  * centring (c - 2^(b-1)) is exact in integers: the logits subtract
//    2^(b-1) sum_i Q_i, and the value accumulator carries an all-ones virtual
//    coordinate whose column gives sum_t P_t (also the softmax denominator).
//
// One wavefront per work item = (unit, context chunk) walks the chunk in
// 64-token tiles. Each lane loads the packed fields its operand fragments need
// straight into registers with buffer loads at loop-invariant offsets (the
// stream layout puts a token's codes of a group of 16 coordinates, and a
// quarter of 16 tokens of one value coordinate, in one bit field whose
// unpacking lands directly in MFMA operand order); the next tile's loads are in
// flight while the current one is computed. Only the K-step holding the tail
// group (r_K % 16 coordinates, token fields that are not word aligned) is staged
// through LDS and read back with funnel shifts. The logit lane (query head,
// column) receives the three limbs of one (head, token) logit and forms it alone;
// the online softmax keeps a lazily raised running max per head; probability
// limbs go through LDS into the A operand of the PV products, whose int32
// accumulators hold every limb of one (head, coordinate) in one lane, so a raise
// of the max rescales them exactly in place. A second kernel merges the chunks
// and applies step_V and the V basis.
//
// What bounds the partials: at 2 bpd (2048 units x 32k) HBM reads, near their ceiling, and each
// wavefront's serial chain per tile (203 VALU instructions, the VALU busy 48 % of the time, wavefronts
// ready but not issued 60 %); at 0.5 bpd (256 units x 128k, 152 VALU instructions per tile) the
// issue of VALU instructions, which keeps it busy 76 %.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <utility>

#include "kvc_append.h"
#include "kvc_device.h"
#include "kvc_internal.h"

namespace kvc {

constexpr int kD = KVC_HEAD_DIM;
constexpr int kTile = KVC_TILE_TOKENS;
constexpr int kPartStride = 132;  // floats per (item, query head): m, l, pad, pad, acc[128]
constexpr int kLimbs = 3;
constexpr float kLazy = 6.f;              // the running max is raised only when a tile beats it by > 2^6
constexpr float kPScale = 33292288.f;     // (2^31 - 2^24) / 2^6: p <= 2^6 maps to P <= 2^31 - 2^24
constexpr float kPBias = 8421504.f;       // 0x808080, the offsets of the three signed low limbs; the fma's
                                          // result is >= 2^23, so its rounding to nearest is the rounding of P
// Tiles per chunk at most: |S_l c| <= 2^15 per token keeps the int32 accumulators below 2^31
// (2^29 per chunk, plus at most 2^24 carried into a limb by a rescale), and bounds the rounding
// loss of a chunk's softmax mass (see kPScale).
constexpr int kMaxChunkTiles = 256;
constexpr int kPRowBytes = 80;            // LDS row of the probability limbs (64 tokens + pad)
constexpr uint32_t kLaneOOB = 0x10000000u;  // lane offset (in plane-width units) past any stream
constexpr int kRsrcWord3 = 0x00020000;    // raw buffer, 32-bit data format (gfx9 family)

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t sh) {
    return __builtin_amdgcn_alignbit(hi, lo, sh);
}

// Maximum over the 16 lanes of a DPP row (row rotations).
template <int N>
__device__ __forceinline__ float row_ror(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_max(float m) {
    m = fmaxf(m, row_ror<8>(m));
    m = fmaxf(m, row_ror<4>(m));
    m = fmaxf(m, row_ror<2>(m));
    return fmaxf(m, row_ror<1>(m));
}

// The partial kernel's work-group is one wavefront, whose LDS accesses execute in program order:
// between an LDS write and a read of the same bytes only the compiler's reordering of memory
// operations has to be stopped, which a wavefront-scope fence does without any wait.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- field unpacking

// One token's field (16 codes) of one plane: up to four 32-bit words, bit 0 aligned.
struct Fld {
    uint32_t w0, w1, w2, w3;
};

// The 16 codes of a field as int8 operand bytes: byte k of dword d holds the code at position
// kidx_b^-1(4 d + k) of the field, i.e. operand index 4 d + k <-> position pos_b(4 d + k).
// f[k] is plane k's field (widest first); hi1 selects the upper 16 bits of the word of a 1-bit
// plane (two tokens share a word there). b = 8 codes come out centred (c - 128).
template <int B>
__device__ __forceinline__ v4i unpack16(const Fld (&f)[3], bool hi1) {
    uint32_t D[4];
    if constexpr (B == 8) {
        D[0] = f[0].w0 ^ 0x80808080u;
        D[1] = f[0].w1 ^ 0x80808080u;
        D[2] = f[0].w2 ^ 0x80808080u;
        D[3] = f[0].w3 ^ 0x80808080u;
    } else if constexpr (B == 4) {  // nibble order
        constexpr uint32_t M = 0x0f0f0f0fu;
        D[0] = f[0].w0 & M;
        D[1] = (f[0].w0 >> 4) & M;
        D[2] = f[0].w1 & M;
        D[3] = (f[0].w1 >> 4) & M;
    } else {  // position 4 k + d -> byte k of dword d, for every plane
        D[0] = D[1] = D[2] = D[3] = 0u;
#pragma unroll
        for (int k = 0; k < n_planes(B); ++k) {
            const int P = plane_w(B, k), SH = plane_sh(B, k);
            uint32_t E[4];
            if (P == 4) {
                constexpr uint32_t M = 0x0f0f0f0fu;
                const uint32_t t02 = perm(f[k].w1, f[k].w0, 0x06040200u), t13 = perm(f[k].w1, f[k].w0, 0x07050301u);
                E[0] = t02 & M;
                E[1] = (t02 >> 4) & M;
                E[2] = t13 & M;
                E[3] = (t13 >> 4) & M;
            } else if (P == 2) {
                constexpr uint32_t M = 0x03030303u;
#pragma unroll
                for (int d = 0; d < 4; ++d) E[d] = (f[k].w0 >> (2 * d)) & M;
            } else {
                constexpr uint32_t M = 0x01010101u;
                const uint32_t x = perm(f[k].w0 >> 4, f[k].w0, hi1 ? 0x07030602u : 0x05010400u);
#pragma unroll
                for (int d = 0; d < 4; ++d) E[d] = (x >> d) & M;
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) D[d] |= E[d] << SH;
        }
    }
    return v4i{(int)D[0], (int)D[1], (int)D[2], (int)D[3]};
}

// Words of a K-step held per lane: 8 p bytes per plane of width p, either the fields of the lane's
// four tokens (direct) or its share of the staged region (the K-step holding the tail group: the
// plane's bytes from 512 p ks on, at most 496 p of them, 8 p bytes per lane).
__host__ __device__ constexpr int k_step_words(int b) { return 2 * b; }
__host__ __device__ constexpr int plane_stage_off(int b, int k) { return 512 * plane_off(b, k); }  // LDS bytes
constexpr int kKBufWords = 16;  // prefetch registers per side
// K-steps' words kept in the prefetch registers: both K-steps of the widths where they fit, also for the
// structure taken at run time (KM < 0); the one K-step of ranks <= 64 (KM >= 2) for every width.
__host__ __device__ constexpr bool k_prefetch_on(int b, int km) {
    return 2 * k_step_words(b) <= kKBufWords || (km >= 2 && k_step_words(b) <= kKBufWords);
}
// The second K-step's load is issued (absent K-steps read past the stream and return zero) wherever
// its words fit the registers, so that every tile issues the same loads.
__host__ __device__ constexpr bool k_second_load(int b) { return 2 * k_step_words(b) <= kKBufWords; }
constexpr int kVBufWords = 16;  // value prefetch registers
constexpr int kPrefetchDepth = 2;  // tiles of K and V loads in flight ahead of the one being processed (the
                                    // general path keeps one: its per-tile width switches need the registers)

// Value groups (v_field_off): a plane of width p keeps the fields of v_group(p) = 8 / p consecutive
// N-tiles of a lane together (16 bytes), so a lane reads a group of one plane with one 16-byte load.
__host__ __device__ constexpr int v_group(int p) { return v_group_ntiles(p); }
__host__ __device__ constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }
// Prefetch registers taken by the groups of the first n N-tiles, plane k's groups starting at word
// v_pf_base(b, k, n), and the N-tiles prefetched for a rank bound of NV N-tiles (whole groups that
// fit kVBufWords; the groups past them are loaded while the tile is processed).
__host__ __device__ constexpr int v_pf_base(int b, int k, int n) {
    int w = 0;
    for (int j = 0; j < k; ++j) w += 4 * cdiv(n, v_group(plane_w(b, j)));
    return w;
}
__host__ __device__ constexpr int v_pf_words(int b, int n) { return v_pf_base(b, n_planes(b), n); }
__host__ __device__ constexpr int v_pf_tiles(int b, int nv) {
    int n = nv;
    while (n > 0 && v_pf_words(b, n) > kVBufWords) --n;
    return n;
}

// Direct loads of one K-step's fields into w[0 .. 2B).
template <int B>
__device__ __forceinline__ void k_load_direct(const __amdgpu_buffer_rsrc_t rs, int r, uint32_t lk, uint32_t* w) {
    int o = 0;
#pragma unroll
    for (int k = 0; k < n_planes(B); ++k) {
        const int P = plane_w(B, k);
        const int voff = (int)(P * lk) + 8 * r * plane_off(B, k);
        if (P == 1) {
            const v2u v = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, 0, 0);
            w[o] = v[0];
            w[o + 1] = v[1];
        } else {
#pragma unroll
            for (int q = 0; q < P / 2; ++q) {
                const v4u v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16 * q, 0, 0);
                w[o + 4 * q] = v[0];
                w[o + 4 * q + 1] = v[1];
                w[o + 4 * q + 2] = v[2];
                w[o + 4 * q + 3] = v[3];
            }
        }
        o += 2 * P;
    }
}

// The lane's share of the staged region goes to LDS at 8 p lane of the plane's area.
template <int B>
__device__ __forceinline__ void k_write_stage(const uint32_t* w, uint8_t* __restrict__ stage, int lane) {
    int o = 0;
#pragma unroll
    for (int k = 0; k < n_planes(B); ++k) {
        const int P = plane_w(B, k);
        uint8_t* dst = stage + plane_stage_off(B, k) + 8 * P * lane;
        if (P == 1) {
            *reinterpret_cast<v2u*>(dst) = v2u{w[o], w[o + 1]};
        } else {
#pragma unroll
            for (int q = 0; q < P / 2; ++q)
                *reinterpret_cast<v4u*>(dst + 16 * q) = v4u{w[o + 4 * q], w[o + 4 * q + 1], w[o + 4 * q + 2], w[o + 4 * q + 3]};
        }
        o += 2 * P;
    }
}

// Fields of token st (0..3 of the lane's four) from one K-step's directly loaded words. A 1-bit plane's
// field is the upper half of its word for odd st (two tokens share a word).
template <int B>
__device__ __forceinline__ void k_fields_direct(const uint32_t* w, int st, Fld (&f)[3]) {
    int o = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k < n_planes(B)) {
            const int P = plane_w(B, k);
            if (P == 1) f[k] = Fld{w[o + (st >> 1)], 0u, 0u, 0u};
            else if (P == 2) f[k] = Fld{w[o + st], 0u, 0u, 0u};
            else if (P == 4) f[k] = Fld{w[o + 2 * st], w[o + 2 * st + 1], 0u, 0u};
            else f[k] = Fld{w[o + 4 * st], w[o + 4 * st + 1], w[o + 4 * st + 2], w[o + 4 * st + 3]};
            o += 2 * P;
        } else {
            f[k] = Fld{0u, 0u, 0u, 0u};
        }
    }
}

// Operand fragment of token st from one K-step's directly loaded fields.
template <int B>
__device__ __forceinline__ v4i k_frag_direct(const uint32_t* w, int st) {
    Fld f[3];
    k_fields_direct<B>(w, st, f);
    return unpack16<B>(f, (st & 1) != 0);
}

// Fields of a token from the staged K-step: its field of plane k starts at bit p * x of the plane's
// staged region.
template <int B>
__device__ __forceinline__ void k_fields_staged(const uint8_t* __restrict__ stage, uint32_t x, Fld (&f)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k < n_planes(B)) {
            const int P = plane_w(B, k);
            const uint32_t bit = x * (uint32_t)P;
            const uint32_t* s32 = reinterpret_cast<const uint32_t*>(stage + plane_stage_off(B, k)) + (bit >> 5);
            const uint32_t d0 = s32[0], d1 = s32[1];
            if (P <= 2) {
                f[k] = Fld{funnel(d1, d0, bit), 0u, 0u, 0u};
            } else if (P == 4) {
                const uint32_t d2 = s32[2];
                f[k] = Fld{funnel(d1, d0, bit), funnel(d2, d1, bit), 0u, 0u};
            } else {
                const uint32_t d2 = s32[2], d3 = s32[3], d4 = s32[4];
                f[k] = Fld{funnel(d1, d0, bit), funnel(d2, d1, bit), funnel(d3, d2, bit), funnel(d4, d3, bit)};
            }
        } else {
            f[k] = Fld{0u, 0u, 0u, 0u};
        }
    }
}

// Operand fragment of a token from the staged K-step.
template <int B>
__device__ __forceinline__ v4i k_frag_staged(const uint8_t* __restrict__ stage, uint32_t x) {
    Fld f[3];
    k_fields_staged<B>(stage, x, f);
    return unpack16<B>(f, false);
}

template <int B>
__device__ __forceinline__ void k_fetch(uint32_t* w, const __amdgpu_buffer_rsrc_t rs, int rk, uint32_t lk) {
    k_load_direct<B>(rs, rk, lk, w);
}

// Prefetch of a unit's first tile (both K-steps, for the widths whose two K-steps fit the prefetch
// registers; wider codes are loaded when their tile is processed).
template <int B, int KM>
__device__ __forceinline__ void k_prefetch(uint32_t (&kb)[kKBufWords], const __amdgpu_buffer_rsrc_t rs, int rk,
                                           const uint32_t (&LK)[2]) {
    constexpr int W0 = k_step_words(B);
    if constexpr (k_prefetch_on(B, KM)) {
        k_fetch<B>(kb, rs, rk, LK[0]);
        if constexpr (k_second_load(B)) k_fetch<B>(kb + W0, rs, rk, LK[1]);
    }
}

// Logit of token 4 col + st for the lane's heads: three int32 limb sums (of scales k0, 254 k2, k2) -> log2-domain
// value + off.
template <int LM>
__device__ __forceinline__ void logit_of(const v4i (&acc)[LM], const float (&k0)[LM], const float (&k2)[LM],
                                         const float (&off)[LM], float (&s)[LM][4], int st) {
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) {
        // Limbs 1 and 2 as one integer (|acc| <= 2^21, so a 24-bit multiply-add): a multiply-add and a
        // conversion fewer per logit. Narrow codes are bound by instructions: 256 units x 128k, 0.5 bpd,
        // 198 -> 191 us, 640 units x 64k, eight heads, 1 bpd, 438 -> 425.
        const float v = fmaf((float)(__mul24(acc[lm][1], 254) + acc[lm][2]), k2[lm], off[lm]);
        s[lm][st] = fmaf((float)acc[lm][0], k0[lm], v);
    }
}

// Logits of one tile: s[lm][st] = logit + off for the lane's four tokens. The K-step holding the tail
// group (if any) is staged in LDS; its token fields start at plane-width units xb + st xs. For the
// widths whose two K-steps are prefetched, each token column is finished right after its MFMAs and
// the next tile's fields are loaded into the freed registers; wider codes load each K-step here.
template <int B, int LM, int KM>
__device__ __forceinline__ void k_tile(uint32_t (&kb)[kKBufWords], uint32_t (&kb_next)[kKBufWords], bool stage_next,
                                       const __amdgpu_buffer_rsrc_t rs,
                                       const __amdgpu_buffer_rsrc_t rs_n, int rk, int nk_rt, int ks_t_rt,
                                       const uint32_t (&LK)[2], uint32_t xb, uint32_t xs, int lane,
                                       uint8_t* __restrict__ stage, const v4i (&qa)[2][LM], const float (&k0)[LM],
                                       const float (&k2)[LM], const float (&off)[LM],
                                       float (&s)[LM][4]) {
    constexpr int W0 = k_step_words(B);
    // K-step structure fixed at compile time when KM >= 0 (see k_mode), else taken at run time
    const int nk = KM >= 0 ? (KM < 2 ? 2 : 1) : nk_rt;
    const int ks_t = KM >= 0 ? (KM == 1 ? 1 : (KM == 3 ? 0 : 2)) : ks_t_rt;
    if constexpr (k_prefetch_on(B, KM)) {
        // The staged K-step goes to LDS first (constant indices into kb: a runtime one would move the
        // array to scratch memory). Every load below is issued unconditionally, in the same order on
        // every tile (absent K-steps read past the stream and return zero), so that the wait for a
        // tile's data counts exactly the younger loads still in flight.
        // The staged K-step of this tile is already in LDS when the caller staged it one tile ahead
        // (stage_next on the previous tile); otherwise it is written now.
        // Widths whose second K-step does not fit are prefetched only with one K-step (KM >= 2), and
        // their code below never forms the second K-step's registers.
        constexpr bool kTwo = k_second_load(B);
        if (!stage_next) {
            if (ks_t == 0) {
                k_write_stage<B>(kb, stage, lane);
                wave_lds_sync();
            } else if constexpr (kTwo) {
                if (ks_t == 1 && nk > 1) {
                    k_write_stage<B>(kb + W0, stage, lane);
                    wave_lds_sync();
                }
            }
        }
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            v4i acc[LM];
            {
                const v4i bk = ks_t == 0 ? k_frag_staged<B>(stage, xb + st * xs) : k_frag_direct<B>(kb, st);
#pragma unroll
                for (int lm = 0; lm < LM; ++lm) acc[lm] = mfma_i8(qa[0][lm], bk, v4i{0, 0, 0, 0});
            }
            if constexpr (kTwo) {
                if (nk > 1) {
                    const v4i bk = ks_t == 1 ? k_frag_staged<B>(stage, xb + st * xs) : k_frag_direct<B>(kb + W0, st);
#pragma unroll
                    for (int lm = 0; lm < LM; ++lm) acc[lm] = mfma_i8(qa[1][lm], bk, acc[lm]);
                }
            }
            logit_of<LM>(acc, k0, k2, off, s, st);
        }
        k_load_direct<B>(rs_n, rk, LK[0], kb);
        if constexpr (kTwo) k_load_direct<B>(rs_n, rk, LK[1], kb + W0);
        // stage the next tile's K-step (loaded into the other register set one tile ago) now, away from
        // the loop head
        if (stage_next) {
            wave_lds_sync();
            if (ks_t == 0) k_write_stage<B>(kb_next, stage, lane);
            else if constexpr (kTwo) {
                if (ks_t == 1 && nk > 1) k_write_stage<B>(kb_next + W0, stage, lane);
            }
            wave_lds_sync();
        }
    } else {
        v4i S[LM][4];
#pragma unroll
        for (int lm = 0; lm < LM; ++lm)
#pragma unroll
            for (int st = 0; st < 4; ++st) S[lm][st] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (ks >= nk) break;
            k_fetch<B>(kb, rs, rk, LK[ks]);
            if (ks == ks_t) {
                k_write_stage<B>(kb, stage, lane);
                wave_lds_sync();
            }
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const v4i bk = ks == ks_t ? k_frag_staged<B>(stage, xb + st * xs) : k_frag_direct<B>(kb, st);
#pragma unroll
                for (int lm = 0; lm < LM; ++lm) S[lm][st] = mfma_i8(qa[ks][lm], bk, S[lm][st]);
            }
            if (ks == ks_t) wave_lds_sync();
        }
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            v4i acc[LM];
#pragma unroll
            for (int lm = 0; lm < LM; ++lm) acc[lm] = S[lm][st];
            logit_of<LM>(acc, k0, k2, off, s, st);
        }
    }
}

// Group Q of plane k for this lane: field index L = 4 col + grp of every N-tile in the group, the
// lane's fields in N-tile order. Groups before the last hold g N-tiles (16 bytes per lane, lanes in
// order); the last holds the remaining m N-tiles, the lanes of coordinates col >= ct (the coordinates
// of a partial last N-tile) one field fewer, so lane L starts A = 4 max(0, col - ct) + [col >= ct] grp
// fields before L m. Groups past the rank read beyond it (bounded by the stream) into accumulator
// columns that are never output.
template <int B>
__device__ __forceinline__ v4u v_group_load(const __amdgpu_buffer_rsrc_t rs, int k, int Q, int r, uint32_t L,
                                            uint32_t A) {
    const int P = plane_w(B, k), g = v_group(P);
    const int nvt = (r + 15) >> 4;
    const int ql = (nvt - 1) / g, m = nvt - g * ql;
    const uint32_t in = Q == ql ? (uint32_t)(2 * P) * (L * (uint32_t)m - A) : 16u * L;
    const int voff = 8 * r * plane_off(B, k) + 1024 * Q + (int)in;
    // A multiple of 4 bytes, except for 1-bit planes, whose last group (the only one, r <= 128) may start
    // a lane's fields at 2 mod 4 bytes: the load takes the dword-aligned 16 bytes below (the lane's
    // fields, at most 14 bytes in that case, stay inside them) and v_tile shifts them into place.
    return __builtin_amdgcn_raw_buffer_load_b128(rs, voff & ~3, 0, 0);
}

// A of the lane (col, grp) for rank r.
__device__ __forceinline__ uint32_t v_lane_adj(int r, int col, int grp) {
    const int ct = r - 16 * (((r + 15) >> 4) - 1);
    return col >= ct ? (uint32_t)(4 * (col - ct) + grp) : 0u;
}

// Loads of the prefetched groups whose last N-tile (below NV) is nt, plane by plane: the prefetch of a
// tile issues them for nt = 0, 1, .. in the same order as the processing of a tile refills them.
template <int B, int NV>
__device__ __forceinline__ void v_refill(uint32_t* vb, const __amdgpu_buffer_rsrc_t rs, int r, uint32_t L, uint32_t A,
                                         int nt) {
    constexpr int NPF = v_pf_tiles(B, NV);
#pragma unroll
    for (int k = 0; k < n_planes(B); ++k) {
        const int g = v_group(plane_w(B, k)), Q = nt / g;
        const int last = (Q + 1) * g < NV ? (Q + 1) * g - 1 : NV - 1;
        if (Q < cdiv(NPF, g) && nt == last) {
            const v4u v = v_group_load<B>(rs, k, Q, r, L, A);
            uint32_t* w = vb + v_pf_base(B, k, NPF) + 4 * Q;
            w[0] = v[0];
            w[1] = v[1];
            w[2] = v[2];
            w[3] = v[3];
        }
    }
}

template <int B, int NV>
__device__ __forceinline__ void v_prefetch(uint32_t (&vb)[kVBufWords], const __amdgpu_buffer_rsrc_t rs, int r,
                                           uint32_t L, uint32_t A) {
#pragma unroll
    for (int nt = 0; nt < NV; ++nt) v_refill<B, NV>(vb, rs, r, L, A, nt);
}

// PV MFMAs of one tile (N-tiles nt < NV, a compile-time bound on the rank's N-tiles; the prefetched
// groups come from vb, the rest are loaded here as their first N-tile comes), then the next tile's
// prefetch (rs_next; a zero-sized descriptor when there is none).
template <int B, int LM, int NV>
__device__ __forceinline__ void v_tile(uint32_t* vb, const __amdgpu_buffer_rsrc_t rs, const __amdgpu_buffer_rsrc_t rs_next,
                                       int r, uint32_t L, uint32_t A, const v4i (&ap)[LM], v4i (&C)[LM][9]) {
    constexpr int NPF = v_pf_tiles(B, NV);
    // Every N-tile below NV is processed, also those past the rank: no branches, and every tile issues
    // the same loads in the same order, so the waits for a tile's data stay exact.
    uint32_t gw[3][4], w1[4];
#pragma unroll
    for (int nt = 0; nt < NV; ++nt) {
        Fld f[3];
        bool hi = false;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k < n_planes(B)) {
                const int P = plane_w(B, k), g = v_group(P), Q = nt / g, j = nt % g;
                const bool pf = Q < cdiv(NPF, g);
                if (!pf && j == 0) {
                    const v4u v = v_group_load<B>(rs, k, Q, r, L, A);
                    gw[k][0] = v[0];
                    gw[k][1] = v[1];
                    gw[k][2] = v[2];
                    gw[k][3] = v[3];
                }
                const uint32_t* w = pf ? vb + v_pf_base(B, k, NPF) + 4 * Q : gw[k];
                if (P == 1) {
                    // one group of m = ceil(r / 16) N-tiles: the lane's fields start at bit 16 (m L - A)
                    // mod 32 of the dword-aligned words; they are shifted down once, on the group's
                    // first N-tile, where the words are used (a shift right after the load would wait
                    // for it)
                    if (j == 0) {
                        const uint32_t sh = ((L * (uint32_t)((r + 15) >> 4) - A) & 1u) << 4;
                        w1[0] = funnel(w[1], w[0], sh);
                        w1[1] = funnel(w[2], w[1], sh);
                        w1[2] = funnel(w[3], w[2], sh);
                        w1[3] = w[3] >> sh;
                    }
                    f[k] = Fld{w1[j >> 1], 0u, 0u, 0u};
                    hi = (j & 1) != 0;
                } else if (P == 2) {
                    f[k] = Fld{w[j], 0u, 0u, 0u};
                } else if (P == 4) {
                    f[k] = Fld{w[2 * j], w[2 * j + 1], 0u, 0u};
                } else {
                    f[k] = Fld{w[0], w[1], w[2], w[3]};
                }
            } else {
                f[k] = Fld{0u, 0u, 0u, 0u};
            }
        }
        const v4i bv = unpack16<B>(f, hi);
#pragma unroll
        for (int pm = 0; pm < LM; ++pm) C[pm][nt] = mfma_i8(ap[pm], bv, C[pm][nt]);
        v_refill<B, NV>(vb, rs_next, r, L, A, nt);
    }
}

// ---------------------------------------------------------------- q~ limbs

// Per unit: q~_g = (step_K log2(e) / sqrt(d)) P_K q_g, sigma_g = max|q~_g| / 127 and three int8
// limbs with q~ ~ sigma (L0 + L1/254 + L2/254^2). The limbs are written as the logit MFMA's A
// operand of every lane: qa[u][ks][lm][lane] = 16 bytes, lane (grp, row = 4 (h % 4) + limb), lm = h / 4,
// operand byte m <-> coordinate 16 (4 ks + grp) + pos_b(m) (zero outside the rank, for limb 3 and for
// heads >= G). qk[u][h] = (sigma, 0, sigma / 254^2, bias) with
// bias = -2^(b-1) sum_limb k_limb sum_i L_limb,i (0 for b = 8, whose codes are centred on load).
typedef _Float16 qp_h8 __attribute__((ext_vector_type(8)));
typedef float qp_f4 __attribute__((ext_vector_type(4)));

// NW wavefronts per unit (1 when the units fill the device, 8 for a few units), wavefront w taking
// row blocks [w 8/NW, (w + 1) 8/NW). The projection Y = P_K Q (rank rows x query-head columns) runs on
// v_mfma_f32_16x16x32_f16 (exact fp16 products, fp32 accumulation): A = 16 basis rows x 32
// coordinates, B = 32 coordinates x 16 heads, four k-steps per row block, every operand loaded
// straight from global memory with up to four row blocks' loads in flight. Lane (kq, col) then holds
// rows 16 rb + 4 kq + v of head col; a head's max and limb sums reduce over its four lanes, then over
// the wavefronts through LDS.
template <int NW>
__device__ __forceinline__ void qprep_unit(const DevSide& K, const uint16_t* __restrict__ q, int G, int LM,
                                           v4i* __restrict__ qa, float4* __restrict__ qk, const int u) {
    constexpr int RB = 8 / NW;                 // row blocks per wavefront
    constexpr int HALF = RB > 4 ? 2 : 1;       // rounds of at most four row blocks' loads
    constexpr int RQ = RB / HALF;
    extern __shared__ uint8_t img[];  // [2][LM][64][16] operand image
    __shared__ float red_m[NW][16];
    __shared__ int red_l[NW][16][kLimbs];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4;
    const int r = K.r[u], b = K.b[u];
    const uint16_t* __restrict__ P = K.basis + K.basis_off[u];
    const int img_words = 2 * LM * 64 * 4;
    for (int k = threadIdx.x; k < img_words; k += 64 * NW) reinterpret_cast<uint32_t*>(img)[k] = 0u;
    __syncthreads();
    qp_f4 C[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) C[j] = qp_f4{0.f, 0.f, 0.f, 0.f};
    for (int h0 = 0; h0 < G; h0 += 16) {  // heads in groups of 16 columns
        const int g = h0 + col;
        qp_h8 B[4];
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4) {
            const uint4 w = g < G ? reinterpret_cast<const uint4*>(q + ((int64_t)u * G + g) * kD + 32 * k4 + 8 * kq)[0]
                                  : uint4{0u, 0u, 0u, 0u};
            B[k4] = __builtin_bit_cast(qp_h8, w);
        }
#pragma unroll
        for (int half = 0; half < HALF; ++half) {
            uint4 A[RQ][4];
#pragma unroll
            for (int rq = 0; rq < RQ; ++rq)
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    const int row = 16 * (RB * wv + RQ * half + rq) + col;
                    A[rq][k4] = row < r ? reinterpret_cast<const uint4*>(P + (int64_t)row * kD + 32 * k4 + 8 * kq)[0]
                                        : uint4{0u, 0u, 0u, 0u};
                }
#pragma unroll
            for (int rq = 0; rq < RQ; ++rq) {
                qp_f4 c = qp_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4)
                    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(qp_h8, A[rq][k4]), B[k4], c, 0, 0, 0);
                C[RQ * half + rq] = c;
            }
        }
        const int hk = b == 8 ? 0 : (1 << (b - 1));
        const float scale0 = K.delta[u] * 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)
        float m = 0.f;
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                C[j][v] *= scale0;
                m = fmaxf(m, fabsf(C[j][v]));
            }
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
        if constexpr (NW > 1) {
            if (kq == 0) red_m[wv][col] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, red_m[w][col]);
        }
        const float sigma = m > 0.f ? m / 127.f : 1.f;
        const int g16 = r >> 4;
        int lsum[kLimbs] = {0, 0, 0};
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * (RB * wv + j) + 4 * kq + v;  // rank coordinate
                if (i < r && g < G) {
                    const float x = C[j][v] / sigma;
                    const float l0 = fminf(fmaxf(rintf(x), -127.f), 127.f);
                    const float r1 = (x - l0) * 254.f;
                    const float l1 = fminf(fmaxf(rintf(r1), -127.f), 127.f);
                    const float r2 = (r1 - l1) * 254.f;
                    const float l2 = fminf(fmaxf(rintf(r2), -127.f), 127.f);
                    const int L[kLimbs] = {(int)l0, (int)l1, (int)l2};
                    // destination of coordinate i in the operand image
                    const int cg = i < 16 * g16 ? (i >> 4) : g16;
                    const int jpos = i - 16 * cg;
                    const int ks = cg >> 2, grp = cg & 3;
                    const int kidx = kidx_b(b, jpos);
#pragma unroll
                    for (int k = 0; k < kLimbs; ++k) {
                        img[(((ks * LM + (g >> 2)) * 64 + 16 * grp + 4 * (g & 3) + k) << 4) + kidx] = (uint8_t)(int8_t)L[k];
                        lsum[k] += L[k];
                    }
                }
            }
#pragma unroll
        for (int k = 0; k < kLimbs; ++k) {
            lsum[k] += __shfl_xor(lsum[k], 16);
            lsum[k] += __shfl_xor(lsum[k], 32);
        }
        if constexpr (NW > 1) {
            if (kq == 0)
#pragma unroll
                for (int k = 0; k < kLimbs; ++k) red_l[wv][col][k] = lsum[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kLimbs; ++k) {
                lsum[k] = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) lsum[k] += red_l[w][col][k];
            }
        }
        if (wv == 0 && kq == 0 && g < G) {
            const float k0 = sigma, k1 = sigma * (1.f / 254.f), k2 = sigma * (1.f / 64516.f);
            const float bias = -(float)hk * ((float)lsum[0] * k0 + (float)lsum[1] * k1 + (float)lsum[2] * k2);
            qk[(int64_t)u * G + g] = float4{k0, 0.f, k2, bias};
        }
        if constexpr (NW > 1) __syncthreads();  // red_m, red_l are rewritten by the next head group
    }
    __syncthreads();
    v4i* dst = qa + (int64_t)u * 2 * LM * 64;
    for (int k = threadIdx.x; k < 2 * LM * 64; k += 64 * NW) dst[k] = reinterpret_cast<const v4i*>(img)[k];
}

template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void qprep_kernel(
    DevSide K, const uint16_t* __restrict__ q, int G, int LM, v4i* __restrict__ qa, float4* __restrict__ qk) {
    qprep_unit<NW>(K, q, G, LM, qa, qk, blockIdx.x);
}

// The first launch of a fused decode step (kvc_decode_step): block (u, 0) projects unit u's queries
// (two wavefronts, four row blocks each), blocks (u, 1) and (u, 2) append the new token's key and
// value to unit u's streams (the append of kvc_encode_kv). The decode partials, launched next on the
// same stream, read the appended codes.
constexpr int kStepPrepThreads = 128;
static_assert(kStepPrepThreads == kAppThreads, "the append uses one thread per coordinate");
// Three wavefronts per SIMD (166 registers, none spilled): 1.5 times the resident blocks of the
// unconstrained allocation, so the 3 x units blocks run in fewer rounds.
#ifndef KVC_DECODE_PARTIALS_UNIT
__global__ __launch_bounds__(kStepPrepThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void step_prep_kernel(
    DevSide K, DevSide V, const uint16_t* __restrict__ q, int G, int LM, v4i* __restrict__ qa, float4* __restrict__ qk,
    const uint16_t* __restrict__ xk, int64_t xk_stride, const uint16_t* __restrict__ xv, int64_t xv_stride, int t_new) {
    if (blockIdx.y == 0) qprep_unit<2>(K, q, G, LM, qa, qk, blockIdx.x);
    else if (blockIdx.y == 1) append_unit(K, KVC_SIDE_K, xk, xk_stride, t_new, 1, blockIdx.x);
    else append_unit(V, KVC_SIDE_V, xv, xv_stride, t_new, 1, blockIdx.x);
}
#endif

// ---------------------------------------------------------------- partials

template <int G> struct Shape {
    static constexpr int LM = (G + 3) / 4;  // M-tiles of 16 rows = 4 heads x 4 limb slots (logits and PV)
    // Wavefronts per SIMD the register budget is cut for (512 / W registers per lane, no spills).
    static constexpr int W = G <= 4 ? 3 : 2;
};

// Runs a KVC_SWITCH_B-style CALL with B_ = the compile-time width BKc (BVc), or switches on the
// runtime width when it is 0.
#define KVC_SW_K(CALL)                                          \
    if constexpr (BKc != 0) {                                   \
        constexpr int B_ = BKc;                                 \
        CALL;                                                   \
    } else {                                                    \
        KVC_SWITCH_B(bk, CALL);                                 \
    }
#define KVC_SW_V(CALL)                                          \
    if constexpr (BVc != 0) {                                   \
        constexpr int B_ = BVc;                                 \
        CALL;                                                   \
    } else {                                                    \
        KVC_SWITCH_B(bv, CALL);                                 \
    }

// One work item (unit u, context chunk [start, end)) with the K and V bit widths fixed at compile
// time (BKc in 1..8, BVc in 1..4), or switched per tile (0: the general path for values wider than 4).
extern __shared__ __attribute__((aligned(16))) uint8_t kvc_dsm[];

// K-step structure of a rank: 0: two K-steps, no tail group; 1: two K-steps, the tail group in the
// second; 2: one K-step, no tail group; 3: one K-step holding the tail group.
__host__ __device__ constexpr int k_mode(int r) {
    return r > 64 ? ((r & 15) ? 1 : 0) : ((r & 15) ? 3 : 2);
}

// Wave-uniform copies of values the compiler cannot prove uniform (kept in scalar registers).
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ const uint8_t* uni(const uint8_t* p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return reinterpret_cast<const uint8_t*>(((uint64_t)hi << 32) | lo);
}

// Raise of the running maxima (rare): each head whose tile beats its max by more than 2^kLazy (every head
// on the first tile) takes the tile's own max, and its accumulators are rescaled (every limb of a (head,
// coordinate) sits in this lane): value = C0 + 2^8 C1 + 2^16 C2 + 2^24 C3 (exact in fp64: |value| <= 2^53)
// -> rint(value alpha), split again into C3 and three bytes. s holds the logits less the old max (the raw
// logits on the first tile), ml the lane's own maxima; mb = bias - max afterwards.
template <int LM>
__device__ __forceinline__ void raise_max(bool first, const float (&ml)[LM], const float (&bias)[LM], float (&s)[LM][4],
                                          float (&mrun)[LM], float (&mb)[LM], v4i (&C)[LM][9]) {
    float mx[LM];
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) mx[lm] = row_max(ml[lm]);
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) {
        if ((first && mx[lm] > -INFINITY) || mx[lm] > kLazy) {
            const float mold = mrun[lm];
            const float shift = first ? 0.f : mold;  // s + shift = the raw logit
            const float mnew = mx[lm] + shift;
            const float alpha = first ? 0.f : exp2f(mold - mnew);
            mrun[lm] = mnew;
            mb[lm] = bias[lm] - mnew;
#pragma unroll
            for (int st = 0; st < 4; ++st) s[lm][st] = (s[lm][st] + shift) - mnew;
            if (!first) {
                const double a = (double)alpha;
#pragma unroll
                for (int nt = 0; nt < 9; ++nt) {
                    const double v = ((double)C[lm][nt][0] + 256.0 * (double)C[lm][nt][1]) +
                                     (65536.0 * (double)C[lm][nt][2] + 16777216.0 * (double)C[lm][nt][3]);
                    const double vs = rint(v * a);
                    const double c3 = floor(vs * (1.0 / 16777216.0));
                    const double r3 = vs - 16777216.0 * c3;  // [0, 2^24): exact from here on
                    const double c2 = floor(r3 * (1.0 / 65536.0));
                    const double r2 = r3 - 65536.0 * c2;
                    const double c1 = floor(r2 * (1.0 / 256.0));
                    C[lm][nt][3] = (int)c3;
                    C[lm][nt][2] = (int)c2;
                    C[lm][nt][1] = (int)c1;
                    C[lm][nt][0] = (int)(r2 - 256.0 * c1);
                }
            }
        }
    }
}

// Probability limbs of the lane's four tokens: P'' = round(p kPScale) + 0x808080; bytes 0, 1, 2 (xor 0x80)
// and 3 are the limbs S0..S3 with P = S0 + 2^8 S1 + 2^16 S2 + 2^24 S3. LDS row 4 h + limb, bytes 4 col + st.
// Every lane writes (heads past G have -inf logits, so zero limbs): no divergent LDS writes.
template <int LM>
__device__ __forceinline__ void write_limbs(const float (&s)[LM][4], uint8_t* __restrict__ pmat, int col, int grp) {
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) {
        uint32_t P[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) P[st] = (uint32_t)fmaf(__builtin_amdgcn_exp2f(s[lm][st]), kPScale, kPBias);
        const uint32_t q01 = perm(P[1], P[0], 0x05010400u), q23 = perm(P[3], P[2], 0x05010400u);
        const uint32_t r01 = perm(P[1], P[0], 0x07030602u), r23 = perm(P[3], P[2], 0x07030602u);
        const uint32_t L0 = perm(q23, q01, 0x05040100u) ^ 0x80808080u;
        const uint32_t L1 = perm(q23, q01, 0x07060302u) ^ 0x80808080u;
        const uint32_t L2 = perm(r23, r01, 0x05040100u) ^ 0x80808080u;
        const uint32_t L3 = perm(r23, r01, 0x07060302u);
        uint8_t* row = pmat + (16 * lm + 4 * grp) * kPRowBytes + 4 * col;
        *reinterpret_cast<uint32_t*>(row) = L0;
        *reinterpret_cast<uint32_t*>(row + kPRowBytes) = L1;
        *reinterpret_cast<uint32_t*>(row + 2 * kPRowBytes) = L2;
        *reinterpret_cast<uint32_t*>(row + 3 * kPRowBytes) = L3;
    }
}

// Partial of each head: m, l = sum of P (all-ones column), centred accumulator. Lane (grp, col)
// holds every limb of head 4 pm + grp at coordinate 16 nt + col; the all-ones column is col 0.
template <int G>
__device__ __forceinline__ void write_partial(const v4i (&C)[Shape<G>::LM][9], const float (&mrun)[Shape<G>::LM], int rv, int hv,
                                              float* __restrict__ out, int lane) {
    const int col = lane & 15, grp = lane >> 4, nv = (rv + 15) >> 4;
#pragma unroll
    for (int pm = 0; pm < Shape<G>::LM; ++pm) {
        const int h = 4 * pm + grp;
        const int o0 = __shfl(C[pm][8][0], lane & 48), o1 = __shfl(C[pm][8][1], lane & 48),
                  o2 = __shfl(C[pm][8][2], lane & 48), o3 = __shfl(C[pm][8][3], lane & 48);
        if (G % 4 == 0 || h < G) {
            float* o = out + h * kPartStride;
            if (col == 0) {
                o[0] = mrun[pm];
                o[1] = ((float)o0 + 256.f * (float)o1) + (65536.f * (float)o2 + 16777216.f * (float)o3);
            }
#pragma unroll
            for (int nt = 0; nt < 8; ++nt) {
                const int cc = 16 * nt + col;
                if (nt < nv) {
                    const int a0 = C[pm][nt][0] - hv * o0, a1 = C[pm][nt][1] - hv * o1, a2 = C[pm][nt][2] - hv * o2,
                              a3 = C[pm][nt][3] - hv * o3;
                    o[4 + cc] = cc < rv ? ((float)a0 + 256.f * (float)a1) + (65536.f * (float)a2 + 16777216.f * (float)a3)
                                        : 0.f;
                }
            }
        }
    }
}

// Inlined into the kernel: each instantiation is a disjoint branch of the dispatch, so registers
// are allocated per branch, and no call frame saves registers to scratch memory on every item.
template <int G, int BKc, int BVc, int KM, int NVc>
__device__ __attribute__((always_inline)) void run_item(const DevSide& K, const DevSide& V, const v4i* __restrict__ qa_u, int ks_stride,
                                         const float4* __restrict__ qk_u, int k_cap_tiles, int v_cap_tiles, int u,
                                         int start, int end, float* __restrict__ out, int lane) {
    constexpr int LM = Shape<G>::LM;
    constexpr int kDepth = KM >= 0 ? kPrefetchDepth : 1;
    uint8_t* pmat = kvc_dsm;                            // [16 LM][kPRowBytes] probability limbs
    uint8_t* stage = kvc_dsm + 16 * LM * kPRowBytes;    // staged tail K-step
    const int col = lane & 15, grp = lane >> 4;
    u = uni(u);
    start = uni(start);
    end = uni(end);
    k_cap_tiles = uni(k_cap_tiles);
    v_cap_tiles = uni(v_cap_tiles);
    const int rk = uni(K.r[u]), bk = uni(K.b[u]), rv = uni(V.r[u]), bv = uni(V.b[u]);
    const int hv = bv == 8 ? 0 : (1 << (bv - 1));
    const int nk = (rk + 63) >> 6;
    const int g16 = rk >> 4, rho = rk & 15;
    const int ks_t = rho ? (g16 >> 2) : 2;  // K-step holding the tail group (2: none)
    const int ktb = 8 * rk * bk, vtb = 8 * rv * bv;
    const int tile0 = start / kTile, tile_last = (end - 1) / kTile;
    const uint8_t* kstream = uni(K.codes + K.code_off[u]);
    const uint8_t* vstream = uni(V.codes + V.code_off[u]);
    // Descriptor of tile t of a stream (bounds: the stream's end); none past the chunk.
    auto k_rs = [&](int t) {
        const bool ok = t <= tile_last;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(kstream + (int64_t)t * ktb), (short)0,
                                                 ok ? (k_cap_tiles - t) * ktb : 0, kRsrcWord3);
    };
    auto v_rs = [&](int t) {
        const bool ok = t <= tile_last;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(vstream + (int64_t)t * vtb), (short)0,
                                                 ok ? (v_cap_tiles - t) * vtb : 0, kRsrcWord3);
    };

    // lane constants (plane-width units): direct K fields of K-step ks (group 4 ks + grp, tokens 4 col ..),
    // value fields (coordinate col of the N-tile, quarter grp), staged tail positions.
    uint32_t LK[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int cg = 4 * ks + grp;
        LK[ks] = ks == ks_t ? (uint32_t)(512 * ks + 8 * lane) : (cg < g16 ? (uint32_t)(128 * cg + 8 * col) : kLaneOOB);
    }
    const uint32_t LV = (uint32_t)(4 * col + grp), VA = v_lane_adj(rv, col, grp);
    uint32_t XB = 0, XS = 0;  // staged token fields start at plane-width units XB + st XS
    {
        const int nf = g16 - 4 * (ks_t < 2 ? ks_t : 0);  // full groups in the staged K-step
        if (grp < nf) { XB = (uint32_t)((64 * grp + 4 * col) * 16); XS = 16; }
        else if (grp == nf) { XB = (uint32_t)(nf * 1024 + 4 * col * rho); XS = (uint32_t)rho; }
    }

    // q~ limbs (A operands of the logits) and per-head scale factors
    v4i qa[2][LM];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int lm = 0; lm < LM; ++lm) qa[ks][lm] = qa_u[ks * ks_stride + lm * 64 + lane];
    float k0[LM], k2[LM], bias[LM], mrun[LM], mb[LM];
#pragma unroll
    for (int lm = 0; lm < LM; ++lm) {
        const int h = 4 * lm + grp;
        const float4 v = h < G ? qk_u[h] : float4{0.f, 0.f, 0.f, 0.f};
        k0[lm] = v.x; k2[lm] = v.z; bias[lm] = v.w;
        mrun[lm] = -INFINITY;
        mb[lm] = 0.f;  // bias - mrun once the first tile has set mrun
    }
    for (int k = lane; k < 16 * LM * kPRowBytes / 4; k += 64) reinterpret_cast<uint32_t*>(pmat)[k] = 0u;
    wave_lds_sync();

    v4i C[LM][9];
#pragma unroll
    for (int pm = 0; pm < LM; ++pm)
#pragma unroll
        for (int nt = 0; nt < 9; ++nt) C[pm][nt] = v4i{0, 0, 0, 0};
    const uint32_t one = col == 0 ? 0x01010101u : 0u;
    const v4i ones = v4i{(int)one, (int)one, (int)one, (int)one};

    // Prefetch registers: with a depth of 2, tile t is processed from set t % 2 while the loads of
    // tile t + 1 (the other set) are in flight, and set t % 2 is refilled with tile t + 2 as it is
    // consumed; with a depth of 1 there is one set, refilled with tile t + 1.
    uint32_t kbA[kKBufWords], vbA[kVBufWords], kbB[kKBufWords], vbB[kVBufWords];
#pragma unroll
    for (int k = 0; k < kKBufWords; ++k) kbA[k] = kbB[k] = 0u;
#pragma unroll
    for (int k = 0; k < kVBufWords; ++k) vbA[k] = vbB[k] = 0u;
    {
        // issued in the loop's own order (K-steps, then value N-tiles, per set), so that the waits at
        // the loop head count the same younger loads on entry as on the back edge
        const auto krs = k_rs(tile0), vrs = v_rs(tile0);
        KVC_SW_K((k_prefetch<B_, KM>(kbA, krs, rk, LK)));
        __builtin_amdgcn_sched_barrier(0);
        KVC_SW_V((v_prefetch<B_, NVc>(vbA, vrs, rv, LV, VA)));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kDepth == 2) {
            const auto krs1 = k_rs(tile0 + 1), vrs1 = v_rs(tile0 + 1);
            KVC_SW_K((k_prefetch<B_, KM>(kbB, krs1, rk, LK)));
            __builtin_amdgcn_sched_barrier(0);
            KVC_SW_V((v_prefetch<B_, NVc>(vbB, vrs1, rv, LV, VA)));
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    auto step = [&](const int tile, uint32_t (&kb)[kKBufWords], uint32_t (&vb)[kVBufWords],
                    uint32_t (&kb_next)[kKBufWords], const bool stage_next) {
        const int tok0 = tile * kTile;
        const bool first = tile == tile0;
        const auto krs = k_rs(tile), vrs = v_rs(tile);
        const auto krs_n = k_rs(tile + kDepth), vrs_n = v_rs(tile + kDepth);
        // Opaque per-tile copies of the lane and rank constants: the offsets every bit width derives
        // from them are recomputed inside the loop instead of being hoisted and kept live across it
        // for all eight widths at once.
        uint32_t LKt[2] = {LK[0], LK[1]}, XBt = XB, XSt = XS, LVt = LV, VAt = VA;
        int rkt = rk, rvt = rv;
        if constexpr (BKc == 0 || BVc == 0) {
            asm volatile("" : "+v"(LKt[0]), "+v"(LKt[1]), "+v"(LVt), "+v"(VAt), "+v"(XBt), "+v"(XSt));
            asm volatile("" : "+s"(rkt), "+s"(rvt));
        }
        const int nkt = nk, kst = ks_t;

        // ---- logits, log2 domain, less the running max (the raw logits on the first tile)
        float s[LM][4];
        {
            float off[LM];
#pragma unroll
            for (int lm = 0; lm < LM; ++lm) off[lm] = first ? bias[lm] : mb[lm];
            KVC_SW_K((k_tile<B_, LM, KM>(kb, kb_next, stage_next, krs, krs_n, rkt, nkt, kst, LKt, XBt, XSt, lane, stage, qa, k0, k2, off, s)));
        }

        // ---- online softmax
        const bool last = tok0 + kTile > end;
        bool raise = first;
        if (last) {  // tokens past the end of the chunk
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
        // A head's row max beats kLazy exactly when one of its lanes' own maxima does: the common
        // path tests the lane maxima only and takes the cross-lane row max inside the rare branch.
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

        // ---- PV (value N-tiles, then the all-ones column)
        KVC_SW_V((v_tile<B_, LM, NVc>(vb, vrs, vrs_n, rvt, LVt, VAt, ap, C)));
#pragma unroll
        for (int pm = 0; pm < LM; ++pm) C[pm][8] = mfma_i8(ap[pm], ones, C[pm][8]);
        wave_lds_sync();  // pmat is rewritten by the next tile
    };
    if constexpr (kDepth == 2) {
        // pairs of tiles in a straight-line body (the load-wait counts stay exact across the back edge)
        // The staged (tail) K-step of tile t + 1 goes to LDS at the end of tile t's logits (the first
        // tile's before the loop); the general path stages each tile itself.
        constexpr bool kAhead = KM >= 0 && k_prefetch_on(BKc, KM);
        if constexpr (kAhead) {
            if (ks_t == 0) k_write_stage<BKc>(kbA, stage, lane);
            else if constexpr (k_second_load(BKc)) {
                if (ks_t == 1) k_write_stage<BKc>(kbA + k_step_words(BKc), stage, lane);
            }
            wave_lds_sync();
        }
        int tile = tile0;
        for (; tile + 1 <= tile_last; tile += 2) {
            step(tile, kbA, vbA, kbB, kAhead);
            step(tile + 1, kbB, vbB, kbA, kAhead);
        }
        if (tile <= tile_last) step(tile, kbA, vbA, kbB, kAhead);
    } else {
        for (int tile = tile0; tile <= tile_last; ++tile) step(tile, kbA, vbA, kbA, false);
    }

    write_partial<G>(C, mrun, rv, hv, out, lane);
}

#undef KVC_SW_K
#undef KVC_SW_V

// Token of logit column col in sub-tile st is 4 col + st: a lane's four tokens are consecutive, so
// its K fields are one contiguous load, and its probability limbs are one dword per limb in LDS.
template <int G>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Shape<G>::W, Shape<G>::W))) void decode_partial_kernel(
    DevSide K, DevSide V, int Gq, const v4i* __restrict__ qa_ws, const float4* __restrict__ qk_ws,
    const int32_t* __restrict__ seq_len, int max_seq, int chunk, int n_chunks, int k_cap_tiles, int v_cap_tiles,
    float* __restrict__ part) {
    constexpr int LM = Shape<G>::LM;

    const int u = blockIdx.y, c = blockIdx.x, lane = threadIdx.x;
    int T = seq_len[u];
    T = T < 0 ? 0 : (T > max_seq ? max_seq : T);
    const int start = c * chunk;
    const int end = min(T, start + chunk);
    // the item's heads: all of the unit's, except that sixteen are two items of eight
    const int Gu = G == 8 ? Gq : G, h0 = G == 8 ? G * (int)blockIdx.z : 0, ks_stride = (Gu + 3) / 4 * 64;
    float* __restrict__ out = part + (((int64_t)u * n_chunks + c) * Gu + h0) * kPartStride;
    if (start >= end) {
        if (lane < G) { out[lane * kPartStride] = -INFINITY; out[lane * kPartStride + 1] = 0.f; }
        return;
    }
    const v4i* __restrict__ qa_u = qa_ws + (int64_t)u * 2 * ks_stride + h0 / 4 * 64;
    const float4* __restrict__ qk_u = qk_ws + (int64_t)u * Gu + h0;
    const int bk = K.b[u], bv = V.b[u];
    // Compiled per (b_K, b_V, K-step structure) for value widths up to 4 and the common group sizes;
    // the general path switches on the widths per tile.
    if constexpr (G == 4 || G == 8) {
        if (bv <= 4) {
            // Value ranks <= 64 (four N-tiles) at 1-3 bits with keys up to 4 bits, and 3-bit values at
            // rank <= 96 (six N-tiles), have instantiations of their own.
            const int rv = V.r[u];
            const int nvc = rv <= 64 && bk <= 4 && bv <= 3 ? 2 : (bv == 3 && rv <= 96 ? 1 : 0);
            switch ((((bk - 1) * 4 + (bv - 1)) * 4 + k_mode(K.r[u])) * 3 + nvc) {
#define KVC_ITEM(BK, BV, KM, NV)                                                                                  \
    case (((BK - 1) * 4 + (BV - 1)) * 4 + KM) * 3 + (NV == 6 ? 1 : (NV == 4 ? 2 : 0)):                          \
        run_item<G, BK, BV, KM, NV>(K, V, qa_u, ks_stride, qk_u, k_cap_tiles, v_cap_tiles, u, start, end, out, lane);    \
        return;
#define KVC_ITEM4(BK, BV) KVC_ITEM(BK, BV, 0, 8) KVC_ITEM(BK, BV, 1, 8) KVC_ITEM(BK, BV, 2, 8) KVC_ITEM(BK, BV, 3, 8)
#define KVC_ITEM4N(BK, BV, NV) KVC_ITEM(BK, BV, 0, NV) KVC_ITEM(BK, BV, 1, NV) KVC_ITEM(BK, BV, 2, NV) KVC_ITEM(BK, BV, 3, NV)
#define KVC_ITEM4S(BK) KVC_ITEM4(BK, 3) KVC_ITEM4N(BK, 3, 6)
#define KVC_ITEMN4(BK) KVC_ITEM4N(BK, 1, 4) KVC_ITEM4N(BK, 2, 4) KVC_ITEM4N(BK, 3, 4)
                KVC_ITEM4(1, 1) KVC_ITEM4(1, 2) KVC_ITEM4S(1) KVC_ITEM4(1, 4) KVC_ITEMN4(1)
                KVC_ITEM4(2, 1) KVC_ITEM4(2, 2) KVC_ITEM4S(2) KVC_ITEM4(2, 4) KVC_ITEMN4(2)
                KVC_ITEM4(3, 1) KVC_ITEM4(3, 2) KVC_ITEM4S(3) KVC_ITEM4(3, 4) KVC_ITEMN4(3)
                KVC_ITEM4(4, 1) KVC_ITEM4(4, 2) KVC_ITEM4S(4) KVC_ITEM4(4, 4) KVC_ITEMN4(4)
                KVC_ITEM4(5, 1) KVC_ITEM4(5, 2) KVC_ITEM4S(5) KVC_ITEM4(5, 4)
                KVC_ITEM4(6, 1) KVC_ITEM4(6, 2) KVC_ITEM4S(6) KVC_ITEM4(6, 4)
                KVC_ITEM4(7, 1) KVC_ITEM4(7, 2) KVC_ITEM4S(7) KVC_ITEM4(7, 4)
                KVC_ITEM4(8, 1) KVC_ITEM4(8, 2) KVC_ITEM4S(8) KVC_ITEM4(8, 4)
#undef KVC_ITEMN4
#undef KVC_ITEM4N
#undef KVC_ITEM4S
#undef KVC_ITEM4
#undef KVC_ITEM
                default: break;
            }
        }
    }
    run_item<G, 0, 0, -1, 8>(K, V, qa_u, ks_stride, qk_u, k_cap_tiles, v_cap_tiles, u, start, end, out, lane);
}

// The instantiations for 4 and 8 query heads per KV head are compiled in translation units of their
// own (kvc_decode_g4.hip, kvc_decode_g8.hip), in parallel with this one.
#ifndef KVC_DECODE_PARTIALS_UNIT
extern template __global__ void decode_partial_kernel<4>(DevSide, DevSide, int, const v4i*, const float4*, const int32_t*, int,
                                                         int, int, int, int, float*);
extern template __global__ void decode_partial_kernel<8>(DevSide, DevSide, int, const v4i*, const float4*, const int32_t*, int,
                                                         int, int, int, int, float*);
#endif

#ifndef KVC_DECODE_PARTIALS_UNIT
// ---------------------------------------------------------------- combine

// One block of four wavefronts per (unit, GB query heads). The chunks' partials merge in the log2 domain
// (M = max m_c, L = sum l_c 2^(m_c - M), A_j = sum acc_c,j 2^(m_c - M)), z_j = step_V (A_j / L + 1/2) is the
// dequantised rank-space average, and o = P_V^T z (the V reconstruction of Lemma lem:head-dist applied after
// the softmax average, which is linear).
//
// The kernel is a chain of latencies, not of bandwidth, so that its loads leave together: a lane takes a
// chunk's (m, l), a thread four coordinates of every (8 / GB)-th chunk of one head (up to eight in flight
// before the weights are known) and four columns of every eighth basis row. With one block per unit that
// merged its chunks serially (a wavefront's chunks one batch after another) the combine took more than the
// partials of a short context: 14.5 us after partials of 6.2 us (8 units x 4k, G = 4), now 5.5; 64 units x 32k
// 11.7 and 5.4, 256 units x 128k 12.2 and 7.4, 640 units, G = 8, 26 and 18.
//
// MANY: more blocks than the chip holds at those registers. The rounds then cost more than the latencies, so the
// basis is read after the merge and fewer chunks are in flight, which leaves room for five or six blocks per
// CU where two or four were: a call of 2048 units x 300 tokens takes 40.9 us with one head (50.8 without it), 43.6
// with two (53.3) and 54.9 with eight (56.8).
constexpr int kCombThreads = 256;
constexpr int kCombRows = kCombThreads / 32;  // rows of 32 threads
// Chunks merged at a time (their weights are in LDS).
__host__ __device__ constexpr int comb_chunks(int gb, bool many) { return many ? 128 : (gb <= 2 ? 512 : 256); }
constexpr int kCombMaxHeads = 8;              // heads per block at most
constexpr int kCombBlocksPerCu = 2;           // blocks at which heads start to share one
// Wavefronts per SIMD, and so blocks per CU, that the registers are cut for.
__host__ __device__ constexpr int comb_waves(int gb, bool many) { return many ? (gb <= 2 ? 6 : 5) : (gb <= 2 ? 2 : 4); }
template <int GB, bool MANY>
__global__ __launch_bounds__(kCombThreads) __attribute__((amdgpu_waves_per_eu(comb_waves(GB, MANY))))
void combine_kernel(DevSide V, int G, int n_chunks, const float* __restrict__ part,
                                                               float* __restrict__ out) {
    static_assert(kCombRows % GB == 0, "a head takes whole rows of threads");
    constexpr int CS = kCombRows / GB, PF = MANY ? 2 : (GB <= 2 ? 8 : 4), RP = kD / kCombRows, NW = kCombThreads / 64;
    constexpr int NB = comb_chunks(GB, MANY), ML = NB / 64;
    // With four or eight heads a thread takes every chunk or every other one: the sum of a pass is formed apart, so
    // that the roundings of the whole sum grow with the passes (in one chain the outputs of 640 units x 64k, G = 8, 16
    // chunks, were 2.4e-6 off fp64; with two chains per unit, before, 2.2e-6).
    constexpr bool kSub = !MANY && GB >= 4;
    __shared__ float wt[GB][NB];                                   // 2^(m_c - M)
    __shared__ float run[3][GB];                                   // M, L, the batch's rescale
    __shared__ __attribute__((aligned(16))) float red[kCombRows][kD];
    __shared__ float zs[GB][kD];
    __shared__ __attribute__((aligned(16))) float os[NW][GB][kD];
    const int u = blockIdx.x, h0 = blockIdx.y * GB, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int q4 = tid & 31, row = tid >> 5, hr = row % GB, cr = row / GB;
    const float* __restrict__ pu = part + ((int64_t)u * n_chunks * G + h0) * kPartStride;
    const int64_t cstride = (int64_t)G * kPartStride;
    const int rv = V.r[u];
    const uint16_t* __restrict__ P4 = V.basis + V.basis_off[u] + 4 * q4;
    uint2 pw[RP];
    float4 A = float4{0.f, 0.f, 0.f, 0.f}, pre[PF];
    // coordinates 4 q4 .. of chunks c0 + cr + k CS of the batch of nb chunks at b0
    auto load_acc = [&](int b0, int nb, int c0) {
        const float* __restrict__ pa = pu + b0 * cstride + hr * kPartStride + 4 + 4 * q4;
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int c = c0 + cr + k * CS;
            if (c < nb) pre[k] = *reinterpret_cast<const float4*>(pa + c * cstride);
        }
    };
    auto load_basis = [&]() {
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            const int i = row + kCombRows * k;
            pw[k] = i < rv ? load_basis4(P4 + i * kD) : uint2{0u, 0u};
        }
    };
    load_acc(0, min(NB, n_chunks), 0);
    if constexpr (!MANY) load_basis();
    for (int b0 = 0; b0 < n_chunks; b0 += NB) {
        const int nb = min(NB, n_chunks - b0);
        const float* __restrict__ pb = pu + b0 * cstride;
        if (b0 > 0) {
            __syncthreads();  // the last batch's weights have been read
            load_acc(b0, nb, 0);
        }
        for (int g = wv; g < GB; g += NW) {
            float2 ml[ML];
            const float Mo = b0 == 0 ? -INFINITY : run[0][g], Lo = b0 == 0 ? 0.f : run[1][g];
            float M = Mo;
#pragma unroll
            for (int k = 0; k < ML; ++k) {
                if (64 * k < nb) {
                    const int c = 64 * k + lane;
                    ml[k] = c < nb ? *reinterpret_cast<const float2*>(pb + c * cstride + g * kPartStride) : float2{-INFINITY, 0.f};
                    if (ml[k].y > 0.f) M = fmaxf(M, ml[k].x);  // an empty chunk has l = 0 and no accumulator
                }
            }
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) M = fmaxf(M, __shfl_xor(M, m));
            float L = 0.f;
#pragma unroll
            for (int k = 0; k < ML; ++k) {
                if (64 * k < nb) {
                    const float w = ml[k].y > 0.f ? exp2f(ml[k].x - M) : 0.f;
                    wt[g][64 * k + lane] = w;
                    if (ml[k].y > 0.f) L = fmaf(ml[k].y, w, L);
                }
            }
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) L += __shfl_xor(L, m);
            const float sc = Mo == -INFINITY ? 0.f : exp2f(Mo - M);
            if (lane == 0) {
                run[0][g] = M;
                run[1][g] = fmaf(Lo, sc, L);
                run[2][g] = sc;
            }
        }
        __syncthreads();
        if (b0 > 0) {
            const float sc = run[2][hr];
            A.x *= sc; A.y *= sc; A.z *= sc; A.w *= sc;
        }
        for (int c0 = 0; c0 < nb; c0 += PF * CS) {
            if (c0 > 0) load_acc(b0, nb, c0);
            float4 p = kSub ? float4{0.f, 0.f, 0.f, 0.f} : A;
#pragma unroll
            for (int k = 0; k < PF; ++k) {
                const int c = c0 + cr + k * CS;
                const float w = c < nb ? wt[hr][c] : 0.f;
                const bool on = w != 0.f;  // an empty chunk's accumulator is not written
                p.x = fmaf(on ? pre[k].x : 0.f, w, p.x);
                p.y = fmaf(on ? pre[k].y : 0.f, w, p.y);
                p.z = fmaf(on ? pre[k].z : 0.f, w, p.z);
                p.w = fmaf(on ? pre[k].w : 0.f, w, p.w);
            }
            if constexpr (kSub) A = float4{A.x + p.x, A.y + p.y, A.z + p.z, A.w + p.w};
            else A = p;
        }
    }
    *reinterpret_cast<float4*>(&red[row][4 * q4]) = A;
    if constexpr (MANY) load_basis();
    __syncthreads();
    const float step = V.delta[u];
    for (int e = tid; e < GB * kD; e += kCombThreads) {
        const int g = e / kD, j = e % kD;
        const float L = run[1][g];
        float a = 0.f;
#pragma unroll
        for (int c = 0; c < CS; ++c) a += red[c * GB + g][j];
        zs[g][j] = (L > 0.f && j < rv) ? step * fmaf(a, 1.f / L, 0.5f) : 0.f;
    }
    __syncthreads();
    // the basis words stay packed until here
#pragma unroll
    for (int k = 0; k < RP; ++k) asm volatile("" : "+v"(pw[k].x), "+v"(pw[k].y));
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        float4 o = float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            const float z = zs[g][row + kCombRows * k];  // zero past the rank
            o.x = fmaf(h2f((uint16_t)(pw[k].x & 0xffffu)), z, o.x);
            o.y = fmaf(h2f((uint16_t)(pw[k].x >> 16)), z, o.y);
            o.z = fmaf(h2f((uint16_t)(pw[k].y & 0xffffu)), z, o.z);
            o.w = fmaf(h2f((uint16_t)(pw[k].y >> 16)), z, o.w);
        }
        o.x += __shfl_xor(o.x, 32);
        o.y += __shfl_xor(o.y, 32);
        o.z += __shfl_xor(o.z, 32);
        o.w += __shfl_xor(o.w, 32);
        if (lane < 32) *reinterpret_cast<float4*>(&os[wv][g][4 * q4]) = o;
    }
    __syncthreads();
    for (int e = tid; e < GB * kD; e += kCombThreads) {
        const int g = e / kD, j = e % kD;
        out[((int64_t)u * G + h0) * kD + e] = (os[0][g][j] + os[1][g][j]) + (os[2][g][j] + os[3][g][j]);
    }
}

// ---------------------------------------------------------------- read probe

// Streaming read of n16 16-byte words (non-temporal loads, grid-stride). The words fold into one
// value per lane, stored to sink only when it equals a constant, so that the loads stay live.
__global__ __launch_bounds__(256) void read_probe_kernel(const v4u* __restrict__ p, size_t n16, uint32_t* __restrict__ sink) {
    uint32_t acc = 0u;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) {
        const v4u v = __builtin_nontemporal_load(p + i);
        acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
    if (acc == 0x9e3779b9u) sink[0] = acc;
}

namespace {


// LDS bytes of the staged tail K-step: the largest over units whose rank has a tail group.
int stage_lds_bytes(const kvc_stream_desc* k) {
    int m = 0;
    for (int u = 0; u < k->n_units; ++u)
        if (k->r_host[u] & 15) m = std::max(m, 512 * k->b_host[u]);
    return m == 0 ? 0 : m + 32;  // funnel reads may look one word past a plane's region
}

// Query heads of one item. Sixteen are two items of eight, which read the codes twice: in one item they take
// one wavefront per SIMD, spill and have no compiled widths (160 units x 16k, 2 bpd: 292 us in one item,
// 84 us in two; 1 bpd 246 and 74, 4 bpd 301 and 130).
int item_heads(int G) { return std::min(G, 8); }

size_t partial_smem(int G, int stage_bytes_) {
    const int LM = (item_heads(G) + 3) / 4;
    return (size_t)16 * LM * kPRowBytes + (size_t)stage_bytes_;
}

template <int G>
int resident_blocks(size_t smem) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, decode_partial_kernel<G>, 64, smem) != hipSuccess || nb <= 0) {
        (void)hipGetLastError();
        nb = 16;
    }
    return nb;
}

// Work items (wavefronts) the device holds at once for this launch.
int64_t resident_slots(int G, size_t smem) {
    const int ncu = device_cus();
    int nb;
    switch (G) {
        case 1: nb = resident_blocks<1>(smem); break;
        case 2: nb = resident_blocks<2>(smem); break;
        case 4: nb = resident_blocks<4>(smem); break;
        default: nb = resident_blocks<8>(smem); break;
    }
    return (int64_t)ncu * nb;
}

// Split of each unit's context into n_chunks equal chunks of whole tiles (at most kMaxChunkTiles
// each). The count minimises
//   rounds x (tiles per item + per-item overhead) + (straggler share) x tiles per item,
// rounds = ceil(items / resident slots): whole rounds with no short remainder, and no more items
// than that (one round of longer items can beat two rounds of items half as long that would fill
// every slot). The two constants are fitted to the partials kernel's times on the 8B-shaped 32k
// workload at 3, 6 and 9 chunks per unit (2, 4 and 6 rounds): about four tiles of work per item,
// and a small straggler share, as the hardware hands each freed slot the next item.
constexpr int kItemOverheadTiles = 4;
constexpr double kStragglerShare = 0.1;

struct WsLayout {
    int chunk, n_chunks, stage_bytes;
    int64_t qa, qk, part, total;  // byte offsets
};

WsLayout ws_layout(const kvc_stream_desc* k, int G, int max_seq) {
    WsLayout L;
    const int U = k->n_units;
    const int LM = (G + 3) / 4;
    L.stage_bytes = stage_lds_bytes(k);
    const int64_t slots = resident_slots(item_heads(G), partial_smem(G, L.stage_bytes));
    const int tpu = (max_seq + kTile - 1) / kTile;
    double best_cost = -1.0;
    L.chunk = std::min(tpu, kMaxChunkTiles) * kTile;
    L.n_chunks = (tpu + kMaxChunkTiles - 1) / kMaxChunkTiles;
    for (int n = 1; n <= tpu && n <= 4096; ++n) {
        const int c = (tpu + n - 1) / n;
        if ((tpu + c - 1) / c != n || c > kMaxChunkTiles) continue;
        const int64_t items = (int64_t)U * (G / item_heads(G)) * n;
        const int64_t rounds = (items + slots - 1) / slots;
        const double cost = (double)rounds * (c + kItemOverheadTiles) + kStragglerShare * c;
        if (best_cost < 0.0 || cost < best_cost) {
            best_cost = cost;
            L.chunk = c * kTile;
            L.n_chunks = n;
        }
    }
    auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
    L.qa = 0;
    L.qk = up(L.qa + (int64_t)U * 2 * LM * 64 * 16);
    L.part = up(L.qk + (int64_t)U * G * 16);
    L.total = L.part + (int64_t)U * L.n_chunks * G * kPartStride * 4;
    return L;
}

int decode_check(const kvc_stream_desc* k, const kvc_stream_desc* v, int32_t G, int32_t max_seq_len) {
    if (int e = validate_desc(k, "kvc_decode_attn(k)")) return e;
    if (int e = validate_desc(v, "kvc_decode_attn(v)")) return e;
    if (k->side != KVC_SIDE_K || v->side != KVC_SIDE_V) return set_error(KVC_EINVAL, "kvc_decode_attn: descriptor sides");
    if (k->n_units != v->n_units) return set_error(KVC_EINVAL, "kvc_decode_attn: K and V unit counts differ");
    if (G != 1 && G != 2 && G != 4 && G != 8 && G != 16)
        return set_error(KVC_EUNSUPPORTED, "kvc_decode_attn: G = %d (1, 2, 4, 8 or 16)", G);
    if (max_seq_len < 1) return set_error(KVC_EINVAL, "kvc_decode_attn: max_seq_len < 1");
    if (max_seq_len > k->capacity || max_seq_len > v->capacity)
        return set_error(KVC_ENOSPACE, "kvc_decode_attn: max_seq_len exceeds capacity");
    // per-unit streams must lie inside their arenas (the kernels bound their loads by the stream)
    const int64_t kct = ((int64_t)k->capacity + kTile - 1) / kTile, vct = ((int64_t)v->capacity + kTile - 1) / kTile;
    for (int u = 0; u < k->n_units; ++u) {
        if (kct * 8 * k->r_host[u] * k->b_host[u] > INT32_MAX || vct * 8 * v->r_host[u] * v->b_host[u] > INT32_MAX)
            return set_error(KVC_EUNSUPPORTED, "kvc_decode_attn: a unit's stream exceeds 2 GiB");
    }
    return KVC_OK;
}

template <int G>
int launch_partials(dim3 grid, int Gq, hipStream_t st, const DevSide& K, const DevSide& V, const v4i* qa, const float4* qk,
                    const int32_t* seq_len, int max_seq, int chunk, int n_chunks, int kct, int vct, float* part,
                    int stage_bytes_) {
    const size_t smem = partial_smem(G, stage_bytes_);
    if (smem > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)decode_partial_kernel<G>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return set_error(KVC_EDEVICE, "hipFuncSetAttribute: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(decode_partial_kernel<G>, grid, dim3(64), smem, st, K, V, Gq, qa, qk, seq_len, max_seq, chunk,
                       n_chunks, kct, vct, part);
    return KVC_OK;
}

}  // namespace
}  // namespace kvc

using namespace kvc;

extern "C" size_t kvc_decode_attn_workspace(const kvc_stream_desc* k, const kvc_stream_desc* v, int32_t G,
                                            int32_t max_seq_len) {
    clear_error();
    if (decode_check(k, v, G, max_seq_len)) return 0;
    return (size_t)ws_layout(k, G, max_seq_len).total;
}

namespace kvc {
namespace {

template <bool MANY>
void launch_combine_g(int gb, dim3 grid, hipStream_t st, const DevSide& V, int G, int n_chunks, const float* part, float* out) {
    const dim3 blk(kCombThreads);
    switch (gb) {
        case 1: hipLaunchKernelGGL((combine_kernel<1, MANY>), grid, blk, 0, st, V, G, n_chunks, part, out); break;
        case 2: hipLaunchKernelGGL((combine_kernel<2, MANY>), grid, blk, 0, st, V, G, n_chunks, part, out); break;
        case 4: hipLaunchKernelGGL((combine_kernel<4, MANY>), grid, blk, 0, st, V, G, n_chunks, part, out); break;
        default: hipLaunchKernelGGL((combine_kernel<8, MANY>), grid, blk, 0, st, V, G, n_chunks, part, out); break;
    }
}

// Combine launch for U units of n_chunks partials each. Heads share a block, and so its basis reads, once one
// head per block makes more blocks than are resident (two per CU at the registers of one or two heads):
// 256 units, G = 4, 12.1 us with a head per block and 7.4 with two. Blocks beyond what is resident even so take
// the variant for many: calls of 300 tokens at 640 units, G = 1, 29.4 us without it and 26.1 with it, at 512 units
// (one round either way) 23.9 and 23.2, at 256 units 15.8 and 16.4.
void launch_combine(int G, int U, const DevSide& V, int n_chunks, const float* part, float* out, hipStream_t st) {
    const int64_t cus = device_cus();
    int gb = 1;
    while (gb < G && gb < kCombMaxHeads && (int64_t)U * G > kCombBlocksPerCu * cus * gb) gb *= 2;
    const dim3 grid(U, G / gb);
    if ((int64_t)U * (G / gb) > comb_waves(gb, false) * cus) launch_combine_g<true>(gb, grid, st, V, G, n_chunks, part, out);
    else launch_combine_g<false>(gb, grid, st, V, G, n_chunks, part, out);
}

// The new token of a fused decode step (none for a plain decode call).
struct StepAppend {
    const uint16_t* xk = nullptr;
    int64_t xk_stride = 0;
    const uint16_t* xv = nullptr;
    int64_t xv_stride = 0;
    int t_new = -1;
};

// Launches of one decode step into the workspace ws (validated by the caller, of layout L); with an
// append, the query projection and the append share the first launch.
int decode_launch(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q, int32_t G,
                  const int32_t* seq_len, int32_t max_seq_len, float* out, void* ws, const WsLayout& L, void* stream,
                  const StepAppend& app = StepAppend()) {
    const int U = k->n_units;
    char* w = reinterpret_cast<char*>(ws);
    v4i* qa = reinterpret_cast<v4i*>(w + L.qa);
    float4* qk = reinterpret_cast<float4*>(w + L.qk);
    float* part = reinterpret_cast<float*>(w + L.part);
    hipStream_t st = (hipStream_t)stream;
    const DevSide K = dev_side(k), V = dev_side(v);
    const int LM = (G + 3) / 4;
    const size_t qsm = (size_t)2 * LM * 64 * 16;
    if (app.t_new >= 0)
        hipLaunchKernelGGL(step_prep_kernel, dim3(U, 3), dim3(kStepPrepThreads), qsm, st, K, V, q, G, LM, qa, qk, app.xk,
                           app.xk_stride, app.xv, app.xv_stride, app.t_new);
    // one wavefront per unit while the units fill the device, eight (one per row block) for a few units
    else if ((int64_t)U * 4 >= (int64_t)device_cus() * 8)
        hipLaunchKernelGGL(qprep_kernel<1>, dim3(U), dim3(64), qsm, st, K, q, G, LM, qa, qk);
    else
        hipLaunchKernelGGL(qprep_kernel<8>, dim3(U), dim3(512), qsm, st, K, q, G, LM, qa, qk);
    const int kct = (k->capacity + kTile - 1) / kTile, vct = (v->capacity + kTile - 1) / kTile;
    const dim3 grid(L.n_chunks, U, G / item_heads(G));
    int e = KVC_OK;
    switch (G) {
        case 1: e = launch_partials<1>(grid, G, st, K, V, qa, qk, seq_len, max_seq_len, L.chunk, L.n_chunks, kct, vct, part, L.stage_bytes); break;
        case 2: e = launch_partials<2>(grid, G, st, K, V, qa, qk, seq_len, max_seq_len, L.chunk, L.n_chunks, kct, vct, part, L.stage_bytes); break;
        case 4: e = launch_partials<4>(grid, G, st, K, V, qa, qk, seq_len, max_seq_len, L.chunk, L.n_chunks, kct, vct, part, L.stage_bytes); break;
        default: e = launch_partials<8>(grid, G, st, K, V, qa, qk, seq_len, max_seq_len, L.chunk, L.n_chunks, kct, vct, part, L.stage_bytes); break;
    }
    if (e) return e;
    launch_combine(G, U, V, L.n_chunks, part, out, st);
    return check_launch("kvc_decode_attn");
}

// Checks shared by both decode entry points (pointers and alignment; the descriptors are checked by
// decode_check).
int decode_args(const char* fn, const uint16_t* q, const int32_t* seq_len, const float* out) {
    if (!q || !seq_len || !out) return set_error(KVC_EINVAL, "%s: null pointer", fn);
    if (reinterpret_cast<uintptr_t>(q) & 15) return set_error(KVC_EINVAL, "%s: q not 16-byte aligned", fn);
    return KVC_OK;
}

// The no-allocation variant's workspace: one file-scope array per device (each GPU holds its own copy
// at its own address, from the library's load until the process ends). Host code never passes the
// array's name to a kernel: its device address comes from hipGetSymbolAddress, taken once per device
// with that device current.
__device__ __align__(256) uint8_t scratch[KVC_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_error(KVC_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return set_error(KVC_EUNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return set_error(KVC_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return KVC_OK;
}

}  // namespace
}  // namespace kvc

extern "C" int kvc_decode_attn(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q, int32_t G,
                               const int32_t* seq_len, int32_t max_seq_len, float* out, void* ws, size_t ws_bytes,
                               void* stream) {
    clear_error();
    if (int e = decode_check(k, v, G, max_seq_len)) return e;
    if (k->n_units == 0) return KVC_OK;
    if (int e = decode_args("kvc_decode_attn", q, seq_len, out)) return e;
    if (!ws) return set_error(KVC_EINVAL, "kvc_decode_attn: null workspace");
    if (reinterpret_cast<uintptr_t>(ws) & 255) return set_error(KVC_EINVAL, "kvc_decode_attn: workspace not 256-byte aligned");
    const WsLayout L = ws_layout(k, G, max_seq_len);
    if ((int64_t)ws_bytes < L.total)
        return set_error(KVC_ENOSPACE, "kvc_decode_attn: workspace %zu < %lld bytes", ws_bytes, (long long)L.total);
    return decode_launch(k, v, q, G, seq_len, max_seq_len, out, ws, L, stream);
}

extern "C" int kvc_decode_step(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* xk,
                               int64_t xk_unit_stride, const uint16_t* xv, int64_t xv_unit_stride, int32_t t_new,
                               const uint16_t* q, int32_t G, const int32_t* seq_len, int32_t max_seq_len, float* out,
                               void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (int e = decode_check(k, v, G, max_seq_len)) return e;
    if (t_new < 0) return set_error(KVC_EINVAL, "kvc_decode_step: negative t_new");
    if ((int64_t)t_new + 1 > k->capacity || (int64_t)t_new + 1 > v->capacity)
        return set_error(KVC_ENOSPACE, "kvc_decode_step: t_new + 1 > capacity");
    if (k->n_units == 0) return KVC_OK;
    for (const auto& xs : {std::make_pair(xk, xk_unit_stride), std::make_pair(xv, xv_unit_stride)})
        if (!xs.first || (reinterpret_cast<uintptr_t>(xs.first) & 15) || (xs.second & 7) || xs.second < (int64_t)kD)
            return set_error(KVC_EINVAL, "kvc_decode_step: xk, xv must be 16-byte aligned with stride a multiple of 8 and >= d");
    if (int e = decode_args("kvc_decode_step", q, seq_len, out)) return e;
    if (!ws) return set_error(KVC_EINVAL, "kvc_decode_step: null workspace");
    if (reinterpret_cast<uintptr_t>(ws) & 255) return set_error(KVC_EINVAL, "kvc_decode_step: workspace not 256-byte aligned");
    const WsLayout L = ws_layout(k, G, max_seq_len);
    if ((int64_t)ws_bytes < L.total)
        return set_error(KVC_ENOSPACE, "kvc_decode_step: workspace %zu < %lld bytes", ws_bytes, (long long)L.total);
    StepAppend app;
    app.xk = xk;
    app.xk_stride = xk_unit_stride;
    app.xv = xv;
    app.xv_stride = xv_unit_stride;
    app.t_new = t_new;
    return decode_launch(k, v, q, G, seq_len, max_seq_len, out, ws, L, stream, app);
}

extern "C" int kvc_decode_attn_rope(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q, int32_t G,
                                    const int32_t* seq_len, int32_t max_seq_len, float rope_base, float* out,
                                    void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (int e = decode_check(k, v, G, max_seq_len)) return e;
    if (!(rope_base > 1.f) || !std::isfinite(rope_base))
        return set_error(KVC_EINVAL, "kvc_decode_attn_rope: rope_base must be finite and > 1");
    if (k->n_units == 0) return KVC_OK;
    if (int e = decode_args("kvc_decode_attn_rope", q, seq_len, out)) return e;
    if (!ws) return set_error(KVC_EINVAL, "kvc_decode_attn_rope: null workspace");
    if (reinterpret_cast<uintptr_t>(ws) & 255) return set_error(KVC_EINVAL, "kvc_decode_attn_rope: workspace not 256-byte aligned");
    const WsLayout L = ws_layout(k, G, max_seq_len);
    if ((int64_t)ws_bytes < L.total)
        return set_error(KVC_ENOSPACE, "kvc_decode_attn_rope: workspace %zu < %lld bytes", ws_bytes, (long long)L.total);
    float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + L.part);
    int n_chunks = L.n_chunks;  // the workspace holds at most that many partials per unit
    if (int e = launch_rope_partials(k, v, q, G, seq_len, max_seq_len, std::log2((double)rope_base), L.stage_bytes, part, &n_chunks,
                                     (hipStream_t)stream))
        return e;
    launch_combine(G, k->n_units, dev_side(v), n_chunks, part, out, (hipStream_t)stream);
    return check_launch("kvc_decode_attn_rope");
}

extern "C" int kvc_decode_attn_noalloc(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* q,
                                       int32_t G, const int32_t* seq_len, int32_t max_seq_len, float* out,
                                       void* stream) {
    clear_error();
    if (int e = decode_check(k, v, G, max_seq_len)) return e;
    if (k->n_units == 0) return KVC_OK;
    if (int e = decode_args("kvc_decode_attn_noalloc", q, seq_len, out)) return e;
    const WsLayout L = ws_layout(k, G, max_seq_len);
    if (L.total > (int64_t)KVC_NOALLOC_SCRATCH_BYTES)
        return set_error(KVC_ENOSPACE, "kvc_decode_attn_noalloc: needs %lld bytes of workspace, the scratch holds %lld",
                         (long long)L.total, (long long)KVC_NOALLOC_SCRATCH_BYTES);
    void* ws = nullptr;
    if (int e = scratch_of_current_device(&ws)) return e;
    return decode_launch(k, v, q, G, seq_len, max_seq_len, out, ws, L, stream);
}

extern "C" int kvc_read_probe(const void* buf, size_t bytes, uint32_t* sink, void* stream) {
    clear_error();
    if (!buf || !sink || (reinterpret_cast<uintptr_t>(buf) & 15) || (bytes & 15) || (reinterpret_cast<uintptr_t>(sink) & 3))
        return set_error(KVC_EINVAL, "kvc_read_probe: buf and bytes must be multiples of 16 bytes, sink a 4-byte aligned word");
    if (bytes == 0) return KVC_OK;
    const size_t n16 = bytes / 16;
    const size_t blocks = std::min<size_t>((n16 + 255) / 256, (size_t)64 * device_cus());
    hipLaunchKernelGGL(read_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<const v4u*>(buf), n16, sink);
    return check_launch("kvc_read_probe");
}
#else
}  // namespace kvc
#endif  // KVC_DECODE_PARTIALS_UNIT
