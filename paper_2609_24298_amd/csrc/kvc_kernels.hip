// Device half of libkvc, compression side: HIP kernels for CDNA4 (gfx950) and
// their C-ABI launchers (kvc_encode, kvc_encode_kv). Decode attention lives in
// kvc_decode.hip, reconstruction in kvc_recon.hip.
//
// Kernels
//  encode_mfma_kernel   bulk encode: per (unit, run of 64-token tiles), the
//                       projection on fp16 matrix cores with fp32 accumulation,
//                       codes decided against a rigorous error bound (undecided
//                       elements settled in fp64, then exactly in 128-bit
//                       integers), bit-packed from LDS group by group.
//  append_kernel        1-4 new tokens per unit (a decode step's append): basis
//                       rows read coalesced, the same bounded decision (undecided
//                       elements settled by their wavefront), and the new fields
//                       written in place (whole words where a token owns them).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <utility>

#include "kvc_append.h"
#include "kvc_device.h"
#include "kvc_internal.h"

namespace kvc {

constexpr int kD = KVC_HEAD_DIM;
constexpr int kTile = KVC_TILE_TOKENS;

// ---------------------------------------------------------------- encode

// ---------------------------------------------------------------- bulk encode on matrix cores

// Bulk encode (any token count above the append path's): one 256-thread block per (unit, run of
// tiles, side); each wavefront encodes whole 64-token tiles, 16 coordinates (a group) at a time.
//
// Projection. y = P x on v_mfma_f32_16x16x32_f16 (exact fp16 products, fp32 accumulation), the basis in
// LDS and the tile's tokens as operand fragments in registers. The four k-steps of an element have an
// accumulator each, added in pairs at the end: a k-step is 32 terms, at worst a truncating addition
// (2^-23) each, and the three rounded additions move the sum by at most 2^-23 of the magnitudes, so
// |y_mma - y| <= 33 2^-23 ||P_i|| ||x||. One chained accumulator (128 terms) has four times the bound and
// so four times the undecided elements, whose settlement was a fifth of the kernel's time.
//
// Decision. Codes are decided in fp32 where y is farther than that bound (plus the rounding of y / step)
// from every threshold; the rare undecided elements are re-evaluated by the whole wavefront in fp64 (exact
// products, a 2^-45 ||P_i|| ||x|| sum bound) and, if still undecided, exactly in 128-bit integers. The
// bound uses the unit's largest row norm and, on the V side, the largest norm of the lane's four tokens
// of a quarter, so that one threshold serves four elements.
//
// Packing. A lane decides four codes (one byte each) of each quarter nt; a 4 x 4 transpose over (nt, lane
// row) with four register swaps leaves every lane with the 16 codes of one field: K, token `lane` of the
// coordinate group; V, quarter lane / 16 of coordinate lane % 16. A K field goes straight to its place
// (2p bytes per plane, consecutive lanes consecutive fields); V fields of a value group gather in
// registers and go out as one 16-byte row per lane and plane. Only the K tail group (r % 16) and a
// V group shorter than 16 bytes a lane pass through LDS. A partial tile masks whole fields (K: a token
// owns its bytes) or merges them once per row (V).
//
// Measured: 256 units x 8192 tokens, both sides, 2 bpd: 356 us (3.4 TB/s; 532 us with one chained
// accumulator, codes packed through LDS and a launch per side); 64 units x 1000 tokens from inside a tile:
// 27 us (177 us with 32 tiles per block and partial tiles rewritten byte by byte). Without any settlement
// (codes no longer guaranteed) the former takes 314 us; three wavefronts per SIMD spill and take longer.
constexpr int kEncMmaThreads = 256;
constexpr int kEncWaves = kEncMmaThreads / 64;
constexpr int kPRow = kD + 8;  // LDS row stride of the staged basis, in halves
constexpr int kEncStage = 1024;  // LDS bytes per wavefront: the K tail group's codes, or a short V group

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f4 mfma_f16(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Four slots (one code per byte of v, already masked to P bits) packed into 4 P consecutive bits.
template <int P>
__device__ __forceinline__ uint32_t compact4(uint32_t v) {
    if constexpr (P == 4) {
        v = (v | (v >> 4)) & 0x00ff00ffu;
        return (v | (v >> 8)) & 0xffffu;
    } else if constexpr (P == 2) {
        return __builtin_amdgcn_udot4(v, 0x40100401u, 0u, false);
    } else if constexpr (P == 1) {
        return __builtin_amdgcn_udot4(v, 0x08040201u, 0u, false);
    } else {
        return v;
    }
}

// Plane K (width P) of the 16 codes c (one byte each, in field order): w[0 .. P / 2) (P = 1: 16 bits).
template <int B, int K>
__device__ __forceinline__ void field_bits(const uint32_t (&c)[4], uint32_t (&w)[4]) {
    constexpr int P = plane_w(B, K), SH = plane_sh(B, K);
    constexpr uint32_t PM = (P == 8 ? 0xffu : ((1u << P) - 1u)) * 0x01010101u;
    uint32_t v[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) v[m] = compact4<P>(n_planes(B) == 1 ? c[m] : (c[m] >> SH) & PM);
    if constexpr (P == 8) {
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
    } else if constexpr (P == 4) {
        w[0] = v[0] | (v[1] << 16);
        w[1] = v[2] | (v[3] << 16);
    } else if constexpr (P == 2) {
        w[0] = v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24);
    } else {
        w[0] = v[0] | (v[1] << 4) | (v[2] << 8) | (v[3] << 12);
    }
}

// Stores the 2P bytes of a field.
template <int P>
__device__ __forceinline__ void store_field(uint8_t* __restrict__ dst, const uint32_t (&w)[4]) {
    if constexpr (P == 1) *reinterpret_cast<uint16_t*>(dst) = (uint16_t)w[0];
    else if constexpr (P == 2) *reinterpret_cast<uint32_t*>(dst) = w[0];
    else if constexpr (P == 4) *reinterpret_cast<uint2*>(dst) = uint2{w[0], w[1]};
    else *reinterpret_cast<uint4*>(dst) = uint4{w[0], w[1], w[2], w[3]};
}

// Transpose over (register, row of 16 lanes): lane row g of the result's register k is row k of
// register g.
__device__ __forceinline__ void transpose_rows(uint32_t (&c)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(c[0], c[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(c[1], c[3], false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    c[0] = lo[0];
    c[1] = lo[1];
    c[2] = hi[0];
    c[3] = hi[1];
}

// The wavefront's LDS accesses execute in program order: between a write and a read of the same
// bytes by other lanes only the compiler's reordering has to be stopped.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// K: a full group's field of token `lane`, if it is encoded (a token owns the bytes of its fields).
template <int B, int K>
__device__ __forceinline__ void pack_k_field(const uint32_t (&c)[4], uint8_t* __restrict__ tbase, int r, int mc, bool mine, int lane) {
    if constexpr (K < n_planes(B)) {
        constexpr int P = plane_w(B, K);
        uint32_t w[4];
        field_bits<B, K>(c, w);
        if (mine) store_field<P>(tbase + 8 * r * plane_off(B, K) + P * (128 * mc + 2 * lane), w);
    }
}

// K tail group: 64 rho codes in sb in slot order (token-major), of which [s0, s1) are encoded. Word w
// of the group's part of a plane holds slots [w 32 / P, (w + 1) 32 / P); a word that also holds other
// tokens' slots keeps their bits.
template <int B, int K>
__device__ __forceinline__ void pack_k_tail(const uint8_t* __restrict__ sb, uint8_t* __restrict__ tbase, int r, int mc, int n_sl,
                                            int s0, int s1, int lane) {
    if constexpr (K < n_planes(B)) {
        constexpr int P = plane_w(B, K), SH = plane_sh(B, K), PPW = 32 / P;
        constexpr uint32_t PM = (P == 8 ? 0xffu : ((1u << P) - 1u)) * 0x01010101u;
        uint32_t* __restrict__ pw = reinterpret_cast<uint32_t*>(tbase + 8 * r * plane_off(B, K)) + 1024 / PPW * mc;
        for (int wi = lane; wi < n_sl / PPW; wi += 64) {
            uint32_t word = 0;
#pragma unroll
            for (int m = 0; m < PPW / 4; ++m)
                word |= compact4<P>((*reinterpret_cast<const uint32_t*>(sb + wi * PPW + 4 * m) >> SH) & PM) << (P == 8 ? 0 : 4 * P * m);
            const int a = min(max(s0 - wi * PPW, 0), PPW), e = min(max(s1 - wi * PPW, 0), PPW);  // encoded slots of the word
            if (a == 0 && e == PPW) {
                pw[wi] = word;
            } else if (a < e) {
                const uint32_t msk = (uint32_t)(((1ull << (P * e)) - 1ull) & ~((1ull << (P * a)) - 1ull));
                pw[wi] = (pw[wi] & ~msk) | (word & msk);
            }
        }
    }
}

// V: the lane's fields of a value group gather in vg (16 bytes, the newest field at the top); once the
// group is complete they are stored at L = 4 c + q of the group. m: N-tiles of the group so far; km:
// the field's bits that are encoded (all of them on a full tile).
template <int B, int K, bool FULL>
__device__ __forceinline__ void pack_v_field(const uint32_t (&c)[4], const uint32_t (&cm)[4], uint32_t (&vg)[3][4],
                                             uint8_t* __restrict__ vst, uint8_t* __restrict__ tbase, int r, int n, int n_last, int lane) {
    if constexpr (K < n_planes(B)) {
        constexpr int P = plane_w(B, K), G = v_group_ntiles(P);
        const int col = lane & 15, grp = lane >> 4;
        uint32_t w[4], km[4];
        field_bits<B, K>(c, w);
        if constexpr (!FULL) field_bits<B, K>(cm, km);
        uint32_t (&g)[4] = vg[K];
        if constexpr (P == 8) {
            g[0] = w[0]; g[1] = w[1]; g[2] = w[2]; g[3] = w[3];
        } else if constexpr (P == 4) {
            g[0] = g[2]; g[1] = g[3]; g[2] = w[0]; g[3] = w[1];
        } else if constexpr (P == 2) {
            g[0] = g[1]; g[1] = g[2]; g[2] = g[3]; g[3] = w[0];
        } else {
            g[0] = __builtin_amdgcn_alignbit(g[1], g[0], 16);
            g[1] = __builtin_amdgcn_alignbit(g[2], g[1], 16);
            g[2] = __builtin_amdgcn_alignbit(g[3], g[2], 16);
            g[3] = __builtin_amdgcn_alignbit(w[0], g[3], 16);
        }
        const int Q = n / G, m = n - G * Q + 1;
        if (m != G && n != n_last) return;
        uint8_t* __restrict__ pbase = tbase + 8 * r * plane_off(B, K) + 1024 * Q;
        if (m == G && 16 * (n + 1) <= r) {  // 16 bytes a lane
            uint4* dst = reinterpret_cast<uint4*>(pbase + 16 * (4 * col + grp));
            uint4 v = uint4{g[0], g[1], g[2], g[3]};
            if constexpr (!FULL) {
                // the field mask is the same for every N-tile of the group
                uint4 o = *dst, k;
                if constexpr (P == 8) k = uint4{km[0], km[1], km[2], km[3]};
                else if constexpr (P == 4) k = uint4{km[0], km[1], km[0], km[1]};
                else if constexpr (P == 2) k = uint4{km[0], km[0], km[0], km[0]};
                else { const uint32_t d = km[0] | (km[0] << 16); k = uint4{d, d, d, d}; }
                v = uint4{(o.x & ~k.x) | (v.x & k.x), (o.y & ~k.y) | (v.y & k.y), (o.z & ~k.z) | (v.z & k.z), (o.w & ~k.w) | (v.w & k.w)};
            }
            *dst = v;
            return;
        }
        // a short last group: m fields a lane (one fewer past the last coordinate), 2P bytes each, through LDS
        const int gbytes = 8 * P * (r - 16 * G * Q);  // a multiple of 16 (r even)
        if constexpr (!FULL) {
            if (16 * lane < gbytes) *reinterpret_cast<uint4*>(vst + 16 * lane) = *reinterpret_cast<const uint4*>(pbase + 16 * lane);
        }
        wave_lds_sync();
        const int ct = r - 16 * n, A = col >= ct ? 4 * (col - ct) + grp : 0, cnt = col >= ct ? m - 1 : m;
        uint8_t* run = vst + 2 * P * (m * (4 * col + grp) - A);
#pragma unroll
        for (int j = 0; j < G; ++j) {  // field j of the group sits j - m + G fields up in g
            if (j < cnt) {
                uint32_t f[4] = {0u, 0u, 0u, 0u};
                const int at = j - m + G;
                if constexpr (P == 1) {
                    const uint32_t d = at < 2 ? g[0] : (at < 4 ? g[1] : (at < 6 ? g[2] : g[3]));
                    f[0] = (at & 1) ? d >> 16 : d & 0xffffu;
                } else if constexpr (P == 2) {
                    f[0] = at == 0 ? g[0] : (at == 1 ? g[1] : (at == 2 ? g[2] : g[3]));
                } else if constexpr (P == 4) {
                    f[0] = at == 0 ? g[0] : g[2];
                    f[1] = at == 0 ? g[1] : g[3];
                } else {
                    f[0] = g[0]; f[1] = g[1]; f[2] = g[2]; f[3] = g[3];
                }
                if constexpr (!FULL) {
                    if constexpr (P == 1) {
                        const uint32_t o = *reinterpret_cast<const uint16_t*>(run + 2 * P * j);
                        f[0] = (o & ~km[0]) | (f[0] & km[0]);
                    } else {
#pragma unroll
                        for (int d = 0; d < P / 2; ++d) {
                            const uint32_t o = reinterpret_cast<const uint32_t*>(run + 2 * P * j)[d];
                            f[d] = (o & ~km[d]) | (f[d] & km[d]);
                        }
                    }
                }
                store_field<P>(run + 2 * P * j, f);
            }
        }
        wave_lds_sync();
        if (16 * lane < gbytes) *reinterpret_cast<uint4*>(pbase + 16 * lane) = *reinterpret_cast<const uint4*>(vst + 16 * lane);
        wave_lds_sync();
    }
}

// The tiles of one wavefront: tl = tl0, tl0 + kEncWaves, ... below tl_end (indices into the call's tiles).
template <int side, int B>
__device__ __forceinline__ void encode_tiles(const uint16_t* __restrict__ Pl, const float* __restrict__ pnrm, float tol,
                                             float* __restrict__ etok, uint8_t* __restrict__ sb, const uint16_t* __restrict__ Pg,
                                             uint8_t* __restrict__ stream, const uint16_t* __restrict__ xu, int r, float step,
                                             int t0, int n_tok, int tile_first, int tl0, int tl_end, int lane) {
    const int col = lane & 15, grp = lane >> 4;
    constexpr int h = 1 << (B - 1);
    constexpr float fmax_code = (float)(2 * h - 1), fh_lo = (float)h - 0.5f;  // t' = t - 1/2
    constexpr float half_amb = 0.5f - (float)(3 * h + 4) * 0x1p-22f;         // 1/2 - c_amb (exact in fp32)
    const float inv = 1.f / step;
    const double inv64 = 1.0 / (double)step;
    const int g16 = r >> 4, rho = r & 15, n_mc = (r + 15) >> 4;

    // Token fragments: operand row 16 nt + col, dims 32 ks + 8 grp + [0, 8). The row holds token
    // 16 nt + col for K; for V, token 16 nt + kidx_b(col), the token whose slot in the quarter is
    // position col (pos_b o kidx_b = identity), so that a lane's four results (rows 4 grp + i) are
    // four consecutive positions of a field. Tokens outside the range read a valid token and never reach
    // the stream. The fragments of a wavefront's next tile are loaded as soon as the last products of the
    // current one have read them, so that the loads overlap the tile's last decisions and packing.
    const int trow = side == KVC_SIDE_K ? col : kidx_b(B, col);
    h8 xf[4][4];
    auto load_x = [&](int tl) {
        const int tok0n = (tile_first + tl) * kTile;
        const int lon = max(t0, tok0n), hin = min(t0 + n_tok, tok0n + kTile);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int tk = tok0n + 16 * nt + trow;
            const h8* row = reinterpret_cast<const h8*>(xu + (int64_t)((tk >= lon && tk < hin ? tk : lon) - t0) * kD);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) xf[nt][ks] = row[4 * ks + grp];
        }
    };
    if (tl0 < tl_end) load_x(tl0);

#pragma unroll 1
    for (int tl = tl0; tl < tl_end; tl += kEncWaves) {
        const int tile = tile_first + tl, tok0 = tile * kTile;
        const int lo = max(t0, tok0), hi = min(t0 + n_tok, tok0 + kTile);
        const bool full = lo == tok0 && hi == tok0 + kTile;
        uint8_t* __restrict__ tbase = stream + (int64_t)tile * 8 * r * B;

        // thr[nt]: an element of quarter nt is undecided where |t' - rint(t')| >= thr. etok is indexed by
        // operand row; a token outside the range has norm 0 there (its elements are dropped below).
        float thr[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int tk = tok0 + 16 * nt + trow;
            float s2 = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const h2 v = {xf[nt][ks][2 * e], xf[nt][ks][2 * e + 1]};
                    s2 = __builtin_amdgcn_fdot2(v, v, s2, false);
                }
            }
            s2 += __shfl_xor(s2, 16);
            s2 += __shfl_xor(s2, 32);
            thr[nt] = tk >= lo && tk < hi ? sqrtf(s2) : 0.f;
            if (grp == 0) etok[16 * nt + col] = thr[nt];
        }
        wave_lds_sync();
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            if constexpr (side == KVC_SIDE_V) {
                const f4 e = *reinterpret_cast<const f4*>(etok + 16 * nt + 4 * grp);
                thr[nt] = fmaxf(fmaxf(e[0], e[1]), fmaxf(e[2], e[3]));
            }
            thr[nt] = fmaf(-thr[nt], tol, half_amb);
        }
        uint32_t vg[3][4], cm[4];  // V: value groups being gathered; all-ones codes at the field positions that are encoded
        if constexpr (side == KVC_SIDE_V) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int d = 0; d < 4; ++d) vg[k][d] = 0u;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                cm[d] = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int tk = tok0 + 16 * grp + kidx_b(B, 4 * d + i);
                    if (tk >= lo && tk < hi) cm[d] |= (uint32_t)(2 * h - 1) << (8 * i);
                }
            }
        }
#pragma unroll 1
        for (int mc = 0; mc < n_mc; ++mc) {
            h8 pf[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                pf[ks] = *reinterpret_cast<const h8*>(Pl + (16 * mc + col) * kPRow + 32 * ks + 8 * grp);
            f4 acc[4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                f4 p[4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    p[ks] = side == KVC_SIDE_K ? mfma_f16(pf[ks], xf[nt][ks], f4{0.f, 0.f, 0.f, 0.f})
                                               : mfma_f16(xf[nt][ks], pf[ks], f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[nt][i] = (p[0][i] + p[1][i]) + (p[2][i] + p[3][i]);
            }
            if (mc == n_mc - 1 && tl + kEncWaves < tl_end) load_x(tl + kEncWaves);
            // K: lane holds coordinates 16 mc + 4 grp + i of token 16 nt + col.
            // V: lane holds rows 16 nt + 4 grp + i of coordinate 16 mc + col.
            if (mc == g16) {  // coordinates past the rank: the value farthest from a threshold
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if ((side == KVC_SIDE_K ? 4 * grp + i : col) >= rho) acc[nt][i] = 0.5f * step;
            }
            // t = y / step + 2^(b-1): its floor, clamped, is the code. With t' = t - 1/2 (one fused
            // multiply-add) the floor is rint(t') wherever t is not within the error bound eps of an
            // integer, i.e. wherever |t' - rint(t')| < 1/2 - eps; the other elements are undecided.
            // eps = (the basis-product bound) / step + c_amb, c_amb covering the rounding of 1 / step and
            // of the multiply-add, (|t| + 2^(b-1) + 1) 2^-22, for every |t| <= 2^b + 1 (beyond, the
            // code is clamped to 0 or 2^b - 1 whatever the error).
            bool any_amb = false;
            uint32_t cw[4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                uint32_t w = 0;
                float dmax = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float tp = fmaf(acc[nt][i], inv, fh_lo);
                    const float m = __builtin_rintf(tp);
                    dmax = fmaxf(dmax, fabsf(tp - m));
                    w = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(m, 0.f, fmax_code), i, w);
                }
                any_amb |= dmax >= thr[nt];
                cw[nt] = w;
            }
            // undecided elements (rare): flag them per lane, then the whole wavefront settles them one by one
            if (__any(any_amb)) {
                uint32_t ambm = 0;
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float tp = fmaf(acc[nt][i], inv, fh_lo);
                        if (fabsf(tp - __builtin_rintf(tp)) >= thr[nt]) ambm |= 1u << (4 * nt + i);
                    }
                // a token long enough makes thr negative and flags even the coordinates past the rank
                if (mc == g16) ambm &= encode_rank_mask(side, r - 16 * mc, col, grp);
                uint64_t pend = __ballot(ambm != 0);
                while (pend) {
                    const int L = __builtin_ctzll(pend);
                    pend &= pend - 1;
                    uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)ambm, L);
                    const int Lcol = L & 15, Lgrp = L >> 4;
                    while (m) {
                        const int bit = __builtin_ctz(m);
                        m &= m - 1;
                        const int nt = bit >> 2, i = bit & 3;
                        int tkn, c, row;  // token, coordinate, operand row of the element
                        if constexpr (side == KVC_SIDE_K) {
                            tkn = row = 16 * nt + Lcol;
                            c = 16 * mc + 4 * Lgrp + i;
                        } else {
                            row = 16 * nt + 4 * Lgrp + i;
                            tkn = 16 * nt + kidx_b(B, 4 * Lgrp + i);
                            c = 16 * mc + Lcol;
                        }
                        if (tok0 + tkn < lo || tok0 + tkn >= hi) continue;
                        const uint16_t* xrow = xu + (int64_t)(tok0 + tkn - t0) * kD;
                        // The token's entries: from its four lanes' fragments by way of LDS, or, once the
                        // fragments hold the next tile, from memory (a load that nothing else would hide).
                        uint32_t xw;
                        if (mc < n_mc - 1) {
                            uint8_t* dst = sb + 16 * grp;
                            if (col == (row & 15)) {
#pragma unroll
                                for (int n = 0; n < 4; ++n)
                                    if (n == nt)
#pragma unroll
                                        for (int ks = 0; ks < 4; ++ks) *reinterpret_cast<h8*>(dst + 64 * ks) = xf[n][ks];
                            }
                            wave_lds_sync();
                            xw = reinterpret_cast<const uint32_t*>(sb)[lane];
                            wave_lds_sync();
                        } else {
                            xw = *reinterpret_cast<const uint32_t*>(xrow + 2 * lane);
                        }
                        const uint32_t code = resolve_code_wave(Pl + c * kPRow, Pg + (int64_t)c * kD, xw, xrow, step, inv64, B,
                                                                pnrm[c], etok[row], lane);
#pragma unroll
                        for (int n = 0; n < 4; ++n)
                            if (n == nt && lane == L) cw[n] = (cw[n] & ~(0xffu << (8 * i))) | (code << (8 * i));
                    }
                }
            }
            transpose_rows(cw);  // K: the 16 codes of token `lane`; V: of quarter grp of coordinate 16 mc + col
            if constexpr (side == KVC_SIDE_K) {
                const bool mine = tok0 + lane >= lo && tok0 + lane < hi;
                if (mc < g16) {
                    pack_k_field<B, 0>(cw, tbase, r, mc, mine, lane);
                    pack_k_field<B, 1>(cw, tbase, r, mc, mine, lane);
                    pack_k_field<B, 2>(cw, tbase, r, mc, mine, lane);
                } else {
#pragma unroll
                    for (int j = 0; j < 7; ++j)
                        if (2 * j < rho)
                            *reinterpret_cast<uint16_t*>(sb + lane * rho + 2 * j) = (uint16_t)(cw[j >> 1] >> (16 * (j & 1)));
                    wave_lds_sync();
                    const int s0 = (lo - tok0) * rho, s1 = (hi - tok0) * rho;
                    pack_k_tail<B, 0>(sb, tbase, r, mc, 64 * rho, s0, s1, lane);
                    pack_k_tail<B, 1>(sb, tbase, r, mc, 64 * rho, s0, s1, lane);
                    pack_k_tail<B, 2>(sb, tbase, r, mc, 64 * rho, s0, s1, lane);
                    wave_lds_sync();
                }
            } else if (full) {
                pack_v_field<B, 0, true>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
                pack_v_field<B, 1, true>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
                pack_v_field<B, 2, true>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
            } else {
                pack_v_field<B, 0, false>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
                pack_v_field<B, 1, false>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
                pack_v_field<B, 2, false>(cw, cm, vg, sb, tbase, r, mc, n_mc - 1, lane);
            }
        }
    }
}

// Block (run of tiles, unit, side): side0 + blockIdx.z (both sides of a kvc_encode_kv in one launch).
__global__ __launch_bounds__(kEncMmaThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void encode_mfma_kernel(
    DevSide ks, DevSide vs, const uint16_t* __restrict__ xk, int64_t xk_stride, const uint16_t* __restrict__ xv,
    int64_t xv_stride, int side0, int t0, int n_tok, int tile_first, int n_tiles, int tpb) {
    extern __shared__ uint8_t esm[];
    uint16_t* Pl = reinterpret_cast<uint16_t*>(esm);          // [128][kPRow] fp16 basis, rows >= r zero
    float* pnrm = reinterpret_cast<float*>(Pl + kD * kPRow);  // [128] ||P_i||
    float* etoks = pnrm + kD;                                 // [waves][64] token norms
    uint8_t* stages = reinterpret_cast<uint8_t*>(etoks + kEncWaves * kTile);  // [waves][kEncStage]
    const int side = side0 + blockIdx.z;
    const DevSide& s = side == KVC_SIDE_K ? ks : vs;
    const int u = blockIdx.y, tid = threadIdx.x;
    const int r = s.r[u], b = s.b[u];
    const float step = s.delta[u];
    const uint16_t* __restrict__ Pg = s.basis + s.basis_off[u];
#pragma unroll
    for (int j = 0; j < kD * (kD / 8) / kEncMmaThreads; ++j) {
        const int q = tid + kEncMmaThreads * j, row = q >> 4, c8 = q & 15;
        uint4 v = {0u, 0u, 0u, 0u};
        if (row < r) v = reinterpret_cast<const uint4*>(Pg + (int64_t)row * kD)[c8];
        *reinterpret_cast<uint4*>(Pl + row * kPRow + 8 * c8) = v;
        const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
        float s2 = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const h2 p = __builtin_bit_cast(h2, w4[e]);
            s2 = __builtin_amdgcn_fdot2(p, p, s2, false);
        }
        s2 = row_sum16(s2);  // the row's 16 lanes
        if (c8 == 0) pnrm[row] = sqrtf(s2);
    }
    __syncthreads();
    const int wv = tid >> 6, lane = tid & 63;
    float pmax = fmaxf(pnrm[lane], pnrm[lane + 64]);
    for (int o = 32; o > 0; o >>= 1) pmax = fmaxf(pmax, __shfl_xor(pmax, o));
    const float tol = 33.f * 0x1p-23f * 1.01f * pmax / step;
    const int64_t xs = side == KVC_SIDE_K ? xk_stride : xv_stride;
    const uint16_t* __restrict__ xu = (side == KVC_SIDE_K ? xk : xv) + (int64_t)u * xs;
    const int tl0 = blockIdx.x * tpb + wv, tl_end = min((int)(blockIdx.x + 1) * tpb, n_tiles);
    uint8_t* __restrict__ stream = s.codes + s.code_off[u];
    if (side == KVC_SIDE_K) {
        KVC_SWITCH_B(b, (encode_tiles<KVC_SIDE_K, B_>(Pl, pnrm, tol, etoks + wv * kTile, stages + wv * kEncStage, Pg, stream, xu, r,
                                                      step, t0, n_tok, tile_first, tl0, tl_end, lane)));
    } else {
        KVC_SWITCH_B(b, (encode_tiles<KVC_SIDE_V, B_>(Pl, pnrm, tol, etoks + wv * kTile, stages + wv * kEncStage, Pg, stream, xu, r,
                                                      step, t0, n_tok, tile_first, tl0, tl_end, lane)));
    }
}

// ---------------------------------------------------------------- append

// One side: one block per unit.
__global__ __launch_bounds__(kAppThreads) void append_kernel(DevSide s, int side, const uint16_t* __restrict__ x,
                                                             int64_t x_stride, int t0, int n_tok) {
    append_unit(s, side, x, x_stride, t0, n_tok, blockIdx.x);
}

// Both sides in one launch: block (u, 0) appends unit u's keys, block (u, 1) its values.
__global__ __launch_bounds__(kAppThreads) void append_kv_kernel(DevSide k, DevSide v, const uint16_t* __restrict__ xk,
                                                                int64_t xk_stride, const uint16_t* __restrict__ xv,
                                                                int64_t xv_stride, int t0, int n_tok) {
    if (blockIdx.y == 0) append_unit(k, KVC_SIDE_K, xk, xk_stride, t0, n_tok, blockIdx.x);
    else append_unit(v, KVC_SIDE_V, xv, xv_stride, t0, n_tok, blockIdx.x);
}

// ---------------------------------------------------------------- host side

namespace {

// Launch of the bulk encoder for `sides` sides of n_units units (side0 the first).
int launch_encode(const DevSide& k, const DevSide& v, const uint16_t* xk, int64_t xk_stride, const uint16_t* xv, int64_t xv_stride,
                  int side0, int sides, int n_units, int t0, int n_tok, void* stream) {
    const int tile_first = t0 / kTile;
    const int n_tiles = (t0 + n_tok - 1) / kTile - tile_first + 1;
    // Tiles per block (whole turns of its wavefronts): the count that minimises rounds of resident blocks
    // (two per CU) x (turns + staging of the basis, about one turn), so that a short run spreads over the
    // chip and a long one stages its basis seldom.
    const int64_t slots = 2ll * device_cus();
    int tpb = kEncWaves;
    int64_t best = -1;
    for (int turns = 1; turns <= 16; ++turns) {
        const int64_t blocks = (int64_t)n_units * sides * ((n_tiles + turns * kEncWaves - 1) / (turns * kEncWaves));
        const int64_t cost = (blocks + slots - 1) / slots * (turns + 1);
        if (best < 0 || cost < best) { best = cost; tpb = turns * kEncWaves; }
    }
    const size_t smem = (size_t)kD * kPRow * 2 + kD * 4 + kEncWaves * (kTile * 4 + kEncStage);
    const dim3 grid((n_tiles + tpb - 1) / tpb, n_units, sides);
    hipLaunchKernelGGL(encode_mfma_kernel, grid, dim3(kEncMmaThreads), smem, (hipStream_t)stream, k, v, xk, xk_stride, xv, xv_stride,
                       side0, t0, n_tok, tile_first, n_tiles, tpb);
    return check_launch("kvc_encode");
}

}  // namespace
}  // namespace kvc

using namespace kvc;

extern "C" int kvc_encode(const kvc_stream_desc* s, const uint16_t* x, int64_t x_unit_stride, int32_t t0, int32_t n_tok,
                          void* stream) {
    clear_error();
    if (int e = validate_desc(s, "kvc_encode")) return e;
    if (t0 < 0 || n_tok < 0) return set_error(KVC_EINVAL, "kvc_encode: negative t0 or n_tok");
    if ((int64_t)t0 + n_tok > s->capacity) return set_error(KVC_ENOSPACE, "kvc_encode: t0 + n_tok > capacity");
    if (n_tok == 0 || s->n_units == 0) return KVC_OK;
    if (!x || (reinterpret_cast<uintptr_t>(x) & 15) || (x_unit_stride & 7) || x_unit_stride < (int64_t)n_tok * kD)
        return set_error(KVC_EINVAL, "kvc_encode: x must be 16-byte aligned with stride a multiple of 8 and >= n_tok*d");
    if (n_tok <= kAppMaxTok) {
        hipLaunchKernelGGL(append_kernel, dim3(s->n_units), dim3(kAppThreads), 0, (hipStream_t)stream, dev_side(s),
                           s->side, x, x_unit_stride, t0, n_tok);
        return check_launch("kvc_encode");
    }
    const DevSide d = dev_side(s);
    return launch_encode(d, d, x, x_unit_stride, x, x_unit_stride, s->side, 1, s->n_units, t0, n_tok, stream);
}

extern "C" int kvc_encode_kv(const kvc_stream_desc* k, const kvc_stream_desc* v, const uint16_t* xk,
                             int64_t xk_unit_stride, const uint16_t* xv, int64_t xv_unit_stride, int32_t t0,
                             int32_t n_tok, void* stream) {
    clear_error();
    if (int e = validate_desc(k, "kvc_encode_kv(k)")) return e;
    if (int e = validate_desc(v, "kvc_encode_kv(v)")) return e;
    if (k->side != KVC_SIDE_K || v->side != KVC_SIDE_V) return set_error(KVC_EINVAL, "kvc_encode_kv: descriptor sides");
    if (k->n_units != v->n_units) return set_error(KVC_EINVAL, "kvc_encode_kv: K and V unit counts differ");
    if (t0 < 0 || n_tok < 0) return set_error(KVC_EINVAL, "kvc_encode_kv: negative t0 or n_tok");
    if ((int64_t)t0 + n_tok > k->capacity || (int64_t)t0 + n_tok > v->capacity)
        return set_error(KVC_ENOSPACE, "kvc_encode_kv: t0 + n_tok > capacity");
    if (n_tok == 0 || k->n_units == 0) return KVC_OK;
    for (const auto& xs : {std::make_pair(xk, xk_unit_stride), std::make_pair(xv, xv_unit_stride)})
        if (!xs.first || (reinterpret_cast<uintptr_t>(xs.first) & 15) || (xs.second & 7) || xs.second < (int64_t)n_tok * kD)
            return set_error(KVC_EINVAL, "kvc_encode_kv: x must be 16-byte aligned with stride a multiple of 8 and >= n_tok*d");
    if (n_tok > kAppMaxTok)  // runs of tiles: the bulk encoder, both sides in one launch
        return launch_encode(dev_side(k), dev_side(v), xk, xk_unit_stride, xv, xv_unit_stride, KVC_SIDE_K, 2, k->n_units, t0, n_tok,
                             stream);
    hipLaunchKernelGGL(append_kv_kernel, dim3(k->n_units, 2), dim3(kAppThreads), 0, (hipStream_t)stream, dev_side(k),
                       dev_side(v), xk, xk_unit_stride, xv, xv_unit_stride, t0, n_tok);
    return check_launch("kvc_encode_kv");
}
