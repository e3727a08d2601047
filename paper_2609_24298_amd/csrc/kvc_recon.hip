// Kernels that rebuild vectors from their codes on CDNA4 (gfx950): kvc_reconstruct
// (x_hat = P^T z, Lemma lem:head-dist). The product is a dense contraction over the rank
// and runs on v_mfma_f32_16x16x32_f16: the centred codes c - 2^(b-1) + 1/2 and the basis
// are exact in fp16, their products exact, the accumulation fp32, and the step multiplies
// the result once.
#define KVC_DECODE_PARTIALS_UNIT
#include "kvc_decode.hip"

#include "kvc_codes.h"

namespace kvc {

// ---------------------------------------------------------------- reconstruct

// One block of four wavefronts per (unit, run of tiles): P^T staged once, each wavefront takes whole
// 64-token tiles, in pairs of 16-token columns that share every P^T operand read.
//  K: the packed fields are the decode's direct loads (lane (col, kq): tokens 4 col + st, group 4 ks + kq),
//     and a field's pairs are the operand itself; only a tail K-step (r % 16) goes through LDS.
//  V: a field is 16 tokens of one coordinate, so the unpacked bytes are transposed (4 x 4 in registers,
//     the rest through LDS, token-major rows of kZbPitch bytes) and widened to fp16 on the way back.
// Lane (col, grp) then holds features 16 rb + 4 grp + v of token column col: 16-byte stores, 64 bytes
// per token and instruction. Bound by writing the fp32 result: 64 units x 4096 tokens, both sides, 2 bpd
// (268 MB written): 68 us (4.2 TB/s with the codes; 1874 us with one scalar unpack per code and an fp32
// VALU product).
constexpr int kRecWaves = 4;
constexpr int kZbPitch = kD + 4;                       // 33 dwords: the quarters' rows fall on different banks
constexpr int kRecWaveLds = kTile * kZbPitch;          // also holds a staged K-step (at most 512 * 8 + 32 bytes)
static_assert(kRecWaveLds >= 512 * 8 + 32, "staged K-step exceeds the wavefront's LDS");
constexpr int kRecShared = kBtBytes;

// The 16 columns of tokens in za and the 16 in zb times P^T, to the rows of tokens ta and tb (< 0: none).
template <int NS>
__device__ __forceinline__ void rec_store_pair(const uint8_t* __restrict__ PT, const rc_h8 (&za)[NS], const rc_h8 (&zb)[NS],
                                               float step, bool vec, float* __restrict__ oa, float* __restrict__ ob,
                                               int col, int grp) {
#pragma unroll
    for (int rb = 0; rb < 8; ++rb) {
        rc_f4 ca = rc_f4{0.f, 0.f, 0.f, 0.f}, cb = ca;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const rc_h8 p = *reinterpret_cast<const rc_h8*>(PT + bt_block(rb, s) + bt_lane(col, grp));
            ca = mfma_h(p, za[s], ca);
            cb = mfma_h(p, zb[s], cb);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) { ca[v] *= step; cb[v] *= step; }
        const int f = 16 * rb + 4 * grp;
        if (vec) {
            if (oa) *reinterpret_cast<rc_f4*>(oa + f) = ca;
            if (ob) *reinterpret_cast<rc_f4*>(ob + f) = cb;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (oa) oa[f + v] = ca[v];
                if (ob) ob[f + v] = cb[v];
            }
        }
    }
}

// K tile: NS = 2 nk matrix steps, nk K-steps of four coordinate groups.
template <int B, int NK>
__device__ __forceinline__ void rec_tile_k(const uint8_t* __restrict__ PT, uint8_t* __restrict__ stage,
                                           const __amdgpu_buffer_rsrc_t rs, int r, float step, bool vec, float* __restrict__ out,
                                           int tok0, int lo, int hi, int lane) {
    const int col = lane & 15, grp = lane >> 4;
    const int g16 = r >> 4, rho = r & 15, ks_t = rho ? (g16 >> 2) : 2;
    constexpr int W0 = k_step_words(B);
    const uint32_t e512 = exp512();
    uint32_t w[NK * W0];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        const int cg = 4 * ks + grp;
        const uint32_t lk = ks == ks_t ? (uint32_t)(512 * ks + 8 * lane) : (cg < g16 ? (uint32_t)(128 * cg + 8 * col) : kLaneOOB);
        k_load_direct<B>(rs, r, lk, w + ks * W0);
    }
    uint32_t xb = 0, xs = 0;  // staged token fields start at plane-width units xb + st xs
    if (ks_t < NK) {
        const int nf = g16 - 4 * ks_t;
        if (grp < nf) { xb = (uint32_t)((64 * grp + 4 * col) * 16); xs = 16; }
        else if (grp == nf) { xb = (uint32_t)(nf * 1024 + 4 * col * rho); xs = (uint32_t)rho; }
        wave_lds_sync();
        if (NK == 1 || ks_t == 0) k_write_stage<B>(w, stage, lane);
        else k_write_stage<B>(w + (NK - 1) * W0, stage, lane);
        wave_lds_sync();
    }
#pragma unroll
    for (int sp = 0; sp < 4; sp += 2) {
        rc_h8 z[2][2 * NK];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                Fld f[3];
                rc_h8 zz[2];
                if (ks == ks_t) {
                    k_fields_staged<B>(stage, xb + (sp + h) * xs, f);
                    k_pairs<B>(f, false, e512, zz);
                } else {
                    k_fields_direct<B>(w + ks * W0, sp + h, f);
                    k_pairs<B>(f, ((sp + h) & 1) != 0, e512, zz);
                }
                z[h][2 * ks] = zz[0];
                z[h][2 * ks + 1] = zz[1];
            }
        const int ta = tok0 + 4 * col + sp, tb = ta + 1;
        rec_store_pair<2 * NK>(PT, z[0], z[1], step, vec, ta >= lo && ta < hi ? out + (int64_t)(ta - lo) * kD : nullptr,
                               tb >= lo && tb < hi ? out + (int64_t)(tb - lo) * kD : nullptr, col, grp);
    }
}

// V tile, NH halves of four N-tiles each (64 coordinates, two matrix steps).
template <int B, int NH>
__device__ __forceinline__ void rec_tile_v(const uint8_t* __restrict__ PT, uint8_t* __restrict__ zb,
                                           const __amdgpu_buffer_rsrc_t rs, int r, float step, bool vec, float* __restrict__ out,
                                           int tok0, int lo, int hi, int lane) {
    const int col = lane & 15, grp = lane >> 4;
    const uint32_t L = (uint32_t)(4 * col + grp), A = v_lane_adj(r, col, grp);
    // every group of every plane in flight (4 p words per plane of width p for a whole rank)
    uint32_t gw[3][4 * (B == 8 ? 8 : 4)];
#pragma unroll
    for (int k = 0; k < n_planes(B); ++k) {
        const int g = v_group(plane_w(B, k));
#pragma unroll
        for (int Q = 0; Q < cdiv(4 * NH, g); ++Q) {
            const v4u v = v_group_load<B>(rs, k, Q, r, L, A);
#pragma unroll
            for (int j = 0; j < 4; ++j) gw[k][4 * Q + j] = v[j];
        }
        if (plane_w(B, k) == 1) {  // the only group may start at 2 mod 4 bytes (see v_tile)
            const uint32_t sh = ((L * (uint32_t)((r + 15) >> 4) - A) & 1u) << 4;
            uint32_t* w = gw[k];
            w[0] = funnel(w[1], w[0], sh);
            w[1] = funnel(w[2], w[1], sh);
            w[2] = funnel(w[3], w[2], sh);
            w[3] = w[3] >> sh;
        }
    }
    wave_lds_sync();  // the previous tile's rows have been read
#pragma unroll
    for (int a = 0; a < NH; ++a) {
        v4i D[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int nt = 4 * a + n;
            Fld f[3];
            bool h1 = false;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (k < n_planes(B)) {
                    const int P = plane_w(B, k), g = v_group(P), j = nt % g;
                    const uint32_t* w = gw[k] + 4 * (nt / g);
                    if (P == 1) { f[k] = Fld{w[j >> 1], 0u, 0u, 0u}; h1 = (j & 1) != 0; }
                    else if (P == 2) f[k] = Fld{w[j], 0u, 0u, 0u};
                    else if (P == 4) f[k] = Fld{w[2 * j], w[2 * j + 1], 0u, 0u};
                    else f[k] = Fld{w[0], w[1], w[2], w[3]};
                } else {
                    f[k] = Fld{0u, 0u, 0u, 0u};
                }
            }
            D[n] = unpack16<B>(f, h1);
        }
        // byte k of D[n][d]: token 16 grp + 4 d + k, coordinate 16 (4 a + n) + col; 4 x 4 transpose over n, k
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t t0 = perm(D[1][d], D[0][d], 0x05010400u), t1 = perm(D[1][d], D[0][d], 0x07030602u);
            const uint32_t s0 = perm(D[3][d], D[2][d], 0x05010400u), s1 = perm(D[3][d], D[2][d], 0x07030602u);
            uint8_t* row = zb + (16 * grp + 4 * d) * kZbPitch + 64 * a + 4 * col;
            *reinterpret_cast<uint32_t*>(row) = perm(s0, t0, 0x05040100u);
            *reinterpret_cast<uint32_t*>(row + kZbPitch) = perm(s0, t0, 0x07060302u);
            *reinterpret_cast<uint32_t*>(row + 2 * kZbPitch) = perm(s1, t1, 0x05040100u);
            *reinterpret_cast<uint32_t*>(row + 3 * kZbPitch) = perm(s1, t1, 0x07060302u);
        }
    }
    wave_lds_sync();
    const _Float16 sh = (_Float16)(0.5f - (float)(1 << (B - 1)));
    const rc_h2 m1024 = rc_h2{(_Float16)-1024.f, (_Float16)-1024.f}, sh2 = rc_h2{sh, sh};
    auto widen = [&](uint32_t w, uint32_t sel) {  // two code bytes under the exponent of 1024, then centred (both adds exact)
        return __builtin_bit_cast(uint32_t, (__builtin_bit_cast(rc_h2, perm(0x64646464u, w, sel)) + m1024) + sh2);
    };
#pragma unroll
    for (int tp = 0; tp < 4; tp += 2) {
        rc_h8 z[2][2 * NH];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 2 * NH; ++s) {
                const uint32_t* p = reinterpret_cast<const uint32_t*>(zb + (16 * (tp + h) + col) * kZbPitch + 32 * s + 8 * grp);
                uint32_t w0 = p[0], w1 = p[1];
                if (B == 8) { w0 ^= 0x80808080u; w1 ^= 0x80808080u; }  // unpack16 centres 8-bit codes
                z[h][s] = __builtin_bit_cast(rc_h8, v4u{widen(w0, 0x05010400u), widen(w0, 0x05030402u),
                                                        widen(w1, 0x05010400u), widen(w1, 0x05030402u)});
            }
        const int ta = tok0 + 16 * tp + col, tb = ta + 16;
        rec_store_pair<2 * NH>(PT, z[0], z[1], step, vec, ta >= lo && ta < hi ? out + (int64_t)(ta - lo) * kD : nullptr,
                               tb >= lo && tb < hi ? out + (int64_t)(tb - lo) * kD : nullptr, col, grp);
    }
}

template <int side, int B, int NK>
__device__ __forceinline__ void rec_tiles(const DevSide& s, const uint8_t* __restrict__ PT, uint8_t* __restrict__ wl, int u, int r,
                                          int cap_tiles, int t0, int n_tok, int tile_first, int n_tiles, int tpb, bool vec,
                                          float* __restrict__ out, int wv, int lane) {
    const float step = s.delta[u];
    const uint8_t* stream = uni(s.codes + s.code_off[u]);
    const int tb = 8 * r * B;
    for (int tt = wv; tt < tpb; tt += kRecWaves) {
        const int tl = blockIdx.x * tpb + tt;
        if (tl >= n_tiles) break;
        const int tile = tile_first + tl;
        const int64_t left = (int64_t)(cap_tiles - tile) * tb;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(stream + (int64_t)tile * tb), (short)0,
                                                          (int)(left < (1 << 30) ? left : (1 << 30)), kRsrcWord3);
        if constexpr (side == KVC_SIDE_K) rec_tile_k<B, NK>(PT, wl, rs, r, step, vec, out, tile * kTile, t0, t0 + n_tok, lane);
        else rec_tile_v<B, NK>(PT, wl, rs, r, step, vec, out, tile * kTile, t0, t0 + n_tok, lane);
    }
}

template <int side>
__global__ __launch_bounds__(64 * kRecWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void reconstruct_kernel(
    DevSide s, int cap_tiles, int t0, int n_tok, int tile_first, int n_tiles, int tpb, int vec, float* __restrict__ out) {
    uint8_t* PT = kvc_dsm;
    const int u = blockIdx.y, wv = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int r = uni(s.r[u]), b = uni(s.b[u]);
    stage_basis_t<side>(PT, s.basis + s.basis_off[u], r, threadIdx.x, 64 * kRecWaves);
    __syncthreads();
    uint8_t* wl = kvc_dsm + kRecShared + wv * kRecWaveLds;
    float* o = out + (int64_t)u * n_tok * kD;
    if (r > 64) {
        KVC_SWITCH_B(b, (rec_tiles<side, B_, 2>(s, PT, wl, u, r, cap_tiles, t0, n_tok, tile_first, n_tiles, tpb, vec != 0, o, wv, lane)));
    } else {
        KVC_SWITCH_B(b, (rec_tiles<side, B_, 1>(s, PT, wl, u, r, cap_tiles, t0, n_tok, tile_first, n_tiles, tpb, vec != 0, o, wv, lane)));
    }
}

}  // namespace kvc

using namespace kvc;

extern "C" int kvc_reconstruct(const kvc_stream_desc* s, int32_t t0, int32_t n_tok, float* out, void* stream) {
    clear_error();
    if (int e = validate_desc(s, "kvc_reconstruct")) return e;
    if (t0 < 0 || n_tok < 0) return set_error(KVC_EINVAL, "kvc_reconstruct: negative t0 or n_tok");
    if ((int64_t)t0 + n_tok > s->capacity) return set_error(KVC_ENOSPACE, "kvc_reconstruct: t0 + n_tok > capacity");
    if (n_tok == 0 || s->n_units == 0) return KVC_OK;
    if (!out) return set_error(KVC_EINVAL, "kvc_reconstruct: null output");
    const int tile_first = t0 / kTile, n_tiles = (t0 + n_tok - 1) / kTile - tile_first + 1;
    const int cap_tiles = (int)(((int64_t)s->capacity + kTile - 1) / kTile);
    // Tiles per block: about two blocks for every place the chip has (two blocks of four wavefronts per
    // CU), a multiple of the four wavefronts; longer runs share one staging of the basis.
    const int64_t want = ((int64_t)s->n_units * n_tiles + 1023) / 1024;
    const int tpb = (int)(want < 4 ? 4 : (want > 64 ? 64 : (want + 3) / 4 * 4));
    const size_t smem = (size_t)kRecShared + (size_t)kRecWaves * kRecWaveLds;
    const int vec = (reinterpret_cast<uintptr_t>(out) & 15) == 0;  // 16-byte stores, else 4-byte ones
    const void* fn = s->side == KVC_SIDE_K ? (const void*)reconstruct_kernel<KVC_SIDE_K> : (const void*)reconstruct_kernel<KVC_SIDE_V>;
    const hipError_t he = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (he != hipSuccess) return set_error(KVC_EDEVICE, "hipFuncSetAttribute: %s", hipGetErrorString(he));
    const dim3 grid((n_tiles + tpb - 1) / tpb, s->n_units), blk(64 * kRecWaves);
    if (s->side == KVC_SIDE_K)
        hipLaunchKernelGGL(reconstruct_kernel<KVC_SIDE_K>, grid, blk, smem, (hipStream_t)stream, dev_side(s), cap_tiles, t0, n_tok,
                           tile_first, n_tiles, tpb, vec, out);
    else
        hipLaunchKernelGGL(reconstruct_kernel<KVC_SIDE_V>, grid, blk, smem, (hipStream_t)stream, dev_side(s), cap_tiles, t0, n_tok,
                           tile_first, n_tiles, tpb, vec, out);
    return check_launch("kvc_reconstruct");
}
