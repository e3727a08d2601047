// Kernels that rebuild vectors from their codes on CDNA4 (gfx950): kvc_reconstruct
// (x_hat = P^T z, Lemma lem:head-dist). The product is a dense contraction over the rank
// and runs on v_mfma_f32_16x16x32_f16: the centred codes c - 2^(b-1) + 1/2 and the basis
// are exact in fp16, their products exact, the accumulation fp32, and the step multiplies
// the result once.
#define KVC_DECODE_PARTIALS_UNIT
#include "kvc_decode.hip"

namespace kvc {

typedef _Float16 rc_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 rc_h2 __attribute__((ext_vector_type(2)));
typedef float rc_f4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- operands

// P^T in LDS: one row of kBtPitch halves per feature, its coordinates in the order of the operand
// that meets it (the order of the contraction index is free):
//  K: matrix step s, lane part kq, element e <-> coordinate 16 (4 (s / 2) + kq) + 4 (s % 2) + e / 2 + 8 (e % 2),
//     which is where the code pairs (m, m + 8) of a token's 16-code field land (k_pairs);
//  V: position 64 a + 4 c + n <-> coordinate 16 (4 a + n) + c, where the transposed value bytes land.
constexpr int kBtPitch = kD + 8;

template <int side>
__host__ __device__ constexpr int bt_coord(int p) {
    if (side == KVC_SIDE_K) {
        const int s = p >> 5, kq = (p >> 3) & 3, e = p & 7;
        return 16 * (4 * (s >> 1) + kq) + 4 * (s & 1) + (e >> 1) + 8 * (e & 1);
    }
    return 16 * (4 * (p >> 6) + (p & 3)) + ((p >> 2) & 15);
}

// Stages P^T (rows of P past the rank are zero, so codes past the rank meet zeros): a thread takes four
// positions and eight features, lanes consecutive positions (conflict-free 8-byte LDS writes).
template <int side, int THREADS>
__device__ __forceinline__ void stage_basis_t(uint16_t* __restrict__ PT, const uint16_t* __restrict__ P, int r, int tid) {
    for (int e = tid; e < (kD / 4) * (kD / 8); e += THREADS) {
        const int w = e & (kD / 4 - 1), f0 = 8 * (e / (kD / 4));
        uint32_t x[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = bt_coord<side>(4 * w + j);
            const uint4 v = i < r ? *reinterpret_cast<const uint4*>(P + (int64_t)i * kD + f0) : uint4{0u, 0u, 0u, 0u};
            x[j][0] = v.x; x[j][1] = v.y; x[j][2] = v.z; x[j][3] = v.w;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t sel = (k & 1) ? 0x07060302u : 0x05040100u;
            *reinterpret_cast<uint2*>(PT + (f0 + k) * kBtPitch + 4 * w) =
                uint2{perm(x[1][k >> 1], x[0][k >> 1], sel), perm(x[3][k >> 1], x[2][k >> 1], sel)};
        }
    }
}

__device__ __forceinline__ uint32_t shl_or_shr(uint32_t x, int right) { return right >= 0 ? x >> right : x << -right; }

// The pairs (m, m + 8) of a field of 16 codes of one plane of width P, their bits shifted up by LS:
// bits [LS, LS + P) and [16 + LS, 16 + LS + P) of pr[m], the rest zero. hi: the upper half of a 1-bit
// plane's word.
template <int P, int LS>
__device__ __forceinline__ void plane_pairs(const Fld& f, bool hi, uint32_t (&pr)[8]) {
    if constexpr (P == 1) {
        const uint32_t y = perm(0u, f.w0, hi ? 0x0c030c02u : 0x0c010c00u);  // code m at bit m, m + 8 at 16 + m
#pragma unroll
        for (int m = 0; m < 8; ++m) pr[m] = shl_or_shr(y, m - LS) & (0x00010001u << LS);
    } else if constexpr (P == 2) {
#pragma unroll
        for (int m = 0; m < 8; ++m) pr[m] = shl_or_shr(f.w0, 2 * m - LS) & (0x00030003u << LS);
    } else if constexpr (P == 4) {
        const uint32_t y0 = perm(f.w1, f.w0, 0x05040100u), y1 = perm(f.w1, f.w0, 0x07060302u);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            pr[m] = shl_or_shr(y0, 4 * m - LS) & (0x000f000fu << LS);
            pr[m + 4] = shl_or_shr(y1, 4 * m - LS) & (0x000f000fu << LS);
        }
    } else {
        const uint32_t w[4] = {f.w0, f.w1, f.w2, f.w3};
#pragma unroll
        for (int m = 0; m < 8; ++m)  // byte m % 4 of dwords m / 4 and m / 4 + 2, zero bytes between
            pr[m] = perm(w[(m >> 2) + 2], w[m >> 2], 0x0c040c00u + 0x00010001u * (uint32_t)(m & 3)) << LS;
    }
}

// A token's 16 codes of a coordinate group as two fp16 operand fragments (matrix steps 2 ks and
// 2 ks + 1): per pair, the code's bits one up under the fp16 exponent of 512 give 512 + c (exact, the
// spacing there is 1/2), and one packed add of -512 - 2^(b-1) + 1/2 the centred code (exact).
template <int B>
__device__ __forceinline__ void k_pairs(const Fld (&f)[3], bool hi, rc_h8 (&z)[2]) {
    const _Float16 sh = (_Float16)(-512.f - ((float)(1 << (B - 1)) - 0.5f));
    const rc_h2 sh2 = rc_h2{sh, sh};
    uint32_t pc[8];
    plane_pairs<plane_w(B, 0), plane_sh(B, 0) + 1>(f[0], hi, pc);
    if constexpr (n_planes(B) > 1) {
        uint32_t pr[8];
        plane_pairs<plane_w(B, 1), plane_sh(B, 1) + 1>(f[1], hi, pr);
#pragma unroll
        for (int m = 0; m < 8; ++m) pc[m] |= pr[m];
    }
    if constexpr (n_planes(B) > 2) {
        uint32_t pr[8];
        plane_pairs<plane_w(B, 2), plane_sh(B, 2) + 1>(f[2], hi, pr);
#pragma unroll
        for (int m = 0; m < 8; ++m) pc[m] |= pr[m];
    }
    uint32_t hw[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) hw[m] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(rc_h2, pc[m] | 0x60006000u) + sh2);
#pragma unroll
    for (int h = 0; h < 2; ++h)
        z[h] = __builtin_bit_cast(rc_h8, v4u{hw[4 * h], hw[4 * h + 1], hw[4 * h + 2], hw[4 * h + 3]});
}

__device__ __forceinline__ rc_f4 mfma_h(rc_h8 a, rc_h8 b, rc_f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

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
constexpr int kRecShared = kD * kBtPitch * 2;

// The 16 columns of tokens in za and the 16 in zb times P^T, to the rows of tokens ta and tb (< 0: none).
template <int NS>
__device__ __forceinline__ void rec_store_pair(const uint16_t* __restrict__ PT, const rc_h8 (&za)[NS], const rc_h8 (&zb)[NS],
                                               float step, bool vec, float* __restrict__ oa, float* __restrict__ ob,
                                               int col, int grp) {
#pragma unroll
    for (int rb = 0; rb < 8; ++rb) {
        rc_f4 ca = rc_f4{0.f, 0.f, 0.f, 0.f}, cb = ca;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const rc_h8 p = *reinterpret_cast<const rc_h8*>(PT + (16 * rb + col) * kBtPitch + 32 * s + 8 * grp);
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
__device__ __forceinline__ void rec_tile_k(const uint16_t* __restrict__ PT, uint8_t* __restrict__ stage,
                                           const __amdgpu_buffer_rsrc_t rs, int r, float step, bool vec, float* __restrict__ out,
                                           int tok0, int lo, int hi, int lane) {
    const int col = lane & 15, grp = lane >> 4;
    const int g16 = r >> 4, rho = r & 15, ks_t = rho ? (g16 >> 2) : 2;
    constexpr int W0 = k_step_words(B);
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
                    k_pairs<B>(f, false, zz);
                } else {
                    k_fields_direct<B>(w + ks * W0, sp + h, f);
                    k_pairs<B>(f, ((sp + h) & 1) != 0, zz);
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
__device__ __forceinline__ void rec_tile_v(const uint16_t* __restrict__ PT, uint8_t* __restrict__ zb,
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
__device__ __forceinline__ void rec_tiles(const DevSide& s, const uint16_t* __restrict__ PT, uint8_t* __restrict__ wl, int u, int r,
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
    uint16_t* PT = reinterpret_cast<uint16_t*>(kvc_dsm);
    const int u = blockIdx.y, wv = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int r = uni(s.r[u]), b = uni(s.b[u]);
    stage_basis_t<side, 64 * kRecWaves>(PT, s.basis + s.basis_off[u], r, threadIdx.x);
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
