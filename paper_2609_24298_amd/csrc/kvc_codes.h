// fp16 operands of packed codes, shared by the kernels that rebuild vectors (kvc_recon.hip, kvc_rope.hip):
// the transposed basis in LDS and the centred K codes of a token as matrix-core fragments. Included after
// kvc_decode.hip (field extraction). CDNA4 / gfx950 only.
#pragma once

namespace kvc {

typedef _Float16 rc_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 rc_h2 __attribute__((ext_vector_type(2)));
typedef float rc_f4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- operands

// P^T in LDS in fragment order: 1 KB per (16 features rb, matrix step s), 16 bytes per lane (feature
// 16 rb + col, positions 32 s + 8 grp + [0, 8)), so that operand reads are contiguous over the wavefront
// (padded feature rows cost 40 % of the reads' LDS cycles in bank conflicts). The 16 lanes of a lane row are
// permuted by their low bits (slot col ^ grp), which spreads the staging writes over four bank groups. The
// coordinates are in the order of the operand that meets them (the order of the contraction index is free):
//  K: matrix step s, lane part kq, element e <-> coordinate 16 (4 (s / 2) + kq) + 4 (s % 2) + e / 2 + 8 (e % 2),
//     which is where the code pairs (m, m + 8) of a token's 16-code field land (k_pairs);
//  V: position 64 a + 4 c + n <-> coordinate 16 (4 a + n) + c, where the transposed value bytes land.
constexpr int kBtBytes = kD * kD * 2;
__host__ __device__ constexpr int bt_block(int rb, int s) { return (4 * rb + s) * 1024; }
__device__ __forceinline__ int bt_lane(int col, int grp) { return 256 * grp + 16 * (col ^ grp); }

template <int side>
__host__ __device__ constexpr int bt_coord(int p) {
    if (side == KVC_SIDE_K) {
        const int s = p >> 5, kq = (p >> 3) & 3, e = p & 7;
        return 16 * (4 * (s >> 1) + kq) + 4 * (s & 1) + (e >> 1) + 8 * (e & 1);
    }
    return 16 * (4 * (p >> 6) + (p & 3)) + ((p >> 2) & 15);
}

// Stages P^T (rows of P past the rank are zero, so codes past the rank meet zeros): a thread takes four
// positions and eight features, lanes consecutive positions.
template <int side>
__device__ __forceinline__ void stage_basis_t(uint8_t* __restrict__ PT, const uint16_t* __restrict__ P, int r, int tid, int threads) {
    for (int e = tid; e < (kD / 4) * (kD / 8); e += threads) {
        const int w = e & (kD / 4 - 1), f0 = 8 * (e / (kD / 4));
        uint32_t x[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = bt_coord<side>(4 * w + j);
            const uint4 v = i < r ? load_basis8(P + (int64_t)i * kD + f0) : uint4{0u, 0u, 0u, 0u};
            x[j][0] = v.x; x[j][1] = v.y; x[j][2] = v.z; x[j][3] = v.w;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t sel = (k & 1) ? 0x07060302u : 0x05040100u;
            const int f = f0 + k;
            *reinterpret_cast<uint2*>(PT + bt_block(f >> 4, w >> 3) + bt_lane(f & 15, (w >> 1) & 3) + 8 * (w & 1)) =
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

// Two fp16 exponents of 512, in a register the compiler does not know: masking a code pair and setting its
// exponents is then one instruction (it cannot hold two 32-bit literals).
__device__ __forceinline__ uint32_t exp512() {
    uint32_t e = 0x60006000u;
    asm volatile("" : "+v"(e));
    return e;
}

// A token's 16 codes of a coordinate group as two fp16 operand fragments (matrix steps 2 ks and
// 2 ks + 1): per pair, the code's bits one up under the fp16 exponent of 512 give 512 + c (exact, the
// spacing there is 1/2), and one packed add of -512 - 2^(b-1) + 1/2 the centred code (exact).
template <int B>
__device__ __forceinline__ void k_pairs(const Fld (&f)[3], bool hi, uint32_t e512, rc_h8 (&z)[2]) {
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
    for (int m = 0; m < 8; ++m) hw[m] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(rc_h2, pc[m] | e512) + sh2);
#pragma unroll
    for (int h = 0; h < 2; ++h)
        z[h] = __builtin_bit_cast(rc_h8, v4u{hw[4 * h], hw[4 * h + 1], hw[4 * h + 2], hw[4 * h + 3]});
}

__device__ __forceinline__ rc_f4 mfma_h(rc_h8 a, rc_h8 b, rc_f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

}  // namespace kvc
