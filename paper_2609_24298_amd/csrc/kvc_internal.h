// Internal declarations shared by the host (kvc_host.cpp) and device (kvc_kernels.hip)
// halves of libkvc. Not part of the public ABI.
#pragma once

#include <cstdint>

#include "kvc.h"

namespace kvc {

// Records a thread-local error message and returns `code`.
int set_error(int code, const char* fmt, ...);
// Clears the thread-local error message.
void clear_error();

// Host-side checks of a stream descriptor (pointers, per-unit r/b/offset/step
// ranges, arena bounds for `capacity` tokens). Returns KVC_OK or an error.
int validate_desc(const kvc_stream_desc* s, const char* name);

// Bytes of a stream holding n_tok tokens: whole 64-token tiles of 8*r*b bytes.
inline int64_t stream_bytes(int64_t n_tok, int r, int b) {
    return ((n_tok + KVC_TILE_TOKENS - 1) / KVC_TILE_TOKENS) * 8LL * r * b;
}

// Elements of one lane of the bulk encoder that are coordinates of the unit, bit 4 nt + i for element i of
// quarter nt, in a group of 16 coordinates of which the first `left` exist. Lane (col, grp) holds
// coordinates 4 grp + i on the K side and coordinate col on the V side. Only these may be settled: the
// basis has no row for the others.
constexpr uint32_t encode_rank_mask(int side, int left, int col, int grp) {
    if (side == KVC_SIDE_V) return col < left ? 0xffffu : 0u;
    const int n = left - 4 * grp;
    return n <= 0 ? 0u : (n >= 4 ? 0xffffu : 0x1111u * ((1u << n) - 1u));
}

}  // namespace kvc
