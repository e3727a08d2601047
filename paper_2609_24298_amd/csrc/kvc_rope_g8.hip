// The RoPE-aware partials kernel for 8 query heads per KV head, compiled apart from kvc_rope.hip (which
// defines it and declares this instantiation external) so that the instantiations build in parallel.
// CDNA4 / gfx950 only.
#define KVC_ROPE_UNIT
#include "kvc_rope.hip"

namespace kvc {
template __global__ void decode_rope_kernel<8>(DevSide, DevSide, const uint16_t*, int, const int32_t*, int, int, int, int, int,
                                               double, int, float*);
}  // namespace kvc
