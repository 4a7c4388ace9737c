// float32 products on split bf16 matrix instructions.
#pragma once
#include "gemm_args.h"

namespace orbit {

// One product on tile x tile blocks (128, 64 or 32; 64: a_kmajor only; 32: one K range only),
// launched on s. The split-K partials (a.splits > 1) are left to the caller.
// Byte offsets within a tile, and of a 32-tile's whole operands, stay below 2^31.
orbit_status gemm_f32_launch(int tile, bool a_kmajor, bool b_kmajor, const GemmKArgs& a, hipStream_t s);

}  // namespace orbit
