// Streaming kernels of the variable aggregation (bf16, 8 or 16 heads, embeddings
// up to 2048): each direction takes the token tensor from HBM once.
#pragma once
#include "common.h"

namespace orbit {

// The streaming path's domain. A function of the descriptor alone, since it
// also fixes the layout of the saved attention weights ([T, V, H] here,
// [T, H, V] on the general path), which forward and backward must agree on.
bool agg_stream_ok(orbit_dtype dt, int V, int d, int H);

// blocks of the backward, each of which leaves one [H, agg_stream_cols(d)] partial of dU
int agg_stream_blocks(int64_t T, int d);
int agg_stream_cols(int d);

// scores, softmax over the variables and xbar in one pass:
// a32 [T, V, H] float32, xbar [T, H, d]
orbit_status agg_stream_fwd(const bf16* tok, const bf16* Ut, float* a32, bf16* xbar, int64_t T, int V, int d, int H,
                            float scale, hipStream_t s);

// dA, softmax backward, dtok and the partials of dU in one kernel; dU [d, H]
// float32 is finished from the partials
orbit_status agg_stream_bwd(const bf16* tok, const bf16* dxbar, const bf16* Ut, const float* a32, bf16* dtok,
                            float* part, float* dU, int64_t T, int V, int d, int H, float scale, hipStream_t s);

}  // namespace orbit
