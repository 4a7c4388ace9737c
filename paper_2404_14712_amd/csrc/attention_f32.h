// float32 attention kernels for small grids (head_dim 32, 64 or 128).
#pragma once
#include "common.h"

namespace orbit {

struct AttnF32Args {
  const float *q, *k, *v, *dO;      // per-sample rows, head h at column h * head_dim
  int64_t ldq, ldk, ldv, lddo;
  float *o, *o32;                   // forward (o32 may be NULL)
  int64_t ldo, ldo32;
  float* lse_out;
  const float *lse, *D;             // backward: [B, H, L]
  const float *qsum, *ksum;         // per (sample, head, feature) sums over the sequence
  float *dq, *dk, *dv;
  int64_t ldg;
  int H, L;
  float sl2, scale;                 // log2(e) / sqrt(head_dim), 1 / sqrt(head_dim)
};

orbit_status attn_f32_forward(const AttnF32Args& a, int B, int dh, hipStream_t s);
orbit_status attn_f32_backward(const AttnF32Args& a, int B, int dh, hipStream_t s);

}  // namespace orbit
