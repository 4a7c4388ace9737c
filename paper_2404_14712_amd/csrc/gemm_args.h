// Kernel arguments and fused epilogues shared by the GEMM kernels.
#pragma once
#include "common.h"

namespace orbit {

struct Epi {
  float alpha;
  int accumulate;
  const void* bias; int64_t sBias;
  void* gelu_out; int64_t ldgo;
  const void* gelu_in; int64_t ldgi;
  const void* res; int64_t ldr, sR; int res_row_mod;
};

struct GemmKArgs {
  const void* A; const void* B; const void* B2; void* C;
  int M, N, K, k_split;
  int64_t lda, ldb, ldc;
  int64_t sA, sB, sB2, sC;
  int batch, splits, k_per_split;
  int vec_ok;      // N, ldc, batch strides and epilogue operands allow 16-byte access
  float* partial;  // splits > 1: float32 partials [splits][batch][M][N]
  float* bsum;     // column sums of B: [splits][bs_groups][batch][N] (A M-major, B N-major)
  int bs_groups;   // tile rows that form them, each from a strided subset of the K slices
  Epi epi;
};

template <typename T, typename OutT>
ORBIT_DEV void epi_apply(const Epi& e, int64_t bz, int r, int c, float v, OutT* C, int64_t ldc) {
  v *= e.alpha;
  const int64_t off = (int64_t)r * ldc + c;
  if (e.accumulate) v += to_f(C[off]);
  if (e.bias) v += to_f(static_cast<const T*>(e.bias)[bz * e.sBias + c]);
  if (e.gelu_out) {
    static_cast<T*>(e.gelu_out)[(int64_t)r * e.ldgo + c] = from_f<T>(v);
    v = gelu_f(v);
  }
  if (e.gelu_in) v *= gelu_grad_f(to_f(static_cast<const T*>(e.gelu_in)[(int64_t)r * e.ldgi + c]));
  if (e.res) {
    const int rr = e.res_row_mod ? r % e.res_row_mod : r;
    v += to_f(static_cast<const T*>(e.res)[bz * e.sR + (int64_t)rr * e.ldr + c]);
  }
  C[off] = from_f<OutT>(v);
}

// 8 consecutive columns c0..c0+7 of row r (16-byte aligned rows)
template <typename T> ORBIT_DEV void ld8(const T* p, float* f) {
  unpack(ld128(p), f, (T*)nullptr);
  if constexpr (sizeof(T) == 4) unpack(ld128(p + 4), f + 4, (T*)nullptr);
}
template <typename T> ORBIT_DEV void st8(T* p, const float* f) {
  st128(p, pack(f, (T*)nullptr));
  if constexpr (sizeof(T) == 4) st128(p + 4, pack(f + 4, (T*)nullptr));
}

// b8: the bias of columns c0..c0+7 when the caller loaded it ahead (else NULL)
template <typename T, typename OutT>
ORBIT_DEV void epi_apply8(const Epi& e, int64_t bz, int r, int c0, float* v, OutT* C, int64_t ldc,
                          const float* b8 = nullptr) {
  const int64_t off = (int64_t)r * ldc + c0;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] *= e.alpha;
  float t[8];
  if (e.accumulate) {
    ld8(C + off, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  if (e.bias) {
    if (b8) {
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] = b8[i];
    } else {
      ld8(static_cast<const T*>(e.bias) + bz * e.sBias + c0, t);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  if (e.gelu_out) {
    st8(static_cast<T*>(e.gelu_out) + (int64_t)r * e.ldgo + c0, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = gelu_f(v[i]);
  }
  if (e.gelu_in) {
    ld8(static_cast<const T*>(e.gelu_in) + (int64_t)r * e.ldgi + c0, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= gelu_grad_f(t[i]);
  }
  if (e.res) {
    const int rr = e.res_row_mod ? r % e.res_row_mod : r;
    ld8(static_cast<const T*>(e.res) + bz * e.sR + (int64_t)rr * e.ldr + c0, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  st8(C + off, v);
}

}  // namespace orbit
