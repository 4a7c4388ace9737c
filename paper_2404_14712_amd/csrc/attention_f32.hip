// float32 attention for small grids.
//
// A block owns 32 queries (keys in the key-major backward) and its four waves
// take every fourth 32-row tile of the other side; operands go from global
// memory (L2) straight into float32 MFMA fragments, so the sweep has no LDS and
// no barrier, and the waves' partial results are combined through LDS in a
// fixed order at the end. The 128-row blocks of the general kernels leave most
// CUs idle here: 1024 tokens x 16 heads are 128 blocks, 128 tokens x 4 heads x 2
// samples 8.
//
// What bounds it is the latency of the fragment loads (the forward has the next
// tile's keys in flight; the backward has no registers left for that) and, once
// the grid fills the chip, the L2 reads of the swept operand, which every block
// reads whole. Measured, general kernels -> these (forward / dK,dV / dQ, us):
//   1 sample x 16 heads x 1024 x 64   80 / 159 / 110 -> 52 / 100 / 81
//   1 x 4 x 300 x 32                  20 / 36 / 24   -> 13 / 18 / 13
//   2 x 4 x 128 x 32                  11 / 18 / 13   -> 8 / 10 / 8
#include "attention_f32.h"

namespace orbit {
namespace {

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// one (sample, head) slice X[row][0 .. DH) as a buffer: rows at and past L read zeros
template <int DH>
struct Slice {
  __amdgpu_buffer_rsrc_t rs;
  int ldb;            // bytes per row
  unsigned ro, co;    // lane offsets of row and column fragments
  ORBIT_DEV void init(const float* X, int64_t ld, int L, int lane) {
    ldb = (int)ld * 4;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X), 0, (L - 1) * ldb + DH * 4, 0x00020000);
    ro = (unsigned)((lane & 31) * ldb + (lane >> 5) * 32);
    co = (unsigned)((lane >> 5) * 4 * ldb + (lane & 31) * 4);
  }
  // rows row0 + lane % 32, features 16 kk + 8 (lane / 32) .. + 7
  ORBIT_DEV void row(Frag<float>& f, int row0, int kk) const {
    const unsigned o = ro + (unsigned)(row0 * ldb + kk * 64);
    f.lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
    f.hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16u, 0, 0));
  }
  // feature 32 c + lane % 32 of the 8 rows that an accumulator's registers
  // 8 kk .. + 7 hold: row0 + 16 kk + 8 (j / 4) + 4 (lane / 32) + j % 4
  ORBIT_DEV void col(Frag<float>& f, int row0, int kk, int c) const {
    const unsigned o = co + (unsigned)((row0 + kk * 16) * ldb + c * 128);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f.lo[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o + (unsigned)(j * ldb), 0, 0));
      f.hi[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o + (unsigned)((j + 8) * ldb), 0, 0));
    }
  }
};

ORBIT_DEV void acc_frag(Frag<float>& f, const f32x16& a, int base) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f.lo[j] = a[base + j];
    f.hi[j] = a[base + 4 + j];
  }
}
template <int N>
ORBIT_DEV void clear(f32x16 (&a)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) a[i][v] = 0.f;
}
// accumulators X^T[feature][position] to stage[position][feature], pitch DH + 4
template <int DH>
ORBIT_DEV void park(float* st, const f32x16 (&a)[DH / 32], int lane) {
  const int g = lane >> 5;
#pragma unroll
  for (int c = 0; c < DH / 32; ++c)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *reinterpret_cast<f32x4*>(st + (lane & 31) * (DH + 4) + c * 32 + r4 * 8 + g * 4) =
          f32x4{a[c][r4 * 4], a[c][r4 * 4 + 1], a[c][r4 * 4 + 2], a[c][r4 * 4 + 3]};
}

template <int DH>
__global__ void __launch_bounds__(256, DH <= 64 ? 2 : 1) attn_f32_fwd(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) float stage[];  // [4][32][DH + 4] | m [4][32] | l [4][32]
  constexpr int SP = 32 * (DH + 4), NC = DH / 32, NK = DH / 16;
  float* sm = stage + 4 * SP;
  float* sl = sm + 128;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, L = a.L, q0 = blockIdx.x * 32;
  const int64_t row0 = (int64_t)b * L;
  Slice<DH> Q, K, V;
  Q.init(a.q + row0 * a.ldq + h * DH, a.ldq, L, lane);
  K.init(a.k + row0 * a.ldk + h * DH, a.ldk, L, lane);
  V.init(a.v + row0 * a.ldv + h * DH, a.ldv, L, lane);
  Frag<float> qf[NK], kf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) Q.row(qf[kk], q0, kk);
  f32x16 o[NC];
  clear(o);
  float m = -INFINITY, lsum = 0.f;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) K.row(kf[kk], wave * 32, kk);
  for (int j0 = wave * 32; j0 < L; j0 += 128) {
    f32x16 s[1];
    clear(s);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) mma16(s[0], kf[kk], qf[kk]);
    // the next tile's keys (zeros past the last) arrive during the rest of this one
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) K.row(kf[kk], j0 + 128, kk);
    // lane: query q0 + lane % 32, keys j0 + 8 (v / 4) + 4 g + v % 4
    float mloc = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if (j0 + (v >> 2) * 8 + g * 4 + (v & 3) >= L) s[0][v] = -INFINITY;
      mloc = fmaxf(mloc, s[0][v]);
    }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float mnew = fmaxf(m, mloc * a.sl2);
    const float mref = mnew == -INFINITY ? 0.f : mnew;  // only logits of -inf so far: they weigh nothing
    const float alpha = __builtin_amdgcn_exp2f(m - mref);
    lsum *= alpha;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] *= alpha;
    m = mnew;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[0][v] = __builtin_amdgcn_exp2f(fmaf(s[0][v], a.sl2, -mref));
      lsum += s[0][v];
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      Frag<float> pf, vf;
      acc_frag(pf, s[0], kk * 8);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        V.col(vf, j0, kk, c);
        mma16(o[c], vf, pf);
      }
    }
  }
  lsum += __shfl_xor(lsum, 32, 64);
  park<DH>(stage + wave * SP, o, lane);
  if (g == 0) {
    sm[wave * 32 + lane] = m;
    sl[wave * 32 + lane] = lsum;
  }
  __syncthreads();
  // 8 threads per query; a wave without tiles has m = -inf and weighs nothing
  const int qr = tid >> 3, qi = q0 + qr;
  if (qi >= L) return;
  float M = sm[qr], w[4], den = 0.f;
#pragma unroll
  for (int i = 1; i < 4; ++i) M = fmaxf(M, sm[i * 32 + qr]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    w[i] = __builtin_amdgcn_exp2f(sm[i * 32 + qr] - M);
    den += w[i] * sl[i * 32 + qr];
  }
  const float inv = 1.f / den;
  float* O = a.o + (row0 + qi) * a.ldo + h * DH;
  float* O32 = a.o32 ? a.o32 + (row0 + qi) * a.ldo32 + h * DH : nullptr;
#pragma unroll
  for (int c = (tid & 7) * 4; c < DH; c += 32) {
    f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) x += w[i] * *reinterpret_cast<const f32x4*>(stage + i * SP + qr * (DH + 4) + c);
    x *= inv;
    *reinterpret_cast<f32x4*>(O + c) = x;
    if (O32) *reinterpret_cast<f32x4*>(O32 + c) = x;
  }
  if ((tid & 7) == 0) a.lse_out[((int64_t)b * a.H + h) * L + qi] = (M + __log2f(den)) * kLn2;
}

// sum of the four waves' stages, in order
template <int DH>
ORBIT_DEV f32x4 sum4(const float* stage, int r, int c) {
  constexpr int SP = 32 * (DH + 4);
  const float* p = stage + r * (DH + 4) + c;
  const f32x4 x0 = *reinterpret_cast<const f32x4*>(p), x1 = *reinterpret_cast<const f32x4*>(p + SP);
  const f32x4 x2 = *reinterpret_cast<const f32x4*>(p + 2 * SP), x3 = *reinterpret_cast<const f32x4*>(p + 3 * SP);
  return (x0 + x1) + (x2 + x3);
}

template <int DH>
__global__ void __launch_bounds__(256, DH <= 64 ? 2 : 1) attn_f32_dq(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) float stage[];  // [4][32][DH + 4]
  constexpr int SP = 32 * (DH + 4), NC = DH / 32, NK = DH / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, L = a.L, q0 = blockIdx.x * 32;
  const int64_t row0 = (int64_t)b * L, bh = (int64_t)b * a.H + h;
  Slice<DH> Q, K, V, G;
  Q.init(a.q + row0 * a.ldq + h * DH, a.ldq, L, lane);
  K.init(a.k + row0 * a.ldk + h * DH, a.ldk, L, lane);
  V.init(a.v + row0 * a.ldv + h * DH, a.ldv, L, lane);
  G.init(a.dO + row0 * a.lddo + h * DH, a.lddo, L, lane);
  Frag<float> qf[NK], of[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    Q.row(qf[kk], q0, kk);
    G.row(of[kk], q0, kk);
  }
  const int qi = q0 + (lane & 31);
  const float lse2 = qi < L ? a.lse[bh * L + qi] * kLog2e : INFINITY;
  const float Dq = qi < L ? a.D[bh * L + qi] : 0.f;
  // dQ_i = sum_j dS_ij (k_j - kbar), since sum_j dS_ij = 0: centred keys keep
  // the product well conditioned when the keys are alike
  float kbar[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) kbar[c] = a.ksum[bh * DH + c * 32 + (lane & 31)] / (float)L;
  f32x16 dq[NC];
  clear(dq);
  for (int j0 = wave * 32; j0 < L; j0 += 128) {
    f32x16 s[2];
    clear(s);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      Frag<float> kf, vf;
      K.row(kf, j0, kk);
      V.row(vf, j0, kk);
      mma16(s[0], kf, qf[kk]);
      mma16(s[1], vf, of[kk]);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const bool in = j0 + (v >> 2) * 8 + g * 4 + (v & 3) < L;
      const float p = in ? __builtin_amdgcn_exp2f(fmaf(s[0][v], a.sl2, -lse2)) : 0.f;
      s[1][v] = p * (s[1][v] - Dq);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      Frag<float> sf, kc;
      acc_frag(sf, s[1], kk * 8);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        K.col(kc, j0, kk, c);
        kc.lo -= kbar[c];
        kc.hi -= kbar[c];
        mma16(dq[c], kc, sf);
      }
    }
  }
  park<DH>(stage + wave * SP, dq, lane);
  __syncthreads();
  const int r = tid >> 3;
  if (q0 + r >= L) return;
  float* dQ = a.dq + (row0 + q0 + r) * a.ldg + h * DH;
#pragma unroll
  for (int c = (tid & 7) * 4; c < DH; c += 32) *reinterpret_cast<f32x4*>(dQ + c) = sum4<DH>(stage, r, c) * a.scale;
}

template <int DH>
__global__ void __launch_bounds__(256, DH <= 64 ? 2 : 1) attn_f32_dkdv(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) float stage[];  // [4][32][DH + 4] | cs [4][32]
  constexpr int SP = 32 * (DH + 4), NC = DH / 32, NK = DH / 16;
  float* scs = stage + 4 * SP;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int h = blockIdx.y, b = blockIdx.z, L = a.L, k0 = blockIdx.x * 32;
  const int64_t row0 = (int64_t)b * L, bh = (int64_t)b * a.H + h;
  Slice<DH> Q, K, V, G;
  Q.init(a.q + row0 * a.ldq + h * DH, a.ldq, L, lane);
  K.init(a.k + row0 * a.ldk + h * DH, a.ldk, L, lane);
  V.init(a.v + row0 * a.ldv + h * DH, a.ldv, L, lane);
  G.init(a.dO + row0 * a.lddo + h * DH, a.lddo, L, lane);
  const __amdgpu_buffer_rsrc_t rl =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.lse + bh * L), 0, L * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rd =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.D + bh * L), 0, L * 4, 0x00020000);
  Frag<float> kf[NK], vf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    K.row(kf[kk], k0, kk);
    V.row(vf[kk], k0, kk);
  }
  float qbar[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) qbar[c] = a.qsum[bh * DH + c * 32 + (lane & 31)] / (float)L;
  // dK_j = sum_i dS_ij (q_i - qbar) + qbar sum_i dS_ij: centred queries, and
  // the rank-one remainder from the column sums cs
  f32x16 dv[NC], dk[NC];
  clear(dv);
  clear(dk);
  float cs = 0.f;
  for (int i0 = wave * 32; i0 < L; i0 += 128) {
    f32x16 s[2];
    clear(s);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      Frag<float> qf, of;
      Q.row(qf, i0, kk);
      G.row(of, i0, kk);
      mma16(s[0], qf, kf[kk]);
      mma16(s[1], of, vf[kk]);
    }
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      // queries i0 + 8 v4 + 4 g .. + 3; column: this lane's key
      const int qr = i0 + v4 * 8 + g * 4;
      const f32x4 le = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rl, (unsigned)qr * 4u, 0, 0));
      const f32x4 dd = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rd, (unsigned)qr * 4u, 0, 0));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = v4 * 4 + u;
        const float p = qr + u < L ? __builtin_amdgcn_exp2f(fmaf(s[0][v], a.sl2, -(le[u] * kLog2e))) : 0.f;
        s[0][v] = p;
        s[1][v] = p * (s[1][v] - dd[u]);
        cs += s[1][v];
      }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      Frag<float> pf, sf, x;
      acc_frag(pf, s[0], kk * 8);
      acc_frag(sf, s[1], kk * 8);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        G.col(x, i0, kk, c);
        mma16(dv[c], x, pf);
        Q.col(x, i0, kk, c);
        x.lo -= qbar[c];
        x.hi -= qbar[c];
        mma16(dk[c], x, sf);
      }
    }
  }
  cs += __shfl_xor(cs, 32, 64);
  if (g == 0) scs[wave * 32 + lane] = cs;
  park<DH>(stage + wave * SP, dv, lane);
  __syncthreads();
  const int r = tid >> 3, kv = k0 + r;
  float* dV = a.dv + (row0 + kv) * a.ldg + h * DH;
  float* dK = a.dk + (row0 + kv) * a.ldg + h * DH;
  if (kv < L)
#pragma unroll
    for (int c = (tid & 7) * 4; c < DH; c += 32) *reinterpret_cast<f32x4*>(dV + c) = sum4<DH>(stage, r, c);
  __syncthreads();
  park<DH>(stage + wave * SP, dk, lane);
  __syncthreads();
  if (kv >= L) return;
  const float ct = (scs[r] + scs[32 + r]) + (scs[64 + r] + scs[96 + r]);
#pragma unroll
  for (int c = (tid & 7) * 4; c < DH; c += 32) {
    const f32x4 qs = *reinterpret_cast<const f32x4*>(a.qsum + bh * DH + c);
    *reinterpret_cast<f32x4*>(dK + c) = (sum4<DH>(stage, r, c) + qs * (ct / (float)L)) * a.scale;
  }
}

template <auto KERN>
orbit_status go(const KernelInfo& k, size_t lds, const AttnF32Args& a, int B, hipStream_t s) {
  static const bool once = [lds] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    return true;
  }();
  (void)once;
  return launch(k, KERN, dim3((unsigned)cdiv(a.L, 32), a.H, B), dim3(256), lds, s, a);
}

template <int DH>
orbit_status fwd(const AttnF32Args& a, int B, hipStream_t s) {
  const double bl = (double)B * a.H * a.L;
  return go<attn_f32_fwd<DH>>(KernelInfo{"attn_f32_fwd", 4.0 * bl * a.L * DH, 16.0 * bl * DH},
                              (4 * 32 * (DH + 4) + 256) * sizeof(float), a, B, s);
}
template <int DH>
orbit_status bwd(const AttnF32Args& a, int B, hipStream_t s) {
  const double bl = (double)B * a.H * a.L;
  ORBIT_TRY(go<attn_f32_dkdv<DH>>(KernelInfo{"attn_f32_dkdv", 4.8 * bl * a.L * DH, 24.0 * bl * DH},
                                  (4 * 32 * (DH + 4) + 128) * sizeof(float), a, B, s));
  return go<attn_f32_dq<DH>>(KernelInfo{"attn_f32_dq", 3.2 * bl * a.L * DH, 20.0 * bl * DH},
                             4 * 32 * (DH + 4) * sizeof(float), a, B, s);
}

}  // namespace

orbit_status attn_f32_forward(const AttnF32Args& a, int B, int dh, hipStream_t s) {
  return dh == 32 ? fwd<32>(a, B, s) : dh == 64 ? fwd<64>(a, B, s) : fwd<128>(a, B, s);
}
orbit_status attn_f32_backward(const AttnF32Args& a, int B, int dh, hipStream_t s) {
  return dh == 32 ? bwd<32>(a, B, s) : dh == 64 ? bwd<64>(a, B, s) : bwd<128>(a, B, s);
}

}  // namespace orbit
