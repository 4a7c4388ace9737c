// float32 products C = alpha * A B (+ epilogue) on bf16 matrix instructions.
//
// The matrix cores run float32 operands at 1/16 of their bf16 rate (157 against
// 2500 TFLOP/s nominal), so a float32 MFMA loop is bound by them. Here every
// operand element is split on its way into LDS into three bf16 parts,
// x = h + m + l (each the remainder so far rounded to nearest), which together
// hold the 24 bits of x, and a product is the sum of the six terms h h', h m',
// m h', m m', h l', l h', accumulated in float32: 6/16 of the float32 MFMA
// time. With |m| <= 2^-8 |x| and |l| <= 2^-17 |x| the dropped terms m l' + l m'
// are at most 2^-24 of the product, half a float32 step (2^-27.5 in the root mean
// square; h cut off instead of rounded: 2^-22 and 2^-25.5). The
// leading term has an accumulator of its own, so the large sum is rounded once
// per 16 k (float32 MFMA: every 2 k); against float64 the results are closer
// than the float32 MFMA's (2048 x 1024 over N(0,1) operands, relative error:
// K = 1024: 1.3e-7 against 2.9e-7; K = 4096: 1.9e-7 against 5.8e-7).
// The split is the triple-bf16 one of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 artificial intelligence datatype for higher-precision computations"
// (ARITH 2019).
//
// Operands are split at 2^16 times their value, so that the last part of the
// smallest float32 numbers is no smaller than the smallest bf16 (unscaled, a
// value below 2^-110 would lose up to 2^-134; the scaling costs 2-4%, finding
// such values while they are split and computing their tile again cost 4-13%).
//
// A tile whose accumulators are not finite is computed again with float32 MFMA:
// an infinity would meet parts that are zero or of the other sign, and values
// from 2^112 or sums from 2^96 on overflow when scaled.
//
// 4 waves per block, a 128x128 or 64x64 tile; 16-deep K slices in two LDS
// buffers (three planes of [row][16] bf16, 48-byte rows: fragment reads are
// free of bank conflicts), one barrier per slice; a slice is split and written
// while the one before it is multiplied, and two more are in flight from
// memory. Two 128x128 blocks share a CU. The matrix cores then do 1.2 PFLOP/s
// of bf16 work, as in the bf16 products: 180-200 TFLOP/s of float32 at 8192
// rows (float32 MFMA: 115-130), and with 1024 rows, N = 4096, K = 1024:
// 61 / 57 / 57 us forward / input / weight gradient against 88 / 85 / 91.
#include <type_traits>

#include "gemm_f32.h"
#include "tile.h"

namespace orbit {
namespace {

constexpr int KD = 16;        // K slice
constexpr int FP = KD + 8;    // plane row pitch (bf16)

constexpr unsigned kOob = 0x80000000u;  // past every num_records: the load returns zeros

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

ORBIT_DEV __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

struct Split4 { uint2 h, m, l; };

ORBIT_DEV uint32_t pk_rn(float lo, float hi) {
  const bf16x2 v = {(bf16)lo, (bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// the operands' scale and the products' way back
constexpr float kUp = 65536.f, kDown = 1.f / (kUp * kUp);

// two floats -> the packed bf16 pairs of the three parts of kUp x
ORBIT_DEV void split2(uint32_t x0, uint32_t x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  float r0 = __uint_as_float(x0) * kUp, r1 = __uint_as_float(x1) * kUp;
  h = pk_rn(r0, r1);
  r0 -= __uint_as_float(h << 16);
  r1 -= __uint_as_float(h & 0xffff0000u);
  m = pk_rn(r0, r1);
  r0 -= __uint_as_float(m << 16);
  r1 -= __uint_as_float(m & 0xffff0000u);
  l = pk_rn(r0, r1);
}
ORBIT_DEV Split4 split4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
  Split4 s;
  split2(x0, x1, s.h.x, s.m.x, s.l.x);
  split2(x2, x3, s.h.y, s.m.y, s.l.y);
  return s;
}

// One operand tile: ROWS x 16 floats loaded into registers, split into three
// LDS planes. Consecutive lanes take consecutive 4-k pieces of one LDS row; an
// M/N-major source is read as blocks of 4 k x 2 rows and transposed in
// registers (64-row tiles have fewer blocks than threads: the caller offsets B's
// thread index, so that the two operands' blocks fall to different waves).
template <int ROWS, bool KMAJ>
struct SplitStage {
  static constexpr int KC = KD / 4;
  static constexpr int NCH = KMAJ ? ROWS * KC : KC * (ROWS / 2);
  static constexpr int PER = (NCH + 255) / 256;
  using V = std::conditional_t<KMAJ, u32x4, u32x2>;
  static constexpr int REGS = KMAJ ? PER : PER * 4;
  static constexpr int PLANE = ROWS * FP;  // elements
  V r[2][REGS];       // two slices in flight
  unsigned voff[PER];
  int kofs[PER];      // K-major: first k of the piece inside a slice

  ORBIT_DEV void init(int64_t ld, int row0, int rlim, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * 256, kc = c % KC, rc = c / KC;
      const int row = KMAJ ? rc : rc * 2;
      const bool ok = c < NCH && row0 + row < rlim;
      kofs[i] = kc * 4;
      voff[i] = !ok ? kOob : KMAJ ? (unsigned)(row * (int)ld + kc * 4) * 4u : (unsigned)(kc * 4 * (int)ld + row) * 4u;
    }
  }
  // slice at k0 of the operand tile whose first row is at X (K-major: X + k,
  // else X + k ld); k >= kend reads zeros
  ORBIT_DEV void load(int st, const float* X, int64_t ld, int k0, int kend) {
    const int left = kend - k0;
    if constexpr (KMAJ) {
      const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(X + k0, left > 0 ? 0x7fffffff : 0);
#pragma unroll
      for (int i = 0; i < PER; ++i)
        r[st][i] = __builtin_amdgcn_raw_buffer_load_b128(rs, kofs[i] < left ? voff[i] : kOob, 0, 0);
    } else {
      const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(X + (int64_t)k0 * ld, left > 0 ? min(left, KD) * (int)ld * 4 : 0);
#pragma unroll
      for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          r[st][i * 4 + j] = __builtin_amdgcn_raw_buffer_load_b64(rs, voff[i] + (unsigned)(j * (int)ld * 4), 0, 0);
    }
  }
  static ORBIT_DEV void put(bf16* S, int row, int kc, const Split4& s) {
    bf16* p = S + row * FP + kc * 4;
    *reinterpret_cast<uint2*>(p) = s.h;
    *reinterpret_cast<uint2*>(p + PLANE) = s.m;
    *reinterpret_cast<uint2*>(p + 2 * PLANE) = s.l;
  }
  ORBIT_DEV void store(int st, bf16* S, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * 256, kc = c % KC, rc = c / KC;
      if (NCH % 256 != 0 && c >= NCH) continue;
      if constexpr (KMAJ) {
        put(S, rc, kc, split4(r[st][i][0], r[st][i][1], r[st][i][2], r[st][i][3]));
      } else {
#pragma unroll
        for (int e = 0; e < 2; ++e)
          put(S, rc * 2 + e, kc, split4(r[st][i * 4][e], r[st][i * 4 + 1][e], r[st][i * 4 + 2][e], r[st][i * 4 + 3][e]));
      }
    }
  }
  static ORBIT_DEV bf16x8 frag(const bf16* S, int plane, int row0, int lane) {
    return *reinterpret_cast<const bf16x8*>(S + plane * PLANE + (row0 + (lane & 31)) * FP + (lane >> 5) * 8);
  }
};

// Both operands M/N-major (weight gradients): waves 0 and 1 stage A, waves 2
// and 3 B, in blocks of 4 k x 4 rows, so every thread has one block of
// one operand (16-byte loads; against 2-row blocks of both operands in
// every thread 4096x1024x8192 went from 468 to 350 us).
struct SplitDual {
  static constexpr int RW = 4, KC = KD / 4;
  static constexpr int PLANE = SplitStage<128, false>::PLANE;
  u32x4 r[2][4];
  unsigned voff;
  int ldb;             // bytes per k
  const float* X;
  int lds_off;

  ORBIT_DEV void init(const float* A, int64_t lda, int m0, int M, const float* B, int64_t ldb_, int n0, int N,
                      int wave, int lane) {
    const bool isb = wave >= 2;
    const int64_t ld = isb ? ldb_ : lda;
    X = isb ? B : A;
    ldb = (int)ld * 4;
    const int c = (wave & 1) * 64 + lane, kc = c % KC, row = (c / KC) * RW;
    const int left = isb ? N - n0 : M - m0;
    voff = row < left ? (unsigned)(kc * 4) * (unsigned)ldb + (unsigned)row * 4u : kOob;
    lds_off = (isb ? 3 * PLANE : 0) + row * FP + kc * 4;
  }
  ORBIT_DEV void load(int st, int k0, int kend) {
    const int left = kend - k0;
    const __amdgpu_buffer_rsrc_t rs =
        buffer_rsrc(reinterpret_cast<const char*>(X) + (int64_t)k0 * ldb, left > 0 ? min(left, KD) * ldb : 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[st][j] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + (unsigned)(j * ldb), 0, 0);
  }
  ORBIT_DEV void store(int st, bf16* S) const {
#pragma unroll
    for (int e = 0; e < RW; ++e) {
      const Split4 s = split4(r[st][0][e], r[st][1][e], r[st][2][e], r[st][3][e]);
      bf16* p = S + lds_off + e * FP;
      *reinterpret_cast<uint2*>(p) = s.h;
      *reinterpret_cast<uint2*>(p + PLANE) = s.m;
      *reinterpret_cast<uint2*>(p + 2 * PLANE) = s.l;
    }
  }
};

template <int BT, bool AK, bool BKM>
__global__ void __launch_bounds__(256, 2) gemm_f32_kernel(GemmKArgs g) {
  constexpr int WT = BT / 2, TW = WT / 32;  // wave tile
  using SA = SplitStage<BT, AK>;
  using SB = SplitStage<BT, BKM>;
  constexpr int BUF = 3 * (SA::PLANE + SB::PLANE);  // elements
  extern __shared__ __attribute__((aligned(16))) char smem[];
  bf16* lds = reinterpret_cast<bf16*>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tidb = tid ^ 128;
  const int wm = wave % 2, wn = wave / 2;
  const int split = blockIdx.z % g.splits;
  const int64_t bz = blockIdx.z / g.splits;

  // tile order: each XCD a contiguous range of tiles, walked in groups of 8 tile rows
  const int tiles_n = (g.N + BT - 1) / BT, tiles_m = (g.M + BT - 1) / BT;
  const int nt = tiles_m * tiles_n;
  int id = blockIdx.x;
  const int full = nt - nt % 8;
  if (id < full) id = (id % 8) * (full / 8) + id / 8;
  const int per_group = 8 * tiles_n;
  const int first_m = (id / per_group) * 8;
  const int gsize = min(tiles_m - first_m, 8);
  const int m0 = (first_m + (id % per_group) % gsize) * BT, n0 = ((id % per_group) / gsize) * BT;

  const float* A = static_cast<const float*>(g.A) + bz * g.sA;
  const float* B = static_cast<const float*>(g.B) + bz * g.sB;
  const int kbeg = split * g.k_per_split, kend = min(g.K, kbeg + g.k_per_split);
  const int nk = (kend - kbeg + KD - 1) / KD;

  // the leading term and the five small ones are summed apart: the large sum
  // is then rounded once per 16 k
  f32x16 acc[TW][TW], accs[TW][TW];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int j = 0; j < TW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = accs[i][j][v] = 0.f;
  };
  clear();
  {
    constexpr bool DUAL = !AK && !BKM;
    static_assert(!DUAL || BT == 128, "weight gradients have 128x128 tiles only");
    SA la;
    SB lb;
    SplitDual lab;
    const float* At = A + (AK ? (int64_t)m0 * g.lda : m0);
    const float* Bt = B + (BKM ? (int64_t)n0 * g.ldb : n0);
    if constexpr (DUAL) {
      lab.init(At, g.lda, m0, g.M, Bt, g.ldb, n0, g.N, __builtin_amdgcn_readfirstlane(wave), lane);
    } else {
      la.init(g.lda, m0, g.M, tid);
      lb.init(g.ldb, n0, g.N, tidb);
    }
    auto load = [&](int st, int kt) {
      if constexpr (DUAL) {
        lab.load(st, kbeg + kt * KD, kend);
      } else {
        la.load(st, At, g.lda, kbeg + kt * KD, kend);
        lb.load(st, Bt, g.ldb, kbeg + kt * KD, kend);
      }
    };
    auto store = [&](int st, int kt) {
      bf16* p = lds + (kt & 1) * BUF;
      if constexpr (DUAL) {
        lab.store(st, p);
      } else {
        la.store(st, p, tid);
        lb.store(st, p + 3 * SA::PLANE, tidb);
      }
    };
    // slices past the last one load zeros (k >= kend)
    load(0, 0);
    load(1, 1);
    store(0, 0);
    load(0, 2);
    __syncthreads();
    auto step = [&](int st, int kt) {
      const bf16* As = lds + (kt & 1) * BUF;
      const bf16* Bs = As + 3 * SA::PLANE;
      bf16x8 af[3][TW], bf[3][TW];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < TW; ++i) {
          af[p][i] = SA::frag(As, p, wm * WT + i * 32, lane);
          bf[p][i] = SB::frag(Bs, p, wn * WT + i * 32, lane);
        }
      // the next slice is split and written during this one's products
      store(st, kt + 1);
      load(st, kt + 3);
      constexpr int TA[5] = {2, 0, 1, 1, 0}, TB[5] = {0, 2, 1, 0, 1};
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[0][i], bf[0][j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int j = 0; j < TW; ++j)
            accs[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[TA[t]][i], bf[TB[t]][j], accs[i][j], 0, 0, 0);
      __syncthreads();
    };
    for (int kt = 0; kt < nk; kt += 2) {
      step(1, kt);
      if (kt + 1 < nk) step(0, kt + 1);
    }
  }
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = (acc[i][j] + accs[i][j]) * kDown;
  float probe = 0.f;
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) probe = fmaf(acc[i][j][v], 0.f, probe);
  if (__syncthreads_or(!(probe == 0.f))) {
    // an infinity or a NaN: again with float32 MFMA
    constexpr int FD = 32;
    using FA = GemmStage<float, BT, FD, 256, AK>;
    using FB = GemmStage<float, BT, FD, 256, BKM>;
    float* Af = reinterpret_cast<float*>(smem);
    float* Bf = Af + FA::SIZE;
    static_assert((FA::SIZE + FB::SIZE) * 4 <= 2 * BUF * 2, "the float32 stages fit the planes");
    clear();
#pragma unroll 1
    for (int k0 = kbeg; k0 < kend; k0 += FD) {
      FA la;
      FB lb;
      la.load(A, nullptr, 0, g.lda, m0, g.M, k0, kend, tid);
      lb.load(B, nullptr, 0, g.ldb, n0, g.N, k0, kend, tid);
      la.store(Af, tid);
      lb.store(Bf, tid);
      __syncthreads();
#pragma unroll 1
      for (int kk = 0; kk < FD / 16; ++kk) {
        Frag<float> af[TW], bf[TW];
#pragma unroll
        for (int i = 0; i < TW; ++i) {
          FA::frag(af[i], Af, wm * WT + i * 32, kk, lane);
          FB::frag(bf[i], Bf, wn * WT + i * 32, kk, lane);
        }
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int j = 0; j < TW; ++j) mma16(acc[i][j], af[i], bf[j]);
      }
      __syncthreads();
    }
  }

  // epilogue through LDS: each wave parks 32 rows of its accumulators in a
  // private region and reads them back as 8 consecutive columns per lane
  constexpr int EP = WT + 8, LPR = WT / 8, RPI = 64 / LPR;
  static_assert(4 * 32 * EP * 4 <= 2 * BUF * 2, "epilogue fits the planes");
  float* ew = reinterpret_cast<float*>(smem) + wave * 32 * EP;
  float* C = static_cast<float*>(g.C) + bz * g.sC;
  const bool raw = g.splits > 1;
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int j = 0; j < TW; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        ew[((v >> 2) * 8 + (lane >> 5) * 4 + (v & 3)) * EP + j * 32 + (lane & 31)] = acc[i][j][v];
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < 32 / RPI; ++it) {
      const int rl = it * RPI + lane / LPR, cl = (lane % LPR) * 8;
      const int r = m0 + wm * WT + i * 32 + rl, c0 = n0 + wn * WT + cl;
      float v8[8];
      ld8(ew + rl * EP + cl, v8);
      if (r < g.M && c0 < g.N) {
        if (raw) {
          float* P = g.partial + (((int64_t)split * g.batch + bz) * g.M + r) * g.N;
          if (g.vec_ok) {
            st8(P + c0, v8);
          } else {
            for (int q = 0; q < 8 && c0 + q < g.N; ++q) P[c0 + q] = v8[q];
          }
        } else if (g.vec_ok) {
          epi_apply8<float, float>(g.epi, bz, r, c0, v8, C, g.ldc);
        } else {
          for (int q = 0; q < 8 && c0 + q < g.N; ++q) epi_apply<float, float>(g.epi, bz, r, c0 + q, v8[q], C, g.ldc);
        }
      }
    }
    __syncthreads();
  }
}

// Small products: a block per 32x32 tile, its four waves on every fourth
// 16-deep K slice, operands straight from global memory into float32 MFMA
// fragments (no LDS, no barrier until the waves' sums are added in order), four
// slices of loads in flight. What bounds these calls is latency: larger tiles
// leave most CUs idle and walk K one barrier at a time (256 x 128, K = 512:
// 10 us against 19 on 64x64 tiles and 13.5 with K split in four, launch
// included).
template <bool KMAJ>
struct TinyOperand {
  __amdgpu_buffer_rsrc_t rs;
  unsigned voff;
  int ldb, kl;
  // tile rows from X; the lane's row is lane % 32, its k 8 (lane / 32) .. + 7 of a slice
  ORBIT_DEV void init(const float* X, int64_t ld, int rows_left, int kend, int lane) {
    const int row = lane & 31;
    kl = (lane >> 5) * 8;
    ldb = (int)ld * 4;
    rs = buffer_rsrc(X, KMAJ ? 0x7fffffff : kend * ldb);
    voff = row >= rows_left ? kOob : KMAJ ? (unsigned)(row * ldb + kl * 4) : (unsigned)(kl * ldb + row * 4);
  }
  ORBIT_DEV void load(Frag<float>& f, int k0, int kend) const {
    if constexpr (KMAJ) {
      const unsigned o = voff + (unsigned)k0 * 4u;
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rs, k0 + kl < kend ? o : kOob, 0, 0);
      const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rs, k0 + kl + 4 < kend ? o + 16u : kOob, 0, 0);
      f.lo = __builtin_bit_cast(f32x4, a);
      f.hi = __builtin_bit_cast(f32x4, b);
    } else {
      const unsigned o = voff + (unsigned)(k0 * ldb);  // rows at and past kend are out of range
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f.lo[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o + (unsigned)(j * ldb), 0, 0));
        f.hi[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o + (unsigned)((j + 4) * ldb), 0, 0));
      }
    }
  }
};

template <bool AK, bool BKM>
__global__ void __launch_bounds__(256) gemm_f32_tiny(GemmKArgs g) {
  __shared__ __attribute__((aligned(16))) float part[4][32][36];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles_n = (g.N + 31) / 32;
  const int m0 = ((int)blockIdx.x / tiles_n) * 32, n0 = ((int)blockIdx.x % tiles_n) * 32;
  const int64_t bz = blockIdx.z;
  const float* A = static_cast<const float*>(g.A) + bz * g.sA + (AK ? (int64_t)m0 * g.lda : m0);
  const float* B = static_cast<const float*>(g.B) + bz * g.sB + (BKM ? (int64_t)n0 * g.ldb : n0);
  TinyOperand<AK> oa;
  TinyOperand<BKM> ob;
  oa.init(A, g.lda, g.M - m0, g.K, lane);
  ob.init(B, g.ldb, g.N - n0, g.K, lane);
  // one accumulator per load slot: each sums every sixteenth slice
  f32x16 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[u][v] = 0.f;
  for (int k0 = wave * 16; k0 < g.K; k0 += 256) {
    Frag<float> fa[4], fb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      oa.load(fa[u], k0 + u * 64, g.K);
      ob.load(fb[u], k0 + u * 64, g.K);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k0 + u * 64 < g.K) mma16(acc[u], fa[u], fb[u]);
  }
  acc[0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
  for (int v = 0; v < 16; ++v) part[wave][(v >> 2) * 8 + (lane >> 5) * 4 + (v & 3)][lane & 31] = acc[0][v];
  __syncthreads();
  if (tid >= 128) return;
  const int rl = tid >> 2, cl = (tid & 3) * 8, r = m0 + rl, c0 = n0 + cl;
  if (r >= g.M || c0 >= g.N) return;
  float v8[8], t8[8];
  ld8(&part[0][rl][cl], v8);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    ld8(&part[w][rl][cl], t8);
#pragma unroll
    for (int q = 0; q < 8; ++q) v8[q] += t8[q];
  }
  float* C = static_cast<float*>(g.C) + bz * g.sC;
  if (g.vec_ok) {
    epi_apply8<float, float>(g.epi, bz, r, c0, v8, C, g.ldc);
  } else {
    for (int q = 0; q < 8 && c0 + q < g.N; ++q) epi_apply<float, float>(g.epi, bz, r, c0 + q, v8[q], C, g.ldc);
  }
}

template <bool AK, bool BKM>
orbit_status run_tiny(const GemmKArgs& a, hipStream_t s) {
  KernelInfo k{"gemm_f32_tiny", 2.0 * a.M * a.N * (double)a.K * a.batch,
               ((double)a.M * a.K + (double)a.K * a.N + (double)a.M * a.N) * 4.0 * a.batch};
  const dim3 grid((unsigned)(cdiv(a.N, 32) * cdiv(a.M, 32)), 1, (unsigned)a.batch);
  return launch(k, gemm_f32_tiny<AK, BKM>, grid, dim3(256), 0, s, a);
}

template <int BT, bool AK, bool BKM>
orbit_status run(const GemmKArgs& a, hipStream_t s) {
  constexpr size_t lds = 12 * (size_t)SplitStage<BT, true>::PLANE * 2;
  static const bool once = [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_f32_kernel<BT, AK, BKM>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    return true;
  }();
  (void)once;
  static const char* names[2] = {"gemm_f32<64>", "gemm_f32<128>"};
  KernelInfo k{names[BT == 128], 2.0 * a.M * a.N * (double)a.K * a.batch,
               ((double)a.M * a.K + (double)a.K * a.N + (double)a.M * a.N) * 4.0 * a.batch};
  const dim3 grid((unsigned)(cdiv(a.N, BT) * cdiv(a.M, BT)), 1, (unsigned)(a.batch * a.splits));
  return launch(k, gemm_f32_kernel<BT, AK, BKM>, grid, dim3(256), lds, s, a);
}

template <int BT>
orbit_status run_layout(bool ak, bool bk, const GemmKArgs& a, hipStream_t s) {
  if constexpr (BT == 128) {
    if (!ak) return run<BT, false, false>(a, s);
  }
  return bk ? run<BT, true, true>(a, s) : run<BT, true, false>(a, s);
}

}  // namespace

orbit_status gemm_f32_launch(int tile, bool a_kmajor, bool b_kmajor, const GemmKArgs& a, hipStream_t s) {
  if (tile == 32) {
    if (a_kmajor) return b_kmajor ? run_tiny<true, true>(a, s) : run_tiny<true, false>(a, s);
    return run_tiny<false, false>(a, s);
  }
  return tile == 128 ? run_layout<128>(a_kmajor, b_kmajor, a, s) : run_layout<64>(a_kmajor, b_kmajor, a, s);
}

}  // namespace orbit
