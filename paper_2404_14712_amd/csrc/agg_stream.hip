// Variable aggregation with the patch-coupling steps inside one kernel per
// direction (bf16).
//
// What bounds these kernels is HBM: the token tensor is the largest of the
// path, and the general path reads it twice forward (scores, xbar) and twice
// backward (dA, dU) besides writing its gradient. Here a block owns whole
// patches and keeps what couples the passes (running softmax, xbar and dU
// accumulators, the folded keys and dxbar as MFMA fragments) in registers, so
// a row of tokens comes from HBM once per direction:
//
//   forward:  S = X U^T, online softmax over the variables, xbar += P^T X
//   backward: dA = X dxbar^T, c = sum_v a_v dA_v,
//             then dS = a (dA - c) scale, dtok = [a | dS][dxbar; U], dU += dS^T X
//
// c couples the rows of a patch, so the backward sweeps a patch twice: its
// second reads (in reverse, the last slot still being in LDS) come from the
// caches. c has to be the sum of the very dA it is subtracted from: what the
// variables of a patch have in common is the same large number in every dA_v
// and in c, and the softmax does not see it. A c known before the sweep (the
// value outputs' product v_h . dzh_h, whose rounding is not that of dxbar) costs
// 15 us less on the first shape below but leaves 2^-9 of the common part in
// dtok: with a common part of 16 times the tokens' spread its largest error was
// 2e-2 to 7e-2 of the largest element, with 256 times up to 1.1 (now 8e-3).
//
// Eight waves share a block; wave w owns columns [w CPW, (w + 1) CPW) of every
// row. Rows arrive in slots of 16 variables x DP = 8 CPW columns, copied by the
// buffer unit straight into an NS-deep LDS ring (64 to 144 KB). A slot is read
// from LDS as row fragments (scores, dA: the reduction runs over the columns,
// wave sums are added in order through LDS) and through transposing reads
// (xbar, dU: the reduction runs over the variables). Copies are non-temporal
// but for the rows that the backward reads again (all of them non-temporal:
// 720 against 626 us for the first shape's whole backward; all of them plain:
// 1-5% slower on five of six large shapes). The 16-byte chunk index of a row is
// XORed with f(r) = 4 (r mod 4) + (r / 4) mod 4, a permutation of 0..15 whose
// four consecutive rows land 64 bytes apart, so both reads are free of bank
// conflicts. Slots of 8 rows (twice as many in flight) were slower everywhere
// (forward 153 against 130 us at d = 2048: the exchange of the wave sums, a
// fixed cost per slot, then bounds it); at DP = 512 two blocks per CU with four
// slots each hide that cost (forward 114 -> 100 us against one with eight).
//
// Measured on MI355X, kernels of the general path -> these:
//   8192 patches x 48 variables x 1024, 16 heads: forward (scores + softmax +
//   xbar) 427 -> 198 us (5.6 TB/s), backward (dA + softmax + dU + dtok)
//   680 -> 357 us (5.3 TB/s);
//   1770 x 67 x 2048, 16 heads: 248 -> 124 us (4.9), 402 -> 254 us (4.3 TB/s:
//   two slots of 64 KB leave little in flight).
#include <algorithm>

#include "agg_stream.h"
#include "tile.h"

namespace orbit {
namespace {

#define ORBIT_LDS __attribute__((address_space(3)))

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr unsigned kOob = 0x80000000u;  // past every num_records: loads read zeros, stores are dropped
constexpr int kThreads = 512;
constexpr int kMaxV = 128;              // each of 8 waves keeps the scores of one 16-row slot
constexpr int kMaxD = 2048;

constexpr int R = 16;                   // rows per slot: 16 variables, or the heads of a [16, DP] matrix

// CPW columns per wave, NS slots, BPC blocks per CU
template <int CPW_, int NS_, int BPC_>
struct StreamCfg {
  static constexpr int CPW = CPW_, NS = NS_, BPC = BPC_;
  static constexpr int DP = 8 * CPW, ROWB = DP * 2, SLOT = R * ROWB;
  static constexpr int NLD = SLOT / 8192;            // 1 KB copies per wave and slot
  static constexpr int KS = CPW / 32, TILES = CPW / 16;
  static_assert(SLOT % 8192 == 0 && CPW % 32 == 0 && DP % 128 == 0, "slot shape");
};

ORBIT_DEV int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

ORBIT_DEV __amdgpu_buffer_rsrc_t rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

ORBIT_DEV void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// wait until at most base + cnt * step vector memory operations are in flight
// (cnt above 3 waits as for 3, which is only stricter)
template <int BASE, int STEP>
ORBIT_DEV void wait_counted(int cnt) {
  static_assert(BASE + 3 * STEP <= 63, "vmcnt has 6 bits");
  if (cnt == 0) wait_vmcnt<BASE>();
  else if (cnt == 1) wait_vmcnt<BASE + STEP>();
  else if (cnt == 2) wait_vmcnt<BASE + 2 * STEP>();
  else wait_vmcnt<BASE + 3 * STEP>();
}

// per-lane source offsets of a wave's copies of one slot
template <typename C>
struct SlotCopy {
  unsigned voff[C::NLD];
  ORBIT_DEV void init(int d, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < C::NLD; ++j) {
      const int byte = (wave * C::NLD + j) * 1024 + lane * 16;
      const int r = byte / C::ROWB, p = (byte % C::ROWB) / 16;
      const int col = (p ^ swz(r)) * 8;
      voff[j] = col < d ? (unsigned)(r * d + col) * 2u : kOob;
    }
  }
  // rows row0.. of the matrix at `base` (`bytes` long; rows past it read zeros)
  template <bool NT>
  ORBIT_DEV void issue(const void* base, int bytes, unsigned row_off, unsigned lds, int wave) const {
    const __amdgpu_buffer_rsrc_t rs = rsrc(base, bytes);
#pragma unroll
    for (int j = 0; j < C::NLD; ++j) {
      if constexpr (NT) dma16nt(rs, lds + (wave * C::NLD + j) * 1024, voff[j] + row_off);
      else dma16(rs, lds + (wave * C::NLD + j) * 1024, voff[j] + row_off);
    }
  }
};

// LDS byte offsets inside a slot of a wave's fragment reads. Steps 4 apart (128
// columns, 256 bytes) share the swizzled low bits, so four bases suffice.
template <typename C>
struct SlotFrag {
  int row[4];  // row fragments: row lane % 16, columns 32 ks + 8 (lane / 16)
  int tr[4];   // transposing reads: rows 4 (lane / 16) + (lane % 16) / 4, columns 32 p + 8 (lane % 4)
  ORBIT_DEV void init(int wave, int lane) {
    const int g = lane >> 4, q = lane & 15;
    const int r0 = q, r1 = 4 * g + (q >> 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k4 = (wave * C::CPW >> 3) + 4 * i;
      row[i] = r0 * C::ROWB + ((k4 | g) ^ swz(r0)) * 16;
      tr[i] = r1 * C::ROWB + ((k4 | (q & 3)) ^ swz(r1)) * 16;
    }
  }
  ORBIT_DEV bf16x8 read_row(const char* slot, int ks) const {
    return *reinterpret_cast<const bf16x8*>(slot + row[ks & 3] + (ks >> 2) * 256);
  }
  // lane l receives column 32 p + 8 (i / 4) + 4 half + i % 4 (i = l % 16) of rows 4 (l / 16) .. + 3
  ORBIT_DEV s16x4 read_tr(const char* slot, int p, int half) const {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (ORBIT_LDS s16x4*)(slot + tr[p & 3] + (p >> 2) * 256 + 8 * half));
  }
};

ORBIT_DEV f32x4 mma32(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
ORBIT_DEV f32x4 mma16x(s16x4 a, s16x4 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }

ORBIT_DEV unsigned pack2(float lo, float hi) {
  const bf16x2 v = {(bf16)lo, (bf16)hi};
  return __builtin_bit_cast(unsigned, v);
}

// x = take ? n : x, kept where it is written: left to itself the compiler sinks
// the selects of all of a patch's fragments behind their reads and then copies
// the old and the new set every iteration
ORBIT_DEV void select_in_place(bf16x8& x, bf16x8 n, bool take) {
  u32x4 a = __builtin_bit_cast(u32x4, x);
  const u32x4 b = __builtin_bit_cast(u32x4, n);
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = take ? b[i] : a[i];
  asm volatile("" : "+v"(a));
  x = __builtin_bit_cast(bf16x8, a);
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
template <typename C>
__global__ void __launch_bounds__(kThreads, 2 * C::BPC) agg_stream_fwd_kernel(const bf16* __restrict__ tok,
                                                                  const bf16* __restrict__ Ut,
                                                                  float* __restrict__ a32, bf16* __restrict__ xbar,
                                                                  int T, int V, int d, int H, float scale_log2) {
  constexpr int NS = C::NS, KS = C::KS;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, q = lane & 15;  // q: the lane's head in scores, weights and xbar
  char* part = smem + NS * C::SLOT;        // wave partials of the scores, two buffers of 8 KB
  const unsigned lds0 = (unsigned)(uintptr_t)(ORBIT_LDS void*)smem;

  // folded keys as MFMA operands: head q, columns wave CPW + 32 ks + 8 g
  bf16x8 uf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int col = wave * C::CPW + ks * 32 + g * 8;
    U128 u = zero128();
    if (q < H && col < d) u = ld128(Ut + (int64_t)q * d + col);
    uf[ks] = __builtin_bit_cast(bf16x8, u);
  }
  SlotCopy<C> cp;
  SlotFrag<C> fr;
  cp.init(d, wave, lane);
  fr.init(wave, lane);

  const int nch = (V + R - 1) / R;
  const int npatch = (T - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int total = npatch * nch;
  // next slot to copy: patch it_t, chunk it_c; past the last one the copies
  // read nothing (every wave issues the same number of operations per slot)
  int it_t = blockIdx.x, it_c = 0, it_n = 0;
  auto issue = [&]() {
    const bool live = it_n < total;
    cp.template issue<true>(tok + (live ? (int64_t)it_t * V * d : 0), live ? V * d * 2 : 0, (unsigned)(it_c * R * d) * 2u,
                            lds0 + (it_n % NS) * C::SLOT, wave);
    ++it_n;
    if (++it_c == nch) { it_c = 0; it_t += gridDim.x; }
  };
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue();

  f32x4 acc[C::TILES];
  f32x4 sk;  // scores of the chunk this wave writes the weights of
  float m = -INFINITY, l32 = 0.f, lb = 0.f;
#pragma unroll
  for (int i = 0; i < C::TILES; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  sk = acc[0];

  constexpr int kStores = C::KS + 4;  // per wave at a patch's end
  unsigned hist = 0;                  // patch ends among the last NS - 1 iterations
  int t = blockIdx.x, c = 0;
  for (int it = 0; it < total; ++it) {
    wait_counted<(NS - 2) * C::NLD, kStores>(__builtin_popcount(hist));
    lds_barrier();
    issue();  // into the slot of iteration it - 1, which every wave has left
    const char* slot = smem + (it % NS) * C::SLOT;
    // S^T [variable, head] of this wave's columns
    f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s4 = mma32(fr.read_row(slot, ks), uf[ks], s4);
    char* pb = part + (it & 1) * 8192;
    *reinterpret_cast<f32x4*>(pb + wave * 1024 + lane * 16) = s4;
    lds_barrier();
    s4 = *reinterpret_cast<const f32x4*>(pb + lane * 16);
#pragma unroll
    for (int w = 1; w < 8; ++w) s4 += *reinterpret_cast<const f32x4*>(pb + w * 1024 + lane * 16);
    // online softmax (log2 units); lane: head q, variables c R + 4 g .. + 3
    float cm = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = c * R + 4 * g + r < V;
      s4[r] = ok ? s4[r] * scale_log2 : -INFINITY;
      cm = fmaxf(cm, s4[r]);
    }
    cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
    cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
    const float mn = fmaxf(m, cm);
    const float mr = mn == -INFINITY ? 0.f : mn;  // only scores of -inf so far: they weigh nothing
    const float al = __builtin_amdgcn_exp2f(m - mr);
    if (c == wave) sk = s4;
    float p[4], ps = 0.f, pbs = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(s4[r] - mr);
      ps += p[r];
    }
    u32x2 pw;
    pw[0] = pack2(p[0], p[1]);
    pw[1] = pack2(p[2], p[3]);
    pbs = (__uint_as_float(pw[0] << 16) + __uint_as_float(pw[0] & 0xffff0000u)) +
          (__uint_as_float(pw[1] << 16) + __uint_as_float(pw[1] & 0xffff0000u));
    l32 = l32 * al + ps;
    lb = lb * al + pbs;
    m = mn;
    if (c > 0 && __builtin_amdgcn_ballot_w64(al != 1.f) != 0) {
#pragma unroll
      for (int i = 0; i < C::TILES; ++i) acc[i] *= al;
    }
    // xbar^T [column, head] += X^T P
    const s16x4 pf = __builtin_bit_cast(s16x4, pw);
#pragma unroll
    for (int i = 0; i < C::TILES; ++i) {
      acc[i] = mma16x(fr.read_tr(slot, i >> 1, i & 1), pf, acc[i]);
    }
    hist = (hist << 1) & ((1u << (NS - 1)) - 1);
    if (++c == nch) {
      l32 += __shfl_xor(l32, 16, 64);
      l32 += __shfl_xor(l32, 32, 64);
      lb += __shfl_xor(lb, 16, 64);
      lb += __shfl_xor(lb, 32, 64);
      const float inv = 1.f / l32, invb = 1.f / lb;
      const __amdgpu_buffer_rsrc_t rx = rsrc(xbar + (int64_t)t * H * d, H * d * 2);
#pragma unroll
      for (int p2 = 0; p2 < KS; ++p2) {
        const int col = wave * C::CPW + p2 * 32 + g * 8;
        const f32x4 a0 = acc[2 * p2] * invb, a1 = acc[2 * p2 + 1] * invb;
        const u32x4 o = {pack2(a0[0], a0[1]), pack2(a0[2], a0[3]), pack2(a1[0], a1[1]), pack2(a1[2], a1[3])};
        __builtin_amdgcn_raw_buffer_store_b128(o, rx, q < H && col < d ? (unsigned)(q * d + col) * 2u : kOob, 0, 0);
      }
      // the weights, [T, V, H]: wave w writes chunk w
      const __amdgpu_buffer_rsrc_t ra = rsrc(a32 + (int64_t)t * V * H, V * H * 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v = wave * R + 4 * g + r;
        const float a = __builtin_amdgcn_exp2f(sk[r] - m) * inv;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a), ra, q < H ? (unsigned)(v * H + q) * 4u : kOob, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < C::TILES; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      m = -INFINITY;
      l32 = lb = 0.f;
      c = 0;
      t += gridDim.x;
      hist |= 1u;
    }
  }
  wait_vmcnt<0>();
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
template <typename C>
__global__ void __launch_bounds__(kThreads, 2 * C::BPC) agg_stream_bwd_kernel(
    const bf16* __restrict__ tok, const bf16* __restrict__ dxbar, const bf16* __restrict__ Ut,
    const float* __restrict__ a32, bf16* __restrict__ dtok, float* __restrict__ dupart, int T, int V, int d, int H,
    float scale) {
  constexpr int NS = C::NS, KS = C::KS;
  constexpr int SP = 20;                   // pitch (bf16) of dS^T
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, q = lane & 15;
  char* aring = smem + NS * C::SLOT;       // per slot 1 KB: the rows' weights
  char* part = aring + NS * 1024;          // 8 KB wave partials of dA
  bf16* ads = reinterpret_cast<bf16*>(part + 8192);   // [2][16 variables][a (16 heads) | dS (16 heads)], swizzled
  bf16* dst = ads + 2 * 16 * 32;                      // dS^T [2][16 heads][16 variables]
  float* red = reinterpret_cast<float*>(dst + 2 * 16 * SP);  // [8][16] chunk sums of a dA
  const unsigned lds0 = (unsigned)(uintptr_t)(ORBIT_LDS void*)smem;
  const unsigned lds_a = lds0 + NS * C::SLOT;

  SlotCopy<C> cp;
  SlotFrag<C> fr;
  cp.init(d, wave, lane);
  fr.init(wave, lane);

  const int nch = (V + R - 1) / R;
  // a patch's slots: dxbar, its chunks of 16 rows (dA), then all but the last
  // of them again in reverse (dS, dtok, dU: the last one is still there); the
  // block's first slot holds U
  const int per = 2 * nch;
  const int npatch = (T - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int total = 1 + npatch * per;
  int it_t = (int)blockIdx.x - (int)gridDim.x, it_k = per - 1;  // U counts as the tail of a patch before the first
  int it_n = 0, it_s = 0;  // slots copied so far, ring position of the next
  auto issue = [&]() {
    const bool live = it_n < total;
    const void* base = tok;
    int bytes = 0, row0 = 0;
    const void* abase = a32;
    int abytes = 0;
    unsigned aoff = 0;
    if (live) {
      if (it_n == 0) {
        base = Ut; bytes = H * d * 2;
      } else if (it_k == 0) {
        base = dxbar + (int64_t)it_t * H * d; bytes = H * d * 2;
      } else {
        base = tok + (int64_t)it_t * V * d; bytes = V * d * 2;
        row0 = (it_k <= nch ? it_k - 1 : 2 * nch - 1 - it_k) * R;
        if (it_k <= nch) {
          abase = a32 + (int64_t)it_t * V * H; abytes = V * H * 4; aoff = (unsigned)(row0 * H) * 4u;
        }
      }
    }
    // rows that come back for the second sweep stay in the caches
    if (it_k == 0 || it_k >= nch) cp.template issue<true>(base, bytes, (unsigned)(row0 * d) * 2u, lds0 + it_s * C::SLOT, wave);
    else cp.template issue<false>(base, bytes, (unsigned)(row0 * d) * 2u, lds0 + it_s * C::SLOT, wave);
    if (wave == 7) dma16(rsrc(abase, abytes), lds_a + it_s * 1024, lane * 16 < R * H * 4 ? (unsigned)lane * 16u + aoff : kOob);
    ++it_n;
    if (++it_s == NS) it_s = 0;
    if (++it_k == per) { it_k = 0; it_t += gridDim.x; }
  };
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue();

  bf16x8 dxf[KS];            // dxbar: head q, columns 32 ks + 8 g
  bf16x8 duf[C::TILES];      // [dxbar; U]^T: column per lane, heads 8 g .. + 7 (U for g >= 2)
  f32x4 du[C::TILES];        // dU^T: columns 8 g.. of the pair, head q
#pragma unroll
  for (int i = 0; i < KS; ++i) dxf[i] = __builtin_bit_cast(bf16x8, zero128());
#pragma unroll
  for (int i = 0; i < C::TILES; ++i) {
    duf[i] = __builtin_bit_cast(bf16x8, zero128());
    du[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // transposed 8-head fragments of a [16, DP] slot for the lanes with `take`
  // (once per patch: the addresses are formed here each time instead of being
  // held in registers across the token slots)
  auto take_tr = [&](const char* slot, bool take) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int gg = ln >> 4, qq = ln & 15;
    int base[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int rr = 8 * (gg & 1) + 4 * hf + (qq >> 2);
        base[i][hf] = rr * C::ROWB + ((((wave * C::CPW >> 3) + 4 * i) | (qq & 3)) ^ swz(rr)) * 16;
      }
#pragma unroll
    for (int i = 0; i < C::TILES; ++i) {
      s16x4 v[2];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
        v[hf] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (ORBIT_LDS s16x4*)(slot + base[(i >> 1) & 3][hf] + (i >> 3) * 256 + 8 * (i & 1)));
      const bf16x8 n = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
      select_in_place(duf[i], n, take);
      if (i & 1) __builtin_amdgcn_sched_barrier(0);
    }
  };

  unsigned hist = 0;  // slots after which dtok was stored among the last NS - 1
  int used = NS - 1;  // ring position of the slot in use
  // wait for the next slot, hand the one before it to the copies
  auto next_slot = [&]() -> const char* {
    const int cnt = __builtin_popcount(hist);
    if (wave == 7) wait_counted<(NS - 2) * (C::NLD + 1), C::KS>(cnt);
    else wait_counted<(NS - 2) * C::NLD, C::KS>(cnt);
    lds_barrier();
    issue();
    hist = (hist << 1) & ((1u << (NS - 1)) - 1);
    if (++used == NS) used = 0;
    return smem + used * C::SLOT;
  };

  take_tr(next_slot(), g >= 2);
  for (int t = blockIdx.x; t < T; t += gridDim.x) {
    const char* slot = next_slot();
    take_tr(slot, g < 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dxf[ks] = fr.read_row(slot, ks);
    // first sweep: dA of every chunk; wave w keeps chunk w (variables 16 w + 4 g
    // .. + 3, head q), with the weights
    f32x4 da = f32x4{0.f, 0.f, 0.f, 0.f}, wa = da;
    for (int c = 0; c < nch; ++c) {
      slot = next_slot();
      // dA [variable, head] of this wave's columns
      f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s4 = mma32(fr.read_row(slot, ks), dxf[ks], s4);
        if ((ks & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      *reinterpret_cast<f32x4*>(part + wave * 1024 + lane * 16) = s4;
      lds_barrier();
      if (c == wave) {
        da = *reinterpret_cast<const f32x4*>(part + lane * 16);
#pragma unroll
        for (int w = 1; w < 8; ++w) da += *reinterpret_cast<const f32x4*>(part + w * 1024 + lane * 16);
        const float* as = reinterpret_cast<const float*>(aring + used * 1024);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool ok = c * R + 4 * g + r < V && q < H;
          wa[r] = ok ? as[(4 * g + r) * H + q] : 0.f;
          da[r] = ok ? da[r] : 0.f;
        }
      }
    }
    // c = sum_v a_v dA_v, then dS of this wave's chunk (zero past the variables and heads)
    float x = (wa[0] * da[0] + wa[1] * da[1]) + (wa[2] * da[2] + wa[3] * da[3]);
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    if (g == 0) red[wave * 16 + q] = x;
    lds_barrier();
    float cs = red[q];
#pragma unroll
    for (int w = 1; w < 8; ++w) cs += red[w * 16 + q];
    auto put = [&](int c, int buf) {
      s16x4 dt;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v = 4 * g + r;
        const bool ok = c * R + v < V && q < H;
        const bf16 ds = (bf16)(ok ? wa[r] * (da[r] - cs) * scale : 0.f);
        bf16* row = ads + (buf * 16 + v) * 32 + (q & 7);
        row[((q >> 3) ^ g) * 8] = (bf16)wa[r];
        row[((2 + (q >> 3)) ^ g) * 8] = ds;
        dt[r] = __builtin_bit_cast(short, ds);
      }
      *reinterpret_cast<s16x4*>(dst + (buf * 16 + q) * SP + 4 * g) = dt;
    };
    if (wave == nch - 1) put(wave, 0);
    lds_barrier();
    // second sweep, last chunk first
    const __amdgpu_buffer_rsrc_t rd = rsrc(dtok + (int64_t)t * V * d, V * d * 2);
    for (int c = nch - 1, buf = 0; c >= 0; --c, buf ^= 1) {
      if (c != nch - 1) slot = next_slot();
      if (wave == c - 1) put(wave, buf ^ 1);
      const bf16x8 adf = *reinterpret_cast<const bf16x8*>(ads + (buf * 16 + q) * 32 + (g ^ (q >> 2)) * 8);
      const s16x4 dsf = *reinterpret_cast<const s16x4*>(dst + (buf * 16 + q) * SP + g * 4);
      const unsigned vo = (unsigned)((c * R + q) * d + wave * C::CPW + g * 8) * 2u;
#pragma unroll
      for (int p = 0; p < KS; ++p) {
        const s16x4 x0 = fr.read_tr(slot, p, 0), x1 = fr.read_tr(slot, p, 1);
        du[2 * p] = mma16x(x0, dsf, du[2 * p]);
        du[2 * p + 1] = mma16x(x1, dsf, du[2 * p + 1]);
        const f32x4 z4 = f32x4{0.f, 0.f, 0.f, 0.f};
        const f32x4 o0 = mma32(duf[2 * p], adf, z4), o1 = mma32(duf[2 * p + 1], adf, z4);
        const u32x4 o = {pack2(o0[0], o0[1]), pack2(o0[2], o0[3]), pack2(o1[0], o1[1]), pack2(o1[2], o1[3])};
        __builtin_amdgcn_raw_buffer_store_b128(o, rd, wave * C::CPW + p * 32 + g * 8 < d ? vo + p * 64u : kOob, 0, 0);
        // two column groups in flight at a time: unbounded, the scheduler's
        // overlap of all of them spills
        if (p & 1) __builtin_amdgcn_sched_barrier(0);
      }
      hist |= 1u;
    }
  }
  wait_vmcnt<0>();
  if (q < H) {
    float* o = dupart + ((int64_t)blockIdx.x * H + q) * C::DP + wave * C::CPW + g * 8;
#pragma unroll
    for (int p = 0; p < KS; ++p) {
      *reinterpret_cast<f32x4*>(o + p * 32) = du[2 * p];
      *reinterpret_cast<f32x4*>(o + p * 32 + 4) = du[2 * p + 1];
    }
  }
}

// dU[i][h] = sum over blocks of part[block][h][i], in order: 64 columns per
// block, four groups of threads take a quarter of the partials each
__global__ void __launch_bounds__(256) agg_stream_du(const float* __restrict__ part, float* __restrict__ dU, int nb,
                                                     int H, int DP, int d) {
  __shared__ float red[4][64];
  const int i = blockIdx.x * 64 + (threadIdx.x & 63), h = blockIdx.y, grp = threadIdx.x >> 6;
  const int per = (nb + 3) / 4, b0 = grp * per, b1 = min(nb, b0 + per);
  float s = 0.f;
  if (i < DP) {
    const float* p = part + (int64_t)h * DP + i;
    const int64_t st = (int64_t)H * DP;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += p[b * st];
  }
  red[grp][threadIdx.x & 63] = s;
  __syncthreads();
  if (grp == 0 && i < d) {
    const int x = threadIdx.x;
    dU[(int64_t)i * H + h] = (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
  }
}

// columns per wave: the smallest instantiation that covers d
int cpw_of(int d) { return d <= 512 ? 64 : d <= 1024 ? 128 : d <= 1536 ? 192 : 256; }

using C64 = StreamCfg<64, 4, 2>;
using C128 = StreamCfg<128, 4, 1>;
using C192 = StreamCfg<192, 3, 1>;
using C256 = StreamCfg<256, 2, 1>;

template <typename C>
int blocks(int64_t T) { return (int)std::min<int64_t>(T, 256 * C::BPC); }

template <typename K>
void lift_lds(K kern, size_t lds) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)hipGetLastError();
}

template <typename C>
orbit_status run_fwd(const bf16* tok, const bf16* Ut, float* a32, bf16* xbar, int64_t T, int V, int d, int H,
                     float scale, hipStream_t s) {
  constexpr size_t lds = C::NS * C::SLOT + 2 * 8192;
  static const bool once = (lift_lds(agg_stream_fwd_kernel<C>, lds), true);
  (void)once;
  KernelInfo k{"agg_stream_fwd", 4.0 * T * V * (double)H * d, (double)T * (V + H) * d * 2.0 + 4.0 * T * V * H};
  return launch(k, agg_stream_fwd_kernel<C>, dim3((unsigned)blocks<C>(T)), dim3(kThreads), lds, s, tok, Ut, a32,
                xbar, (int)T, V, d, H, scale * 1.4426950408889634f);
}

template <typename C>
orbit_status run_bwd(const bf16* tok, const bf16* dxbar, const bf16* Ut, const float* a32, bf16* dtok, float* part,
                     int64_t T, int V, int d, int H, float scale, hipStream_t s) {
  constexpr size_t lds = C::NS * (C::SLOT + 1024) + 8192 + 2 * 16 * 32 * 2 + 2 * 16 * 20 * 2 + 8 * 16 * 4;
  static_assert(lds * C::BPC <= 160 * 1024, "LDS");
  static const bool once = (lift_lds(agg_stream_bwd_kernel<C>, lds), true);
  (void)once;
  KernelInfo k{"agg_stream_bwd", 8.0 * T * V * (double)H * d,
               (double)T * (2 * V + H) * d * 2.0 + 4.0 * T * V * H};
  return launch(k, agg_stream_bwd_kernel<C>, dim3((unsigned)blocks<C>(T)), dim3(kThreads), lds, s, tok, dxbar, Ut, a32,
                dtok, part, (int)T, V, d, H, scale);
}

}  // namespace

// The upper limits are the kernels' own: 16 heads fill an MFMA tile (8 leave half
// of it empty), a wave keeps the scores of one 16-variable slot (V <= 128), and
// the accumulators of 2048 columns fill the registers of a CU. Below d = 256 a
// block works on mostly padded columns: with few variables the forward is
// slower than the general path's (4096 patches x 2 x 64, 8 heads: 30 -> 37 us; x
// 12 x 64: 36 -> 38; x 12 x 128: 1.10 times as fast). Inside the limits both
// directions are faster at every size measured (64 to 8192 patches, 2 to 128
// variables, 64 to 2048 columns).
bool agg_stream_ok(orbit_dtype dt, int V, int d, int H) {
  return dt == ORBIT_BF16 && (H == 8 || H == 16) && V <= kMaxV && d <= kMaxD && d % 8 == 0 &&
         (d >= 256 || V * d >= 1024);
}
int agg_stream_blocks(int64_t T, int d) { return cpw_of(d) == 64 ? blocks<C64>(T) : blocks<C128>(T); }
int agg_stream_cols(int d) { return 8 * cpw_of(d); }

orbit_status agg_stream_fwd(const bf16* tok, const bf16* Ut, float* a32, bf16* xbar, int64_t T, int V, int d, int H,
                            float scale, hipStream_t s) {
  switch (cpw_of(d)) {
    case 64: return run_fwd<C64>(tok, Ut, a32, xbar, T, V, d, H, scale, s);
    case 128: return run_fwd<C128>(tok, Ut, a32, xbar, T, V, d, H, scale, s);
    case 192: return run_fwd<C192>(tok, Ut, a32, xbar, T, V, d, H, scale, s);
    default: return run_fwd<C256>(tok, Ut, a32, xbar, T, V, d, H, scale, s);
  }
}

orbit_status agg_stream_bwd(const bf16* tok, const bf16* dxbar, const bf16* Ut, const float* a32, bf16* dtok,
                            float* part, float* dU, int64_t T, int V, int d, int H, float scale, hipStream_t s) {
  orbit_status st;
  switch (cpw_of(d)) {
    case 64: st = run_bwd<C64>(tok, dxbar, Ut, a32, dtok, part, T, V, d, H, scale, s); break;
    case 128: st = run_bwd<C128>(tok, dxbar, Ut, a32, dtok, part, T, V, d, H, scale, s); break;
    case 192: st = run_bwd<C192>(tok, dxbar, Ut, a32, dtok, part, T, V, d, H, scale, s); break;
    default: st = run_bwd<C256>(tok, dxbar, Ut, a32, dtok, part, T, V, d, H, scale, s); break;
  }
  ORBIT_TRY(st);
  const int nb = agg_stream_blocks(T, d), DP = agg_stream_cols(d);
  KernelInfo k{"agg_stream_du", 0.0, (double)nb * H * DP * 4.0};
  return launch(k, agg_stream_du, dim3((unsigned)cdiv(d, 64), (unsigned)H), dim3(256), 0, s, (const float*)part, dU, nb,
                H, DP, d);
}

}  // namespace orbit
