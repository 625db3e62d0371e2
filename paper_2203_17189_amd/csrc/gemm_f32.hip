// float32 GEMM on the matrix units.  Small problems run on v_mfma_f32_32x32x2_f32 (float32 operands, products and sums),
// larger ones on the bf16 units with every operand in three parts (second kernel below).
//
//   C[m,n] = sum_s sum_k A_s(m,k) B_s(n,k)
//
// Bound: the float32 matrix rate, 157 TFLOP/s nominal (a vendor GEMM of 4096^3 sustains 148 here); one MFMA of 4096
// FLOP keeps its unit busy for 64 cycles and needs two registers of operands, so neither LDS nor the L2 is near a
// limit from 64x64 tiles on and the operands go through registers into LDS in plain code: that is where ragged edges
// are filled with zeros, so the kernel takes any shape, leading dimension and alignment (float4 where the alignment
// allows it, single elements elsewhere).
//
// Tiles: BM x BN per workgroup, k-tiles of BK, WM x WN x WK wavefronts.  WK > 1 gives each of WK wavefronts its share
// of every k-tile; their sums meet in LDS in a fixed order: two wavefronts with 64x64 tiles, eight with 32x64.  (Problems of few
// tiles have a kernel of their own, below.)
//
// Operand layouts in LDS (floats):
//   k-contiguous (A[m][k])  rows of BK k, padded by 4: a lane reads 4 consecutive k of its row (ds_read_b128; 16 rows
//                           cover the 64 banks once);
//   m-contiguous (A[k][m])  rows of BM m, padded by 8: a lane reads its column from 4 consecutive rows (ds_read_b32;
//                           the two lane halves read rows 4 apart, 32 banks apart).
// MFMA e of a group of 8 k contracts k = 4*half + e of both operands: any pairing serves as long as both agree.
//
// Measured on the layer d 512, 6 heads, d_ff 1024, 4000 tokens (forward + backward): GEMMs 5.0 ms with the FMA kernel
// this replaced for float32 (64x64 tiles, 4x4 products a thread, one load in flight), 650 us with float32 instructions
// everywhere, 610 us now.
#include "kernels.h"
#include <algorithm>
#include <atomic>

namespace t5mi {

namespace {

// Workgroup -> (n tile, m tile, k-slice).  Consecutive workgroups go to different XCDs, so each XCD takes a contiguous run of
// the tiles in the order n, m, slice: the tiles that share rows of A (or a slice's k range) meet in one L2.
struct TilePos {
  int x, y, z;
};
__device__ __forceinline__ TilePos tile_pos(int gx, int gy) {
  const uint32_t n = gridDim.x, id = blockIdx.x, q = n / 8, r = n % 8, xcd = id % 8;
  uint32_t t = xcd * q + (xcd < r ? xcd : r) + id / 8;
  TilePos p;
  p.x = (int)(t % (uint32_t)gx);
  t /= (uint32_t)gx;
  p.y = (int)(t % (uint32_t)gy);
  p.z = (int)(t / (uint32_t)gy);
  return p;
}

struct F32Src {  // where a thread's float4 slot of an operand comes from
  size_t off;    // elements from (segment base + tile start)
  int row;       // position along the contraction (m-contiguous) or first k of the slot (k-contiguous)
  int nv;        // m-contiguous: valid elements of the slot; k-contiguous: 1 if the row exists
};

// Slot of a thread: four elements at base + off of which the first nv exist.  VEC (every slot exists whole or not at
// all): one load from an address that is valid either way, zeroed by the caller when it is used -- a branch around
// the load makes the compiler wait for it on the spot.  Otherwise element by element.
template <bool VEC>
__device__ __forceinline__ f32x4 ld4(const float* base, size_t off, int nv) {
  if constexpr (VEC) {
    return *reinterpret_cast<const f32x4*>(base + (nv > 0 ? off : 0));
  } else {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < nv) v[q] = base[off + q];
    return v;
  }
}

// Epilogue of a wavefront's MI x NI tiles from (mw, nw) on: register r of a 32x32 tile is row (r/4)*8 + half*4 + r%4,
// column lane%32: a wavefront writes 128-byte runs of two rows.  Operands of the epilogue are fetched for a whole row of tiles before the first store:
// the compiler cannot move a load across a store that might alias it, and one at a time each costs a round trip
// (the gated-GELU backward at 64 tokens: 23 us, most of it here).
template <bool FULL, int MI, int NI, int EPI>
__device__ __forceinline__ void f32_epilogue_part(const GemmDesc& g, const GemmEpi& e, int split_k, const f32x16 (&acc)[MI][NI],
                                             int mw, int nw, int slice, int lane) {
  const int g2 = lane >> 5, l32 = lane & 31;
  constexpr bool AUX = EPI == EPI_RESID || EPI == EPI_GEGLU_BWD || EPI == EPI_SPLIT_F32;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int mb = mw + i * 32 + (g2 << 2), nb = nw + l32;
    float xa[AUX ? 16 : 1][NI], xb[EPI == EPI_GEGLU_BWD ? 16 : 1][NI];
    if (AUX && (EPI != EPI_SPLIT_F32 || (split_k == 1 && e.accumulate))) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int m = mb + ((r >> 2) << 3) + (r & 3), n = nb + j * 32;
          const int mc = FULL || m < g.M ? m : g.M - 1, nc = FULL || n < g.N ? n : g.N - 1;
          if constexpr (EPI == EPI_SPLIT_F32) {
            const int which = nc / e.split_n;  // (one slice)
            const float* d = (const float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2);
            xa[r][j] = d[(size_t)mc * e.ld0 + (nc - which * e.split_n)];
          } else if constexpr (AUX) {
            const size_t oa = (size_t)mc * (e.ld_aux ? e.ld_aux : e.ld0) + nc;
            xa[r][j] = ((const float*)e.aux0)[oa];
            if constexpr (EPI == EPI_GEGLU_BWD) xb[r][j] = ((const float*)e.aux1)[oa];
          }
        }
    } else if (AUX) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < NI; ++j) xa[AUX ? r : 0][j] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mb + ((r >> 2) << 3) + (r & 3);
      if (!FULL && m >= g.M) continue;
      const uint32_t k1 = e.drop.on ? drop_row_key(e.drop, (uint32_t)m) : 0u;
      if constexpr (EPI == EPI_GEGLU_FWD) {
#pragma unroll
        for (int j = 0; j < NI; j += 2) {
          const int f = ((nw + j * 32) >> 1) + l32;
          if (!FULL && f >= (g.N >> 1)) continue;
          float gl, dgl;
          gelu_both(e.act, acc[i][j][r], gl, dgl);
          const float w = acc[i][j + 1][r];
          const float mk = e.drop.on ? drop_mult(e.drop, k1, (uint32_t)f) : 1.f;
          const size_t o = (size_t)m * e.ld0 + f;
          ((float*)e.out0)[o] = w * dgl * mk;
          ((float*)e.out1)[o] = gl * mk;
          ((float*)e.out2)[o] = gl * w * mk;
        }
      } else {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int n = nb + j * 32;
          if (!FULL && n >= g.N) continue;
          const float v = acc[i][j][r];
          const size_t o = (size_t)m * e.ld0 + n;
          if constexpr (EPI == EPI_STORE) {
            const float mk = e.drop.on ? drop_mult(e.drop, k1, (uint32_t)n) : 1.f;
            ((float*)e.out0)[o] = (e.act == ACT_RELU ? fmaxf(v, 0.f) : v) * mk;
          } else if constexpr (EPI == EPI_RESID) {
            const float a = xa[r][j], sc = e.drop.on ? e.drop.scale : 1.f;
            const float mk = e.drop.on && !e.aux_mask ? drop_mult(e.drop, k1, (uint32_t)n) : 1.f;
            ((float*)e.out0)[o] = e.aux_mask ? (a > 0.f ? v * sc : 0.f) : v * mk + a;
          } else if constexpr (EPI == EPI_GEGLU_BWD) {
            ((float*)e.out0)[o] = v * xa[r][j];
            ((float*)e.out1)[o] = v * xb[r][j];
          } else {  // EPI_SPLIT_F32
            if (split_k > 1) {  // this slice's sums, for launch_split_reduce
              ((float*)const_cast<void*>(e.aux0))[((size_t)slice * g.M + m) * g.N + n] = v;
            } else {
              const int which = n / e.split_n;
              float* dst = (float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2);
              dst[(size_t)m * e.ld0 + (n - which * e.split_n)] = xa[r][j] + v;
            }
          }
        }
      }
    }
  }
}

// FULL: every element of the wavefront's tiles exists, no test and no branch per element.
template <int MI, int NI, int EPI>
__device__ __forceinline__ void f32_epilogue(const GemmDesc& g, const GemmEpi& e, int split_k, const f32x16 (&acc)[MI][NI],
                                             int mw, int nw, int slice, int lane) {
  if (mw + MI * 32 <= g.M && nw + NI * 32 <= g.N) f32_epilogue_part<true, MI, NI, EPI>(g, e, split_k, acc, mw, nw, slice, lane);
  else f32_epilogue_part<false, MI, NI, EPI>(g, e, split_k, acc, mw, nw, slice, lane);
}

template <int BM, int BN, int WM, int WN, int WK, int BK, bool A_KC, bool B_KC, int EPI, bool VEC>
__global__ __launch_bounds__(WM * WN * WK * 64) void gemm_f32_kernel(GemmDesc g, GemmEpi e, int split_k) {
  constexpr int NT = WM * WN * WK * 64;
  constexpr int TMW = BM / WM, TNW = BN / WN, MI = TMW / 32, NI = TNW / 32;
  constexpr int A_LD = A_KC ? BK + 4 : BM + 8, B_LD = B_KC ? BK + 4 : BN + 8;
  constexpr int A_FL = (A_KC ? BM : BK) * A_LD, B_FL = (B_KC ? BN : BK) * B_LD, STG = A_FL + B_FL;
  constexpr int A_SL = BM * BK / 4 / NT, B_SL = BN * BK / 4 / NT;  // float4 slots per thread
  static_assert(BM * BK % (4 * NT) == 0 && BN * BK % (4 * NT) == 0 && BK % (8 * WK) == 0, "tile vs threads");
  static_assert(EPI != EPI_GEGLU_FWD || NI % 2 == 0, "u and w columns in one wavefront");
  extern __shared__ __attribute__((aligned(16))) float sm[];

  const int tid = threadIdx.x, lane = tid & 63, g2 = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WM * WN), wmn = wave % (WM * WN), wm = wmn / WN, wn = wmn % WN;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

  // this slice's run of k-tiles (several segments are never sliced)
  int nt = 0;
  for (int s = 0; s < g.nseg; ++s) nt += (g.seg[s].K + BK - 1) / BK;
  const int per = (nt + split_k - 1) / split_k;
  const int t_begin = blockIdx.z * per, t_end = t_begin + per < nt ? t_begin + per : nt;

  const int lda = g.seg[0].lda, ldb = g.seg[0].ldb;
  F32Src sa[A_SL], sb[B_SL];
#pragma unroll
  for (int i = 0; i < A_SL; ++i) {
    const int q = tid + i * NT;
    if constexpr (A_KC) {
      const int r = q / (BK / 4), k = (q % (BK / 4)) * 4, m = m0 + r;
      sa[i].off = (size_t)(m < g.M ? m : 0) * lda + k;
      sa[i].row = k;
      sa[i].nv = m < g.M;
    } else {
      const int k = q / (BM / 4), m = m0 + (q % (BM / 4)) * 4;
      sa[i].off = (size_t)k * lda + m;
      sa[i].row = k;
      sa[i].nv = g.M - m < 0 ? 0 : g.M - m;
    }
  }
  const float* b_src[B_SL];  // operand of the slot where columns come from several matrices (nsrc > 1)
#pragma unroll
  for (int i = 0; i < B_SL; ++i) {
    const int q = tid + i * NT;
    b_src[i] = nullptr;
    if constexpr (B_KC) {
      const int r = q / (BK / 4), k = (q % (BK / 4)) * 4, n = n0 + r;
      sb[i].off = (size_t)(n < g.N ? n : 0) * ldb + k;
      sb[i].row = k;
      sb[i].nv = n < g.N;
    } else {
      const int k = q / (BN / 4), c = (q % (BN / 4)) * 4;
      int n = n0 + c, lim = g.N;
      if constexpr (EPI == EPI_GEGLU_FWD) {  // packed columns: 32 of wi0, 32 of wi1, ...
        b_src[i] = (const float*)(c & 32 ? g.seg[1].B : g.seg[0].B);
        n = (n0 >> 1) + ((c >> 6) << 5) + (c & 31);
        lim = g.N >> 1;
      } else if (g.nsrc > 1) {  // N = nsrc matrices of nsrc_cols columns side by side (a tile may straddle two)
        int s = n / g.nsrc_cols;
        s = s < g.nsrc ? s : g.nsrc - 1;
        b_src[i] = (const float*)g.seg[s].B;
        n -= s * g.nsrc_cols;
        lim = g.nsrc_cols;
      }
      sb[i].off = (size_t)k * ldb + n;
      sb[i].row = k;
      sb[i].nv = lim - n < 0 ? 0 : lim - n;
    }
  }

  f32x4 ra[A_SL], rb[B_SL];
  bool oka[A_SL], okb[B_SL];
  int seg = 0, kt = t_begin;  // tile kt of segment seg comes next
  int seg_nt = (g.seg[0].K + BK - 1) / BK;
  auto fetch = [&]() __attribute__((always_inline)) {
    while (kt >= seg_nt) {  // next segment
      kt -= seg_nt;
      ++seg;
      seg_nt = (g.seg[seg].K + BK - 1) / BK;
    }
    const int k0 = kt * BK, left = g.seg[seg].K - k0;
    const float* A = (const float*)g.seg[seg].A;
    const float* B = (const float*)g.seg[seg].B;
    const size_t oa = A_KC ? (size_t)k0 : (size_t)k0 * lda, ob = B_KC ? (size_t)k0 : (size_t)k0 * ldb;
#pragma unroll
    for (int i = 0; i < A_SL; ++i) {
      const int nv = A_KC ? (sa[i].nv ? left - sa[i].row : 0) : (sa[i].row < left ? sa[i].nv : 0);
      oka[i] = nv > 0;
      ra[i] = ld4<VEC>(A, sa[i].off + oa, nv);
    }
#pragma unroll
    for (int i = 0; i < B_SL; ++i) {
      const int nv = B_KC ? (sb[i].nv ? left - sb[i].row : 0) : (sb[i].row < left ? sb[i].nv : 0);
      okb[i] = nv > 0;
      rb[i] = ld4<VEC>(b_src[i] ? b_src[i] : B, sb[i].off + ob, nv);
    }
    ++kt;
  };
  auto put = [&](int st) __attribute__((always_inline)) {
    float* pa = sm + st * STG;
    float* pb = pa + A_FL;
#pragma unroll
    for (int i = 0; i < A_SL; ++i) {
      const int q = tid + i * NT;
      constexpr int W = (A_KC ? BK : BM) / 4;
      f32x4 v = ra[i];
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = !VEC || oka[i] ? v[x] : 0.f;
      *reinterpret_cast<f32x4*>(pa + (q / W) * A_LD + (q % W) * 4) = v;
    }
#pragma unroll
    for (int i = 0; i < B_SL; ++i) {
      const int q = tid + i * NT;
      constexpr int W = (B_KC ? BK : BN) / 4;
      f32x4 v = rb[i];
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = !VEC || okb[i] ? v[x] : 0.f;
      *reinterpret_cast<f32x4*>(pb + (q / W) * B_LD + (q % W) * 4) = v;
    }
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto compute = [&](int st) __attribute__((always_inline)) {
    const float* pa = sm + st * STG;
    const float* pb = pa + A_FL;
#pragma unroll
    for (int s = 0; s < BK / WK / 8; ++s) {
      const int kb = wk * (BK / WK) + s * 8 + g2 * 4;
      f32x4 fa[MI], fb[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int m = wm * TMW + i * 32 + l32;
        if constexpr (A_KC) fa[i] = *reinterpret_cast<const f32x4*>(pa + m * A_LD + kb);
        else
#pragma unroll
          for (int q = 0; q < 4; ++q) fa[i][q] = pa[(kb + q) * A_LD + m];
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n = wn * TNW + j * 32 + l32;
        if constexpr (B_KC) fb[j] = *reinterpret_cast<const f32x4*>(pb + n * B_LD + kb);
        else
#pragma unroll
          for (int q = 0; q < 4; ++q) fb[j][q] = pb[(kb + q) * B_LD + n];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[j][q], acc[i][j], 0, 0, 0);
    }
  };

  // Two stages: tile t+1 travels through registers while tile t is multiplied; its stage was last read at tile t-1,
  // before the barrier that ended it.
  if (t_begin < t_end) {
    fetch();
    put(0);
    __syncthreads();
    for (int t = t_begin; t < t_end; ++t) {
      const int cur = (t - t_begin) & 1;
      if (t + 1 < t_end) fetch();
      compute(cur);
      if (t + 1 < t_end) put(cur ^ 1);
      __syncthreads();
    }
  }
  if constexpr (WK > 1) {  // sums of the WK shares, in order, in the wavefronts of share 0
    constexpr int PW = MI * NI * 16 * 64;  // floats per wavefront
    if (wk > 0) {
      float* d = sm + ((wk - 1) * WM * WN + wmn) * PW + lane;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) d[((i * NI + j) * 16 + r) * 64] = acc[i][j][r];
    }
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int w = 1; w < WK; ++w) {
      const float* d = sm + ((w - 1) * WM * WN + wmn) * PW + lane;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += d[((i * NI + j) * 16 + r) * 64];
    }
  }

  f32_epilogue_part<false, MI, NI, EPI>(g, e, split_k, acc, m0 + wm * TMW, n0 + wn * TNW, blockIdx.z, lane);
}

// ------------------------------------------------------------------ the same on the bf16 matrix units
// Every operand as three bf16 parts, a = a0 + a1 + a2 exactly, and eight of the nine products of parts:
//   a b = a0 b0 + (a0 b1 + a1 b0 + a1 b1 + a0 b2 + a2 b0 + a1 b2 + a2 b1),  what is left out is 2^-34 of it and less.
// (|a1| is up to 2^-8 of |a| and |a2| up to 2^-17: a1 b2 + a2 b1 reaches 2^-24, as much as the rounding of a float32 product, and
// a sum with one term in it shows that.)  The parts are those of 2^16 a: the last bit of any float32 number, 2^-149, is then
// 2^-133, the last of bf16, and the matrix unit keeps subnormal numbers; at the other end, from 2^112 on, the parts are
// not finite, which shows in the sum.
// Eight bf16 products of 32x32x16 take 256 cycles where the float32 instructions take 512 for the same k, and the sums lose less:
// a0 b0 meets in one accumulator (one rounding in 16 k; float32 instructions round every two), the seven small
// products in another, whose roundings are 2^-7 of the first one's.  Error of a layer's results against 64 bits, d 512,
// 16 x 250 tokens: y 4.2e-7 -> 1.8e-7, weight gradients 7.0e-7..1.04e-6 -> 2.9e-7..6.6e-7; one term alone: 2^-24, as before.
// Bound: the vector instructions of the conversion (6 a value) and the LDS round trips between the barriers, beside the matrix
// unit; d 768, 4000 tokens: products of a layer 1828 -> 1501 us (134 TFLOP/s with 1024 tiles), d 512: 665 -> 611.  With six
// products (without a1 b2 and a2 b1) and unscaled parts 1402 and 562, at up to 1.7 times the error for one term and
// fewer than 24 bits of values below 2^-110.
// Results that are formed again: a layer of 16 x 250 tokens, d 512, takes 2.1 ms instead of 0.83 with one token that is not
// finite (all its weight gradients are not) and 2.4 with all of them.
// A tile is requested D k-tiles ahead into registers, converted once and written to one of two LDS stages (rows of
// BK k of each part, padded by 16 bytes: 16 rows cover the banks once) while the other one is multiplied.
// Measured and left: parts by truncation instead of rounding (same time, y 2.0e-7); fragments read one k-tile ahead
// (dn2 of d 512 92 -> 83 us, but one wavefront a SIMD: weight gradients a fifth slower); k-tiles of 32 at 128x128.

constexpr float kUp = 65536.f;  // the parts are those of this times the operand (above)

// Four float32 values as three bf16 parts each (two 32-bit words per part), x = p0 + p1 + p2 exactly: every part is the
// rounded remainder of the ones before it, eight significant bits at a time.
struct Split3 {
  u32x2 p[3];
};
__device__ __forceinline__ Split3 split3(f32x4 v) {
  Split3 s;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t u = pack_bf16x2(v[2 * h], v[2 * h + 1]);
      s.p[p][h] = u;
      if (p < 2) {
        v[2 * h] -= __builtin_bit_cast(float, u << 16);
        v[2 * h + 1] -= __builtin_bit_cast(float, u & 0xFFFF0000u);
      }
    }
  }
  return s;
}

// MANY: the columns of B come from several matrices
template <int BM, int BN, int WM, int WN, int BK, int D, bool A_KC, bool B_KC, int EPI, bool MANY>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_f32x3_kernel(GemmDesc g, GemmEpi e, int split_k) {
  constexpr int NT = WM * WN * 64;
  constexpr int TMW = BM / WM, TNW = BN / WN, MI = TMW / 32, NI = TNW / 32;
  constexpr int LD = BK * 2 + 16;                        // bytes of a row of one part in LDS
  constexpr int A_PL = BM * LD, B_PL = BN * LD;          // one part of a tile
  constexpr int STG = 3 * (A_PL + B_PL);
  constexpr int A_SL = BM * BK / 4 / NT, B_SL = BN * BK / 4 / NT;  // slots of four k per thread
  static_assert(NT % BM == 0 && NT % BN == 0 && BM >= 64 && BN >= 64, "a wavefront's slots share their four k");
  static_assert(EPI != EPI_GEGLU_FWD || NI % 2 == 0, "u and w columns in one wavefront");
  extern __shared__ __attribute__((aligned(16))) char smx[];

  const int tid = threadIdx.x, lane = tid & 63, g2 = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const TilePos pos = tile_pos((g.N + BN - 1) / BN, (g.M + BM - 1) / BM);
  const int m0 = pos.y * BM, n0 = pos.x * BN;

  int nt = 0;
  for (int s = 0; s < g.nseg; ++s) nt += (g.seg[s].K + BK - 1) / BK;
  const int per = (nt + split_k - 1) / split_k;
  const int t_begin = pos.z * per, t_end = t_begin + per < nt ? t_begin + per : nt;
  const int lda = g.seg[0].lda, ldb = g.seg[0].ldb;

  // Column c of this tile of B: its matrix (MANY) and its column there.  Rows and columns past the end repeat the last
  // one: their results are not stored.
  auto b_col = [&](int c, const float*& src) __attribute__((always_inline)) {
    int n = n0 + c, lim = g.N;
    if constexpr (EPI == EPI_GEGLU_FWD) {  // packed columns: 32 of wi0, 32 of wi1, ...
      src = (const float*)(c & 32 ? g.seg[1].B : g.seg[0].B);
      n = (n0 >> 1) + ((c >> 6) << 5) + (c & 31);
      lim = g.N >> 1;
    } else if constexpr (MANY) {  // N = nsrc matrices of nsrc_cols columns side by side (a tile may straddle two)
      int s = n / g.nsrc_cols;
      s = s < g.nsrc ? s : g.nsrc - 1;
      src = (const float*)(s == 0 ? g.seg[0].B : s == 1 ? g.seg[1].B : g.seg[2].B);
      n -= s * g.nsrc_cols;
      lim = g.nsrc_cols;
    }
    return n < lim ? n : lim - 1;
  };

  // Slot i of a thread: row r, k = 4 * (...) of a k-contiguous operand, offset from the tile's first row; or column c
  // and wavefront-uniform rows of an m-contiguous one.
  uint32_t oa[A_KC ? A_SL : 1], ob[B_KC ? B_SL : 1];
  const float* b_src = nullptr;
  const int wka = (wave * 64) / BM, wkb = (wave * 64) / BN;  // m-contiguous: first group of four k of the wavefront
  if constexpr (A_KC) {
#pragma unroll
    for (int i = 0; i < A_SL; ++i) {
      const int q = tid + i * NT, r = q / (BK / 4), k = (q % (BK / 4)) * 4;
      oa[i] = (uint32_t)((m0 + r < g.M ? r : g.M - 1 - m0) * lda + k);
    }
  } else {
    const int c = tid % BM;
    oa[0] = (uint32_t)(m0 + c < g.M ? c : g.M - 1 - m0);
  }
  if constexpr (B_KC) {
#pragma unroll
    for (int i = 0; i < B_SL; ++i) {
      const int q = tid + i * NT, r = q / (BK / 4), k = (q % (BK / 4)) * 4;
      ob[i] = (uint32_t)((n0 + r < g.N ? r : g.N - 1 - n0) * ldb + k);
    }
  } else {
    const float* src = nullptr;
    const int n = b_col(tid % BN, src);
    ob[0] = MANY ? 0u : (uint32_t)(n - n0);
    if (MANY) b_src = src + n;
  }

  f32x4 raw_a[D][A_SL], raw_b[D][B_SL];  // tiles on their way
  int left[D];                           // k from the start of each on
  // The tile that is requested next: its segment (in scalar registers, chosen without a branch) and number.
  int seg = 0, kt = t_begin;
  const int K0 = g.seg[0].K, K1 = g.seg[1].K, K2 = g.seg[2].K, nseg = g.nseg;
  const float *A0 = (const float*)g.seg[0].A, *A1 = (const float*)g.seg[1].A, *A2 = (const float*)g.seg[2].A;
  const float *B0 = (const float*)g.seg[0].B, *B1 = (const float*)g.seg[1].B, *B2 = (const float*)g.seg[2].B;
  auto pick = [&](auto x0, auto x1, auto x2) __attribute__((always_inline)) { return seg == 0 ? x0 : seg == 1 ? x1 : x2; };
  while (seg + 1 < nseg && kt >= (pick(K0, K1, K2) + BK - 1) / BK) kt -= (pick(K0, K1, K2) + BK - 1) / BK, ++seg;
  auto advance = [&]() __attribute__((always_inline)) {  // stays on the last tile
    const bool same = (kt + 1) * BK < pick(K0, K1, K2), next = !same && seg + 1 < nseg;
    kt = next ? 0 : same ? kt + 1 : kt;
    seg = next ? seg + 1 : seg;
  };
  auto fetch = [&](f32x4 (&ra)[A_SL], f32x4 (&rb)[B_SL], int& left) __attribute__((always_inline)) {
    const int k0 = kt * BK;
    left = pick(K0, K1, K2) - k0;
    const float* A = pick(A0, A1, A2) + (A_KC ? (size_t)m0 * lda + k0 : (size_t)k0 * lda + m0);
    const float* B = pick(B0, B1, B2) + (B_KC ? (size_t)n0 * ldb + k0 : (size_t)k0 * ldb + n0);
    if constexpr (A_KC) {
      const int k = (tid % (BK / 4)) * 4;
#pragma unroll
      for (int i = 0; i < A_SL; ++i) {
        ra[i] = *reinterpret_cast<const f32x4*>(A + (k < left ? oa[i] : oa[i] - k));
      }
    } else {
#pragma unroll
      for (int i = 0; i < A_SL; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = (wka + i * (NT / BM)) * 4 + q;
          ra[i][q] = (A + (size_t)(k < left ? k : left - 1) * lda)[oa[0]];
        }
    }
    if constexpr (B_KC) {
      const int k = (tid % (BK / 4)) * 4;
#pragma unroll
      for (int i = 0; i < B_SL; ++i) {
        rb[i] = *reinterpret_cast<const f32x4*>(B + (k < left ? ob[i] : ob[i] - k));
      }
    } else {
#pragma unroll
      for (int i = 0; i < B_SL; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = (wkb + i * (NT / BN)) * 4 + q;
          const size_t o = (size_t)(k < left ? k : left - 1) * ldb;
          rb[i][q] = MANY ? b_src[(size_t)k0 * ldb + o] : (B + o)[ob[0]];
        }
    }
    advance();
  };
  // Values times kUp, so that the parts of the smallest of them are bf16 numbers too.  Rows of A past the end of k become
  // zeros; those of B repeat its last one (where that is not finite, the check behind the loop sees it).
  auto put = [&](char* st, f32x4 (&ra)[A_SL], const f32x4 (&rb)[B_SL], int left) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_SL; ++i) {
      const int q = tid + i * NT;
      const int r = A_KC ? q / (BK / 4) : tid % BM, k = A_KC ? (q % (BK / 4)) * 4 : (wka + i * (NT / BM)) * 4;
#pragma unroll
      for (int x = 0; x < 4; ++x) ra[i][x] *= k + (A_KC ? 0 : x) < left ? kUp : 0.f;  // (k-contiguous: k % 4 == 0)
      const Split3 s = split3(ra[i]);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2*>(st + p * A_PL + r * LD + k * 2) = s.p[p];
    }
#pragma unroll
    for (int i = 0; i < B_SL; ++i) {
      const int q = tid + i * NT;
      const int r = B_KC ? q / (BK / 4) : tid % BN, k = B_KC ? (q % (BK / 4)) * 4 : (wkb + i * (NT / BN)) * 4;
      const Split3 s = split3(rb[i] * kUp);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2*>(st + 3 * A_PL + p * B_PL + r * LD + k * 2) = s.p[p];
    }
  };

  f32x16 acc[MI][NI], lo[MI][NI];  // products of the first parts; the five that are 2^-8 of them and less
  auto clear = [&](f32x16 (&c)[MI][NI]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[i][j][r] = 0.f;
  };
  clear(acc);
  clear(lo);

  if (t_begin < t_end) {
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(raw_a[u], raw_b[u], left[u]);
    put(smx, raw_a[0], raw_b[0], left[0]);
    fetch(raw_a[0], raw_b[0], left[0]);
    for (int t0 = t_begin; t0 < t_end; t0 += D)
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int t = t0 + u, v = (u + 1) % D;
      if (t >= t_end) break;
      char* cur = smx + ((t - t_begin) & 1) * STG;
      char* nxt = smx + STG - ((t - t_begin) & 1) * STG;
      __syncthreads();
      constexpr int NS = BK / 16, NP = 8;  // steps of 16 k; products of parts
      bf16x8 fa[NS][MI][3], fb[NS][NI][3];
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
          for (int i = 0; i < MI; ++i)
            fa[s][i][p] = *reinterpret_cast<const bf16x8*>(cur + p * A_PL + (wm * TMW + i * 32 + l32) * LD + s * 32 + g2 * 16);
#pragma unroll
          for (int j = 0; j < NI; ++j)
            fb[s][j][p] = *reinterpret_cast<const bf16x8*>(cur + 3 * A_PL + p * B_PL + (wn * TNW + j * 32 + l32) * LD + s * 32 + g2 * 16);
        }
      put(nxt, raw_a[v], raw_b[v], left[v]);  // tile t + 1 (behind the last one: that one again, unread)
      fetch(raw_a[v], raw_b[v], left[v]);     // tile t + 1 + D
      constexpr int PA[NP] = {0, 1, 2, 2, 0, 1, 1, 0}, PB[NP] = {0, 2, 1, 0, 2, 1, 0, 1};
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
              f32x16& c = p == 0 ? acc[i][j] : lo[i][j];
              c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][i][PA[p]], fb[s][j][PB[p]], c, 0, 0, 0);
            }
      // one product, then its share of the next tile's conversion: a matrix instruction keeps its unit busy for 32 cycles,
      // in which the wavefront issues eight others
      constexpr int NMF = NS * NP * MI * NI, VAL = ((A_SL + B_SL) * 28 + NMF - 1) / NMF + 1;
      __builtin_amdgcn_sched_group_barrier(0x100, NS * 3 * (MI + NI), 0);
#pragma unroll
      for (int x = 0; x < NMF; ++x) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, VAL, 0);
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = (acc[i][j][r] + lo[i][j][r]) * (1.f / kUp / kUp);

  // A result that is not finite: infinite operands and those from 2^112 on have no parts, products from 2^96 on no sum.  The
  // wavefront forms its tiles again from the float32 values themselves (rare; operands from global memory) and takes
  // those results for these elements and no others: its row and its column alone decide the bits of a result.
  float chk = 0.f;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) chk = fmaf(acc[i][j][r], 0.f, chk);
  if (__builtin_expect(__any(chk != 0.f), 0)) {
    clear(lo);
    seg = 0;
    kt = t_begin;
    while (seg + 1 < nseg && kt >= (pick(K0, K1, K2) + BK - 1) / BK) kt -= (pick(K0, K1, K2) + BK - 1) / BK, ++seg;
    for (int t = t_begin; t < t_end; ++t) {
      const int K = pick(K0, K1, K2);
      const float* A = pick(A0, A1, A2);
      const float* B = pick(B0, B1, B2);
      for (int k0 = kt * BK; k0 < (kt + 1) * BK && k0 < K; k0 += 2) {
        const int k = k0 + g2, kc = k < K ? k : K - 1;
        float va[MI], vb[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          int m = m0 + wm * TMW + i * 32 + l32;
          m = m < g.M ? m : g.M - 1;
          const float v = A_KC ? A[(size_t)m * lda + kc] : A[(size_t)kc * lda + m];
          va[i] = k < K ? v : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const float* src = B;
          const int n = b_col(wn * TNW + j * 32 + l32, src);
          const float v = B_KC ? src[(size_t)n * ldb + kc] : src[(size_t)kc * ldb + n];
          vb[j] = k < K ? v : 0.f;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) lo[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i], vb[j], lo[i][j], 0, 0, 0);
      }
      advance();
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = fabsf(acc[i][j][r]) < INFINITY ? acc[i][j][r] : lo[i][j][r];
  }
  f32_epilogue<MI, NI, EPI>(g, e, split_k, acc, m0 + wm * TMW, n0 + wn * TNW, pos.z, lane);
}

template <int BM, int BN, int BK, int D, bool A_KC, bool B_KC, int EPI, bool MANY>
hipError_t launch_x3_cols(const GemmDesc& g, const GemmEpi& e, int split_k, hipStream_t st) {
  constexpr int lds = 6 * (BM + BN) * (BK * 2 + 16);
  auto kern = gemm_f32x3_kernel<BM, BN, 2, 2, BK, D, A_KC, B_KC, EPI, MANY>;
  if constexpr (lds > 65536) {
    static std::atomic<bool> attr_set{false};  // once per instantiation; setting it twice is harmless
    if (!attr_set.load(std::memory_order_relaxed)) {
      hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (err != hipSuccess) return err;
      attr_set.store(true, std::memory_order_relaxed);
    }
  }
  const unsigned grid = (unsigned)ceil_div(g.N, BN) * ceil_div(g.M, BM) * split_k;
  kern<<<grid, 256, lds, st>>>(g, e, split_k);
  return hipGetLastError();
}
template <int BM, int BN, int BK, int D, bool A_KC, bool B_KC, int EPI>
hipError_t launch_x3(const GemmDesc& g, const GemmEpi& e, int split_k, hipStream_t st) {
  if constexpr (EPI == EPI_GEGLU_FWD) return launch_x3_cols<BM, BN, BK, D, A_KC, B_KC, EPI, true>(g, e, split_k, st);
  if constexpr (EPI == EPI_STORE && !B_KC)
    if (g.nsrc > 1) return launch_x3_cols<BM, BN, BK, D, A_KC, B_KC, EPI, true>(g, e, split_k, st);
  if constexpr (EPI != EPI_GEGLU_FWD) return launch_x3_cols<BM, BN, BK, D, A_KC, B_KC, EPI, false>(g, e, split_k, st);
}

// ------------------------------------------------------------------ few tiles
// 32x32 results (32x32 pairs of u and w columns for the gated inputs) per workgroup of WK wavefronts, float32 matrix
// instructions.  At 64 tokens a product is one round trip to memory and a short chain of products, and the code of the
// launch is read for the first time as often as not, so: every wavefront takes its own batches of 32 k straight into registers
// in the order of the instruction's operands, the next batch on its way (no staging, no barrier), the operands of the
// epilogue are requested before the products, the wavefronts' sums meet in LDS once, in pairs, and all of them
// share the epilogue.  (The kernel it replaced staged through LDS and left the epilogue, a branch an element, to one of
// four wavefronts.)  Layer of d 64, 64 tokens: its 12 products 132 -> 86 us, 140 -> 104 us in all; dn2 of d 768, 200 tokens
// (k 4096) 66 -> 42 us.  Eight wavefronts from 128 k on: with fewer k some of them would have nothing to do.
// A wavefront keeps the two halves of its batches apart, so that no more than 16 k of a batch follow one another in a sum:
// with one accumulator the weight gradients over 64 tokens had 2.5e-7 of error, now 2.2e-7.
// One workgroup has a compute unit, hence two wavefronts a SIMD: left to aim at four, the compiler holds back the loads
// (200 x 768 x 2048 with residual 26 us, 22 like this).
template <int WK, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(WK * 64) __attribute__((amdgpu_waves_per_eu(WK / 4, 2))) void gemm_f32_small_kernel(GemmDesc g, GemmEpi e) {
  constexpr bool GF = EPI == EPI_GEGLU_FWD;
  constexpr int NJ = GF ? 2 : 1, U = 4;  // column tiles; steps of 8 k in a batch
  __shared__ float part[WK][NJ][32][32];
  const int tid = threadIdx.x, lane = tid & 63, g2 = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;  // (GF: n0 counts hidden units)
  const int lda = g.seg[0].lda, ldb = g.seg[0].ldb, N = GF ? g.N >> 1 : g.N;

  // epilogue: thread -> column tid % 32, rows tid / 32 + (threads / 32) * i
  constexpr int RS = WK * 2, NE = 32 / RS;
  const int en = n0 + (tid & 31), er = m0 + (tid >> 5);
  const bool add = EPI == EPI_SPLIT_F32 && e.accumulate;
  float xa[NE], xb[NE];
  size_t eo[NE];
  float* out0 = (float*)e.out0;
  if constexpr (EPI == EPI_SPLIT_F32) {
    const int which = en / e.split_n;
    out0 = (float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2);
    for (int i = 0; i < NE; ++i) eo[i] = (size_t)(er + RS * i) * e.ld0 + (en - which * e.split_n);
  } else {
    for (int i = 0; i < NE; ++i) eo[i] = (size_t)(er + RS * i) * e.ld0 + en;
  }
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const bool ok = er + RS * i < g.M && en < N;
    xa[i] = xb[i] = 0.f;
    if constexpr (EPI == EPI_RESID || EPI == EPI_GEGLU_BWD) {
      const size_t o = ok ? (size_t)(er + RS * i) * (e.ld_aux ? e.ld_aux : e.ld0) + en : 0;
      xa[i] = ((const float*)e.aux0)[o];
      if constexpr (EPI == EPI_GEGLU_BWD) xb[i] = ((const float*)e.aux1)[o];
    } else if constexpr (EPI == EPI_SPLIT_F32) {
      if (add && ok) xa[i] = out0[eo[i]];
    }
  }

  // this lane's row of A and columns of B (past the end: the last one, its results are not stored)
  const int m = m0 + l32 < g.M ? m0 + l32 : g.M - 1;
  int n[NJ];
  const float* bsrc = nullptr;  // columns from several matrices
  n[0] = n0 + l32 < N ? n0 + l32 : N - 1;
  if constexpr (GF) n[NJ - 1] = n[0];
  if constexpr (!GF && !B_KC) {
    if (g.nsrc > 1) {
      const int q = n[0] / g.nsrc_cols;
      bsrc = (const float*)(q == 0 ? g.seg[0].B : q == 1 ? g.seg[1].B : g.seg[2].B);
      n[0] -= q * g.nsrc_cols;
    }
  }
  f32x16 acc[2][NJ];  // the two halves of every batch
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[h][j][r] = 0.f;

  f32x4 va[2][U], vb[2][NJ][U];
  auto load = [&](const float* A, const float* B, const float* B1, int K, int b, f32x4 (&a)[U], f32x4 (&bb)[NJ][U])
                  __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = b * (8 * U) + u * 8 + g2 * 4;
      if constexpr (A_KC) {
        a[u] = ld4<true>(A, (size_t)m * lda + k, K - k);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) a[u][q] = A[(size_t)(k + q < K ? k + q : K - 1) * lda + m];
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float* Bj = j ? B1 : B;
        if constexpr (B_KC) {
          bb[j][u] = ld4<true>(Bj, (size_t)n[j] * ldb + k, K - k);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) bb[j][u][q] = Bj[(size_t)(k + q < K ? k + q : K - 1) * ldb + n[j]];
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[u][q] = k + q < K ? a[u][q] : 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) bb[j][u][q] = k + q < K ? bb[j][u][q] : 0.f;
      }
    }
  };
  auto mul = [&](const f32x4 (&a)[U], const f32x4 (&bb)[NJ][U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          f32x16& c = acc[u / (U / 2)][j];
          c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][q], bb[j][u][q], c, 0, 0, 0);
        }
  };
  int b0 = wave;  // batches wave, wave + WK, ... over all segments
  for (int s = 0; s < g.nseg; ++s) {
    const int K = g.seg[s].K, nb = (K + 8 * U - 1) / (8 * U);
    const float* A = (const float*)g.seg[s].A;
    const float* B = bsrc ? bsrc : (const float*)g.seg[s].B;
    const float* B1 = (const float*)g.seg[GF ? 1 : 0].B;
    int b = b0;
    if (b < nb) {
      load(A, B, B1, K, b, va[0], vb[0]);
      for (;;) {
        if (b + WK < nb) load(A, B, B1, K, b + WK, va[1], vb[1]);
        mul(va[0], vb[0]);
        b += WK;
        if (b >= nb) break;
        if (b + WK < nb) load(A, B, B1, K, b + WK, va[0], vb[0]);
        mul(va[1], vb[1]);
        b += WK;
        if (b >= nb) break;
      }
    }
    b0 = b - nb;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][j][((r >> 2) << 3) + (g2 << 2) + (r & 3)][l32] = acc[0][j][r] + acc[1][j][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int row = er + RS * i;
    auto sum = [&](int j) __attribute__((always_inline)) {
      float t[WK];
#pragma unroll
      for (int k = 0; k < WK; ++k) t[k] = part[k][j][row - m0][tid & 31];
#pragma unroll
      for (int n = WK / 2; n > 0; n /= 2)
#pragma unroll
        for (int k = 0; k < n; ++k) t[k] += t[k + n];
      return t[0];
    };
    const float v = sum(0), w = GF ? sum(NJ - 1) : 0.f;
    if (row >= g.M || en >= N) continue;
    const float mk = e.drop.on && !(EPI == EPI_RESID && e.aux_mask) ? drop_mult(e.drop, drop_row_key(e.drop, (uint32_t)row), (uint32_t)en) : 1.f;
    if constexpr (GF) {
      float gl, dgl;
      gelu_both(e.act, v, gl, dgl);
      out0[eo[i]] = w * dgl * mk;
      ((float*)e.out1)[eo[i]] = gl * mk;
      ((float*)e.out2)[eo[i]] = gl * w * mk;
    } else if constexpr (EPI == EPI_STORE) {
      out0[eo[i]] = (e.act == ACT_RELU ? fmaxf(v, 0.f) : v) * mk;
    } else if constexpr (EPI == EPI_RESID) {
      out0[eo[i]] = e.aux_mask ? (xa[i] > 0.f ? v * (e.drop.on ? e.drop.scale : 1.f) : 0.f) : v * mk + xa[i];
    } else if constexpr (EPI == EPI_GEGLU_BWD) {
      out0[eo[i]] = v * xa[i];
      ((float*)e.out1)[eo[i]] = v * xb[i];
    } else {
      out0[eo[i]] = xa[i] + v;
    }
  }
}
template <bool A_KC, bool B_KC, int EPI>
hipError_t launch_small(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  dim3 grid(ceil_div(EPI == EPI_GEGLU_FWD ? g.N / 2 : g.N, 32), ceil_div(g.M, 32));
  int K = 0;
  for (int s = 0; s < g.nseg; ++s) K += g.seg[s].K;
  if (K > 128) gemm_f32_small_kernel<8, A_KC, B_KC, EPI><<<grid, 512, 0, st>>>(g, e);
  else gemm_f32_small_kernel<4, A_KC, B_KC, EPI><<<grid, 256, 0, st>>>(g, e);
  return hipGetLastError();
}

// All sliced weight gradients of a layer in one launch: a thread adds four columns of one row over the slices, in their
// order.  Bound: bytes, the slices once, the outputs twice.  (Float atomics of the slices on the outputs took longer, and
// their order varied from run to run: layer of d 512 over 4000 tokens 893 us, 880 with this.)
struct SplitArgs {
  SplitJobs jobs;
  int first[SPLIT_JOBS];  // first block of each job
};
__global__ __launch_bounds__(256) void split_reduce_kernel(SplitArgs s) {
  int i = 0;
  while (i + 1 < s.jobs.count && (int)blockIdx.x >= s.first[i + 1]) ++i;
  const SplitJob& j = s.jobs.j[i];
  const uint32_t idx = ((blockIdx.x - (uint32_t)s.first[i]) * 256 + threadIdx.x) * 4, mn = (uint32_t)j.M * (uint32_t)j.N;
  if (idx >= mn) return;
  const uint32_t m = idx / (uint32_t)j.N, n = idx - m * (uint32_t)j.N;
  const float* p = j.part + idx;
  f32x4 acc = *reinterpret_cast<const f32x4*>(p);
#pragma unroll 8
  for (int k = 1; k < j.slices; ++k) {
    p += mn;
    const f32x4 v = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] += v[q];
  }
  uint32_t which = n / (uint32_t)j.split_n, col = n - which * (uint32_t)j.split_n;
  if (col + 4 <= (uint32_t)j.split_n) {
    typedef f32x4 __attribute__((aligned(4))) f32x4_any;  // (an output may start anywhere)
    float* o = (which == 0 ? j.out[0] : which == 1 ? j.out[1] : j.out[2]) + (size_t)m * j.ld0 + col;
    f32x4 v = *reinterpret_cast<const f32x4_any*>(o);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] += acc[q];
    *reinterpret_cast<f32x4_any*>(o) = v;
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // the four columns belong to two outputs
    if (col == (uint32_t)j.split_n) { ++which; col = 0; }
    float* o = which == 0 ? j.out[0] : which == 1 ? j.out[1] : j.out[2];
    o[(size_t)m * j.ld0 + col] += acc[q];
    ++col;
  }
}

template <int BM, int BN, int WM, int WN, int WK, int BK, bool A_KC, bool B_KC, int EPI, bool VEC>
hipError_t launch_tile(const GemmDesc& g, const GemmEpi& e, int split_k, hipStream_t st) {
  constexpr int a_fl = A_KC ? BM * (BK + 4) : BK * (BM + 8), b_fl = B_KC ? BN * (BK + 4) : BK * (BN + 8);
  constexpr int red = (WK - 1) * BM * BN;  // floats of the exchange between the k shares
  constexpr int lds = (2 * (a_fl + b_fl) > red ? 2 * (a_fl + b_fl) : red) * 4;
  auto kern = gemm_f32_kernel<BM, BN, WM, WN, WK, BK, A_KC, B_KC, EPI, VEC>;
  if constexpr (lds > 65536) {
    static std::atomic<bool> attr_set{false};  // once per instantiation; setting it twice is harmless
    if (!attr_set.load(std::memory_order_relaxed)) {
      hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (err != hipSuccess) return err;
      attr_set.store(true, std::memory_order_relaxed);
    }
  }
  dim3 grid(ceil_div(g.N, BN), ceil_div(g.M, BM), split_k);
  kern<<<grid, WM * WN * WK * 64, lds, st>>>(g, e, split_k);
  return hipGetLastError();
}

// float4 loads: every row of the operands starts on a 16-byte boundary and no slot of four lies half outside
bool vec_ok(const GemmDesc& g) {
  bool vec = g.seg[0].lda % 4 == 0 && g.seg[0].ldb % 4 == 0;
  for (int s = 0; s < (g.nsrc > 1 ? g.nsrc : g.nseg); ++s) vec = vec && ((uintptr_t)g.seg[s].B & 15) == 0;
  for (int s = 0; s < g.nseg; ++s) {
    vec = vec && ((uintptr_t)g.seg[s].A & 15) == 0;
    if (g.a_kc || g.b_kc) vec = vec && g.seg[s].K % 4 == 0;
  }
  if (!g.a_kc) vec = vec && g.M % 4 == 0;
  if (!g.b_kc) vec = vec && g.N % 4 == 0;
  return vec;
}
// Weight gradients: few tiles, long k.  Slices of at least 256 k until one workgroup of 128x128 tiles, or two of 64x64,
// per compute unit are busy (two of 128x128: the sum of their slices takes half as long again; layer of d 768, 4000 tokens 1914
// against 1886 us, d 512 840 against 833).
int wgrad_slices(const GemmDesc& g, bool& big) {
  const int64_t t128 = (int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 128);
  const int64_t t64 = (int64_t)ceil_div(g.M, 64) * ceil_div(g.N, 64), K = g.seg[0].K;
  big = t128 * (K / 256) >= 256;
  const int64_t t = big ? t128 : t64;
  return (int)std::max<int64_t>(1, std::min<int64_t>(K / 256, ((big ? 256 : 512) + t - 1) / t));
}

template <bool A_KC, bool B_KC, int EPI>
hipError_t launch_kind(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  if (!vec_ok(g)) return launch_tile<64, 64, 2, 1, 2, 32, A_KC, B_KC, EPI, false>(g, e, 1, st);
  const int64_t t128 = (int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 128);
  const int64_t t64 = (int64_t)ceil_div(g.M, 64) * ceil_div(g.N, 64);
  if constexpr (EPI == EPI_SPLIT_F32) {
    if (e.aux0 && e.accumulate && g.seg[0].K >= 512) {
      bool big;
      const int sk = wgrad_slices(g, big);
      if (big) return launch_x3<128, 128, 16, 2, A_KC, B_KC, EPI>(g, e, sk, st);
      return launch_tile<64, 64, 2, 1, 2, 32, A_KC, B_KC, EPI, true>(g, e, sk, st);
    }
  }
  int64_t K = 0;
  for (int i = 0; i < g.nseg; ++i) K += g.seg[i].K;
  // Split operands from about as many tiles as keep the conversion off the critical path; us for native / split:
  //   128x128, 4000 tokens: qkv of d 512 (288 tiles) 62 / 57, dn2 of d 768 (192) 247 / 201, wi of d 768 (1024) 231 / 187;
  //            with 128 tiles (4000 x 512 x 2048) 85 / 104, but 80 on 64x64 ones;
  //   64x64:   1024 x 512 x 2048 (128 tiles) 57 / 46, 200 x 2048 x 768 (128) 27 / 23; with n-contiguous weights no faster
  //            (800 x 768 x 2048 61 / 61, 1200 x 2304 x 768 54 / 60) nor over few tokens (gradient of 768 x 4096 over 200
  //            32 / 35, over 400 42 / 52): their sums lose half as much.
  // The gated inputs need 64 columns a wavefront, which 64x64 tiles of four do not have.  32x32 tiles with the
  // reduction over the wavefronts where even the 64x64 ones leave half the chip idle.  From 64 of those on the 32x32 ones are two
  // rounds of workgroups: products with k-contiguous weights (gradients of the norms' outputs) take 32x64 tiles instead, one
  // round, staged, every k-tile shared by eight wavefronts: 400 x 768, k 4096 80 -> 63 us, k 2304 47 -> 40, 300 x 1024, k 8192
  // 150 -> 116, 640 x 512, k 2048 46 -> 36; one round of 32x32: 320 x 768, k 4096 42, with 32x64 66.  The others are as fast either
  // way, and gated-GELU backward loses (300 x 1024, k 512: 16 and 29): one of the eight wavefronts does the epilogue.
  if (t128 >= 192 && K >= 384) return launch_x3<128, 128, 16, 2, A_KC, B_KC, EPI>(g, e, 1, st);
  if (t64 >= 128) {
    if constexpr (EPI == EPI_GEGLU_FWD) return launch_tile<64, 64, 2, 1, 2, 32, A_KC, B_KC, EPI, true>(g, e, 1, st);
    else return launch_x3<64, 64, 32, 3, A_KC, B_KC, EPI>(g, e, 1, st);
  }
  if constexpr (EPI == EPI_STORE && B_KC)
    if (t64 > 64) return launch_tile<32, 64, 1, 1, 8, 64, A_KC, B_KC, EPI, true>(g, e, 1, st);
  return launch_small<A_KC, B_KC, EPI>(g, e, st);
}

}  // namespace

int gemm_f32_slices(const GemmDesc& g, const GemmEpi& e) {
  if (!gemm_f32_supported(g, e) || e.kind != EPI_SPLIT_F32 || !e.accumulate || g.seg[0].K < 512 || !vec_ok(g)) return 1;
  bool big;
  return wgrad_slices(g, big);
}

hipError_t launch_split_reduce(const SplitJobs& jobs, hipStream_t st) {
  int blocks = 0;
  SplitArgs s;
  for (int i = 0; i < jobs.count; ++i) {
    if (jobs.j[i].N % 4 != 0 || (int64_t)jobs.j[i].M * jobs.j[i].N >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    s.first[i] = blocks;
    blocks += ceil_div((int64_t)jobs.j[i].M * jobs.j[i].N / 4, 256);
  }
  if (blocks == 0) return hipSuccess;
  s.jobs = jobs;
  split_reduce_kernel<<<blocks, 256, 0, st>>>(s);
  return hipGetLastError();
}

bool gemm_f32_supported(const GemmDesc& g, const GemmEpi& e) {
  if (g.in_type != IN_F32 || g.nseg < 1 || g.nseg > 3 || g.ngroups > 1 || e.out_type != IN_F32) return false;
  if (g.M < 1 || g.N < 1) return false;
  for (int s = 0; s < g.nseg; ++s)
    if (g.seg[s].K < 1 || g.seg[s].lda != g.seg[0].lda || g.seg[s].ldb != g.seg[0].ldb) return false;
  if (ceil_div(g.M, 32) > 65535) return false;  // grid.y
  if (g.nsrc > 1 && (g.nseg != 1 || g.nsrc > 3 || g.b_kc || g.nsrc_cols % 4 != 0 || g.nsrc * g.nsrc_cols != g.N)) return false;
  switch (e.kind) {
    case EPI_STORE: return g.a_kc != 0;
    case EPI_RESID: return g.a_kc != 0 && e.aux_type == IN_F32;
    case EPI_GEGLU_FWD: return g.a_kc != 0 && !g.b_kc && g.nsrc == 2 && g.nsrc_cols % 32 == 0;
    case EPI_GEGLU_BWD: return g.a_kc != 0 && g.b_kc != 0 && e.aux_type == IN_F32;
    case EPI_SPLIT_F32: return !g.a_kc && !g.b_kc && g.nseg == 1;
    default: return false;
  }
}

hipError_t launch_gemm_f32(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  switch (e.kind) {
    case EPI_STORE:
      return g.b_kc ? launch_kind<true, true, EPI_STORE>(g, e, st) : launch_kind<true, false, EPI_STORE>(g, e, st);
    case EPI_RESID:
      return g.b_kc ? launch_kind<true, true, EPI_RESID>(g, e, st) : launch_kind<true, false, EPI_RESID>(g, e, st);
    case EPI_GEGLU_FWD: return launch_kind<true, false, EPI_GEGLU_FWD>(g, e, st);
    case EPI_GEGLU_BWD: return launch_kind<true, true, EPI_GEGLU_BWD>(g, e, st);
    case EPI_SPLIT_F32: return launch_kind<false, false, EPI_SPLIT_F32>(g, e, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace t5mi
