// float32 attention on the matrix units (v_mfma_f32_32x32x2_f32), forward and backward, with the relative-position
// bias, causal masking and dropout of the probabilities, any lengths, heads of up to 128 channels.  The scores never
// leave registers.
//
// A wavefront owns 32 queries (forward, dq: lane = query, S^T = K Q^T) or 32 keys (dk/dv: lane = key, S = Q K^T).  In
// the 32x32 result layout register r of lane half g is row 8*(r/4) + 4*g + r%4, and one float32 MFMA contracts two
// values, one from each lane half: register r of the probabilities is therefore, as it stands, the operand of an MFMA
// that contracts rows 8*(r/4) + r%4 and + 4, and the other operand is one column read per lane from the tile in LDS.
//
// Bound: the float32 matrix rate (157 TFLOP/s nominal): 32 keys x 32 queries of 64 channels are 64 MFMAs of 64 cycles in
// the forward against some 200 vector instructions.  Tiles of 32 rows travel through registers while the previous
// tile is used; rows past the end repeat the last one with probability zero (where that row is not finite, what it
// contributes to is not either) and channels past d_kv are zeros, so no shape needs another path.
//
// Causal rows and values that are not finite: a masked element's zero times an infinity is not zero, so the tiles that the
// mask cuts through are looked over.  A value row that is not finite reaches only the queries at or after it; a query row
// (or its output gradient) only the keys at or before it, whose dk and dv are NaN then.  dq needs no such care: a key that
// is not finite makes dk of every earlier position not finite, and with it their dx.
//
// A bias table masks with -inf or with the lowest float32, which times log2(e) overflows to -inf, and a whole tile may be
// masked so: scores stay in natural units until the maximum (forward) or the log-sum (backward) has been taken off them,
// and the running maximum may be -inf.
//
// The bias gradient (dq) adds each ds element to its diagonal in LDS and one global atomic per diagonal and workgroup
// follows; one global atomic per element took longer than everything else.
#include "kernels.h"

namespace t5mi {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// A tile of 32 rows x DKP channels on its way from global memory to LDS (row stride LD floats).  Rows past the end
// repeat the last one (their scores are masked), channels past d_kv become zeros on the way into LDS: with VEC the
// loads carry no branch, around which the compiler would wait for them on the spot.
template <int DKP, int NT, bool VEC>
struct Tile32 {
  static constexpr int N = 32 * DKP / 4 / NT, W = DKP / 4;
  f32x4 v[N];
  __device__ __forceinline__ void load(const float* src, size_t ld, int rows, int dk, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = tid + i * NT, row = q / W < rows ? q / W : rows - 1, c = (q % W) * 4;
      const float* p = src + (size_t)row * ld;
      if constexpr (VEC) {
        v[i] = *reinterpret_cast<const f32x4*>(p + (c < dk ? c : 0));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = p[c + e < dk ? c + e : 0];
      }
    }
  }
  template <int LD>
  __device__ __forceinline__ void put(float* dst, int dk, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = tid + i * NT, c = (q % W) * 4;
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = c + e < dk ? v[i][e] : 0.f;
      *reinterpret_cast<f32x4*>(dst + (q / W) * LD + c) = x;
    }
  }
  __device__ __forceinline__ bool finite(int i) const {  // slot i of this thread
    bool ok = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) ok &= __builtin_fabsf(v[i][e]) <= 3.402823466e38f;
    return ok;
  }
  // 1 in bad[row] for every row of the tile that holds a value that is not finite
  __device__ __forceinline__ void mark(int* bad, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (!finite(i)) bad[(tid + i * NT) / W] = 1;
  }
  // clears the rows of `bad` in LDS
  template <int LD>
  static __device__ __forceinline__ void clear_rows(float* dst, uint32_t bad, int tid) {
#pragma unroll 1
    for (int q = tid; q < 32 * W; q += NT)
      if ((bad >> (q / W)) & 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[(q / W) * LD + (q % W) * 4 + e] = 0.f;
  }
};
// One row's channels as MFMA operands: group s of 8 channels gives this lane half channels 8s + 4g .. + 3.
template <int DKP, bool VEC>
__device__ __forceinline__ void load_row(f32x4 (&f)[DKP / 8], const float* row, int dk, int g) {
#pragma unroll
  for (int s = 0; s < DKP / 8; ++s) {
    const int c = s * 8 + g * 4;
    f32x4 x;
    if constexpr (VEC) x = *reinterpret_cast<const f32x4*>(row + (c < dk ? c : 0));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (!VEC) x[e] = row[c + e < dk ? c + e : 0];
      x[e] = c + e < dk ? x[e] : 0.f;
    }
    f[s] = x;
  }
}
// acc += T F^T for the 32 rows of a tile (MFMA rows) and the rows held as operands (MFMA columns)
template <int DKP, int LD>
__device__ __forceinline__ void mul_rows(f32x16& acc, const float* tile, const f32x4 (&f)[DKP / 8], int lane) {
  const float* p = tile + (lane & 31) * LD + (lane >> 5) * 4;
  f32x4 a[2];  // (requested one group ahead of its products)
  a[0] = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
  for (int s = 0; s < DKP / 8; ++s) {
    if (s + 1 < DKP / 8) a[(s + 1) & 1] = *reinterpret_cast<const f32x4*>(p + (s + 1) * 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s & 1][e], f[s][e], acc, 0, 0, 0);
  }
}
// acc[ct] += T^T P for a tile (channels become MFMA rows, its 32 rows are contracted) and P in the result layout
template <int CT, int LD>
__device__ __forceinline__ void mul_cols(f32x16 (&acc)[CT], const float* tile, const f32x16& p, int lane) {
  const float* t = tile + (lane >> 5) * 4 * LD + (lane & 31);
  float a[2][4][CT];  // (four rows' columns, requested one group ahead of their products)
  auto columns = [&](int rq) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) a[rq & 1][e][ct] = t[(rq * 8 + e) * LD + ct * 32];
  };
  columns(0);
#pragma unroll
  for (int rq = 0; rq < 4; ++rq) {
    if (rq + 1 < 4) columns(rq + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        acc[ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[rq & 1][e][ct], p[rq * 4 + e], acc[ct], 0, 0, 0);
  }
}
__device__ __forceinline__ void clear(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}
// Result columns of a wavefront (one row of the output per lane): channels ct*32 + 8*(r/4) + 4*g + r%4.
template <int CT, bool VEC>
__device__ __forceinline__ void store_cols(float* row, const f32x16 (&acc)[CT], float f, int dk, int g) {
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const int c = ct * 32 + rq * 8 + g * 4;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = acc[ct][rq * 4 + e] * f;
      if constexpr (VEC) {
        if (c < dk) *reinterpret_cast<f32x4*>(row + c) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < dk) row[c + e] = o[e];
      }
    }
}

// mul_cols for a tile whose rows some lanes must not see (row j counts for a lane where j <= last), without multiplying
// what they must not see: a zero probability times an infinity is not zero.  Plain multiply-adds, for the causal
// forward's diagonal tiles that hold a value that is not finite (a padding position's, say).  Rolled, so that it holds
// one row's operands: unrolled it took the whole kernel from two wavefronts per SIMD to one.
template <int CT, int LD>
__device__ __forceinline__ void mul_cols_masked(f32x16 (&acc)[CT], const float* tile, const f32x16& p, int last, int lane) {
  const int g = lane >> 5;
#pragma unroll 1
  for (int j = 0; j < 32; ++j) {
    const float mine = p[(j >> 3) * 4 + (j & 3)], other = __shfl_xor(mine, 32, 64);
    const float pj = ((j >> 2) & 1) == g ? mine : other;
    const float* t = tile + j * LD + g * 4;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(t + ct * 32 + rq * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[ct][rq * 4 + e] = j <= last ? fmaf(pj, v[e], acc[ct][rq * 4 + e]) : acc[ct][rq * 4 + e];
      }
  }
}

// ---- forward.  One workgroup per (b, h, NW*32 queries).  Up to 64 channels two wavefronts share a SIMD (three up to 32):
// one hides the other's softmax arithmetic and the barriers around the tiles (one less where a single wavefront loads whole
// tiles element by element, which would spill).
template <int DKP, int NW, bool VEC, bool CAUSAL>
__global__ __launch_bounds__(NW * 64, DKP == 128 ? 1 : (DKP == 32 ? 3 : 2) - (NW == 1 && !VEC))
void attn_fwd_f32_kernel(AttnIO io, const float* __restrict__ diag, float* __restrict__ c, float* __restrict__ lse,
                         AttnDims a, int n_tiles) {
  constexpr int CT = DKP / 32, KL = DKP + 4, VL = DKP + 8, NT = NW * 64;
  __shared__ __attribute__((aligned(16))) float Kt[32 * KL];
  __shared__ __attribute__((aligned(16))) float Vt[32 * VL];
  __shared__ int v_bad;  // the tile holds a value that is not finite
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, wave = tid >> 6;
  const int S = a.S, Sk = a.Sk, I = a.H * a.dk;
  int qt = blockIdx.x % n_tiles;
  const int bh = blockIdx.x / n_tiles, h = bh % a.H, b = bh / a.H;
  if (CAUSAL) qt = n_tiles - 1 - qt;  // long rows first
  const int i0 = qt * NW * 32, iw = i0 + wave * 32, i = iw + (lane & 31), il = i < S ? i : S - 1;
  const float* kb = (const float*)io.k + (size_t)b * Sk * io.ldkv + h * a.dk;
  const float* vb = (const float*)io.v + (size_t)b * Sk * io.ldkv + h * a.dk;
  const float* dg = a.bias ? diag + (size_t)h * (2 * S - 1) + (S - 1) - il : nullptr;  // dg[j] = bias(j - i)
  f32x4 q[DKP / 8];
  load_row<DKP, VEC>(q, (const float*)io.q + ((size_t)b * S + il) * io.ldq + h * a.dk, a.dk, g);
  uint32_t k1 = 0;
  if (a.drop.on) k1 = drop_row_pre(drop_row_key(a.drop, (uint32_t)(((size_t)b * a.H + h) * S + il)));
  f32x16 o[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) clear(o[ct]);
  float m = -INFINITY, l = 0.f;
  const int keys = CAUSAL ? (i0 + NW * 32 < S ? i0 + NW * 32 : S) : Sk;
  const int my_keys = CAUSAL ? (iw + 32 < keys ? iw + 32 : keys) : Sk;  // keys this wavefront's queries see
  Tile32<DKP, NT, VEC> tk, tv;
  tk.load(kb, io.ldkv, Sk, a.dk, tid);
  tv.load(vb, io.ldkv, Sk, a.dk, tid);
  for (int j0 = 0; j0 < keys; j0 += 32) {
    __syncthreads();  // the tile before this one has been used
    bool bad = false;
    if (CAUSAL && j0 + 31 > i0) {  // (the tiles that a mask cuts through)
      if (tid == 0) v_bad = 0;
#pragma unroll
      for (int q = 0; q < Tile32<DKP, NT, VEC>::N; ++q) bad |= !tv.finite(q);
    }
    tk.template put<KL>(Kt, a.dk, tid);
    tv.template put<VL>(Vt, a.dk, tid);
    __syncthreads();
    if (CAUSAL && j0 + 31 > i0) {
      if (bad) v_bad = 1;
      __syncthreads();
    }
    // (requested before the next tile: loads return in order, and these are needed first)
    float bias[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      bias[r] = a.bias ? dg[j < Sk ? j : Sk - 1] : 0.f;
    }
    if (j0 + 32 < keys) {
      tk.load(kb + (size_t)(j0 + 32) * io.ldkv, io.ldkv, Sk - j0 - 32, a.dk, tid);
      tv.load(vb + (size_t)(j0 + 32) * io.ldkv, io.ldkv, Sk - j0 - 32, a.dk, tid);
    }
    if (j0 >= my_keys) continue;  // (uniform in the wavefront; the barriers are at the top of the loop)
    f32x16 s;
    clear(s);
    mul_rows<DKP, KL>(s, Kt, q, lane);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      float x = fmaf(s[r], a.scale, bias[r]);
      if ((CAUSAL && j > i) || j >= Sk) x = -INFINITY;
      s[r] = x;
      mx = fmaxf(mx, x);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), base = mn == -INFINITY ? 0.f : mn;  // (no visible key so far: every p and l are zero)
    const float alpha = __builtin_amdgcn_exp2f((m - base) * kLog2e);
    m = mn;
    float ls = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      const float p = __builtin_amdgcn_exp2f((s[r] - base) * kLog2e);
      ls += p;  // the normaliser is that of the undropped probabilities
      s[r] = a.drop.on ? (drop_keep16(a.drop, k1 ^ (uint32_t)j) ? p : 0.f) : p;
    }
    l = l * alpha + ls;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
    if constexpr (CAUSAL) {
      if (j0 + 31 > iw && v_bad) {
        mul_cols_masked<CT, VL>(o, Vt, s, i - j0, lane);
        continue;
      }
    }
    mul_cols<CT, VL>(o, Vt, s, lane);
  }
  l += __shfl_xor(l, 32, 64);
  if (i < S) {
    store_cols<CT, VEC>(c + ((size_t)b * S + i) * I + h * a.dk, o, (a.drop.on ? a.drop.scale : 1.f) / l, a.dk, g);
    if (g == 0) lse[((size_t)b * a.H + h) * S + i] = fmaf(__builtin_amdgcn_logf(l), kLn2, m);
  }
}

// ---- dq, dvec = rowsum(dO * O) and the per-diagonal bias gradient.  Ownership as in the forward.
// Dynamic LDS: with bias, one float per diagonal the workgroup can touch (S + NW*32 - 1).
template <int DKP, int NW, bool VEC>
__global__ __launch_bounds__(NW * 64, DKP == 32 || (DKP == 64 && NW > 1) ? 2 : 1)
void attn_bwd_dq_f32_kernel(AttnIO io, const float* __restrict__ o, const float* __restrict__ dout,
                            const float* __restrict__ diag, const float* __restrict__ lse, float* __restrict__ dvec,
                            float* __restrict__ ddiag, AttnDims a, int n_tiles) {
  constexpr int CT = DKP / 32, LD = DKP + 4, NT = NW * 64;
  __shared__ __attribute__((aligned(16))) float Kt[32 * LD];
  __shared__ __attribute__((aligned(16))) float Vt[32 * LD];
  extern __shared__ float win[];  // diagonal j - i sits at j - i + i0 + NW*32 - 1
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, wave = tid >> 6;
  const int S = a.S, Sk = a.Sk, I = a.H * a.dk;
  int qt = blockIdx.x % n_tiles;
  const int bh = blockIdx.x / n_tiles, h = bh % a.H, b = bh / a.H;
  if (a.causal) qt = n_tiles - 1 - qt;
  const int i0 = qt * NW * 32, iw = i0 + wave * 32, i = iw + (lane & 31), il = i < S ? i : S - 1;
  const float* kb = (const float*)io.k + (size_t)b * Sk * io.ldkv + h * a.dk;
  const float* vb = (const float*)io.v + (size_t)b * Sk * io.ldkv + h * a.dk;
  const float* dg = a.bias ? diag + (size_t)h * (2 * S - 1) + (S - 1) - il : nullptr;
  const int nwin = S + NW * 32 - 1;
  if (a.bias)
    for (int t = tid; t < nwin; t += NT) win[t] = 0.f;
  const size_t srow = ((size_t)b * a.H + h) * S + il;
  f32x4 q[DKP / 8], d[DKP / 8];
  float dsum = 0.f;
  {
    f32x4 x[DKP / 8];
    load_row<DKP, VEC>(q, (const float*)io.q + ((size_t)b * S + il) * io.ldq + h * a.dk, a.dk, g);
    load_row<DKP, VEC>(d, dout + ((size_t)b * S + il) * I + h * a.dk, a.dk, g);
    load_row<DKP, VEC>(x, o + ((size_t)b * S + il) * I + h * a.dk, a.dk, g);
#pragma unroll
    for (int s = 0; s < DKP / 8; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) dsum = fmaf(d[s][e], x[s][e], dsum);
  }
  dsum += __shfl_xor(dsum, 32, 64);
  if (g == 0 && i < S) dvec[srow] = dsum;
  const float lse_q = lse[srow];
  uint32_t k1 = 0;
  if (a.drop.on) k1 = drop_row_pre(drop_row_key(a.drop, (uint32_t)srow));
  f32x16 dq[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) clear(dq[ct]);
  const int keys = a.causal ? (i0 + NW * 32 < S ? i0 + NW * 32 : S) : Sk;
  const int my_keys = a.causal ? (iw + 32 < keys ? iw + 32 : keys) : Sk;
  Tile32<DKP, NT, VEC> tk, tv;
  tk.load(kb, io.ldkv, Sk, a.dk, tid);
  tv.load(vb, io.ldkv, Sk, a.dk, tid);
  for (int j0 = 0; j0 < keys; j0 += 32) {
    __syncthreads();
    tk.template put<LD>(Kt, a.dk, tid);
    tv.template put<LD>(Vt, a.dk, tid);
    __syncthreads();
    float bias[16];  // (requested before the next tile, as in the forward)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      bias[r] = a.bias ? dg[j < Sk ? j : Sk - 1] : 0.f;
    }
    if (j0 + 32 < keys) {
      tk.load(kb + (size_t)(j0 + 32) * io.ldkv, io.ldkv, Sk - j0 - 32, a.dk, tid);
      tv.load(vb + (size_t)(j0 + 32) * io.ldkv, io.ldkv, Sk - j0 - 32, a.dk, tid);
    }
    if (j0 >= my_keys) continue;
    f32x16 s, dp;
    clear(s);
    clear(dp);
    mul_rows<DKP, LD>(s, Kt, q, lane);
    mul_rows<DKP, LD>(dp, Vt, d, lane);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      const float p = __builtin_amdgcn_exp2f((fmaf(s[r], a.scale, bias[r]) - lse_q) * kLog2e);
      float x = dp[r];
      if (a.drop.on) x = drop_keep16(a.drop, k1 ^ (uint32_t)j) ? x * a.drop.scale : 0.f;
      const float ds = p * (x - dsum);
      const bool ok = i < S && j < Sk && !(a.causal && j > i);
      s[r] = ok ? ds : 0.f;
      if (a.bias && ok) atomicAdd(&win[j - i + i0 + NW * 32 - 1], ds);
    }
    mul_cols<CT, LD>(dq, Kt, s, lane);
  }
  if (i < S) store_cols<CT, VEC>((float*)io.dq + ((size_t)b * S + i) * io.lddq + h * a.dk, dq, a.scale, a.dk, g);
  if (a.bias) {
    __syncthreads();
    float* dd = ddiag + (size_t)h * (2 * S - 1) + (S - 1) - (i0 + NW * 32 - 1);
    for (int t = tid; t < nwin; t += NT) {
      const float x = win[t];
      // (slots of queries past the end lie below the first diagonal; they are zero)
      if (t - (i0 + NW * 32 - 1) > -S && x != 0.f) unsafeAtomicAdd(dd + t, x);
    }
  }
}

// ---- dk and dv.  One workgroup per (b, h, NW*32 keys); lane = key.
template <int DKP, int NW, bool VEC, bool CAUSAL>
__global__ __launch_bounds__(NW * 64, DKP == 32 || (DKP == 64 && NW == 4) ? 2 : 1)
void attn_bwd_dkv_f32_kernel(AttnIO io, const float* __restrict__ dout, const float* __restrict__ diag,
                             const float* __restrict__ lse, const float* __restrict__ dvec, AttnDims a, int n_tiles) {
  constexpr int CT = DKP / 32, LD = DKP + 4, NT = NW * 64;
  __shared__ __attribute__((aligned(16))) float Qt[32 * LD];
  __shared__ __attribute__((aligned(16))) float Dt[32 * LD];
  __shared__ float row_l[32], row_d[32];     // lse and dvec of the tile's queries
  __shared__ uint32_t row_k[32];             // their dropout row keys
  // tiles that the mask cuts through: not zero where q or dO of the query is not finite, and the last such query
  __shared__ int row_bad[NW * 32];
  int last_bad = -1;
  typedef Tile32<DKP, NT, VEC> Tile;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, wave = tid >> 6;
  const int S = a.S, Sk = a.Sk, I = a.H * a.dk;
  const int kt = blockIdx.x % n_tiles, bh = blockIdx.x / n_tiles, h = bh % a.H, b = bh / a.H;
  const int jw = kt * NW * 32 + wave * 32, j = jw + (lane & 31), jl = j < Sk ? j : Sk - 1;
  const float* qb = (const float*)io.q + (size_t)b * S * io.ldq + h * a.dk;
  const float* db = dout + (size_t)b * S * I + h * a.dk;
  const float* dg = a.bias ? diag + (size_t)h * (2 * S - 1) + (S - 1) + jl : nullptr;  // dg[-i] = bias(j - i)
  const size_t srow = ((size_t)b * a.H + h) * S;
  f32x4 k[DKP / 8], v[DKP / 8];
  load_row<DKP, VEC>(k, (const float*)io.k + ((size_t)b * Sk + jl) * io.ldkv + h * a.dk, a.dk, g);
  load_row<DKP, VEC>(v, (const float*)io.v + ((size_t)b * Sk + jl) * io.ldkv + h * a.dk, a.dk, g);
  f32x16 dk[CT], dv[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) { clear(dk[ct]); clear(dv[ct]); }
  const int ibeg = CAUSAL ? kt * NW * 32 : 0;  // a multiple of 32
  Tile tq, td;
  tq.load(qb + (size_t)ibeg * io.ldq, io.ldq, S - ibeg, a.dk, tid);
  td.load(db + (size_t)ibeg * I, I, S - ibeg, a.dk, tid);
  float rl = 0.f, rd = 0.f;  // lse and dvec of query i0 + tid of the tile to come (first 32 threads)
  auto load_consts = [&](int i0) __attribute__((always_inline)) {
    const int i = i0 + (tid & 31) < S ? i0 + (tid & 31) : S - 1;
    rl = lse[srow + i];
    rd = dvec[srow + i];
  };
  load_consts(ibeg);
  if (CAUSAL && tid < NW * 32) row_bad[tid] = 0;
  for (int i0 = ibeg; i0 < S; i0 += 32) {
    __syncthreads();
    const bool cut = CAUSAL && i0 < ibeg + NW * 32;  // some key of the workgroup comes after some query
    int* bad_row = row_bad + (i0 - ibeg);
    if (cut) {
      tq.mark(bad_row, tid);
      td.mark(bad_row, tid);
    }
    tq.template put<LD>(Qt, a.dk, tid);
    td.template put<LD>(Dt, a.dk, tid);
    float bias[16];  // (requested before the next tile, as in the forward)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      bias[r] = a.bias ? dg[-(i < S ? i : S - 1)] : 0.f;
    }
    if (tid < 32) {
      row_l[tid] = rl;
      row_d[tid] = rd;
      if (a.drop.on) row_k[tid] = drop_row_pre(drop_row_key(a.drop, (uint32_t)(srow + (i0 + tid < S ? i0 + tid : S - 1))));
    }
    __syncthreads();
    if (cut) {
      const uint32_t bad = (uint32_t)__ballot(bad_row[lane & 31] != 0);  // (the same in every wavefront)
      if (bad) {  // such a query takes no part in the products; the keys that see it are marked
        Tile::template clear_rows<LD>(Qt, bad, tid);
        Tile::template clear_rows<LD>(Dt, bad, tid);
        if (tid < 32 && bad_row[tid]) {
          row_l[tid] = INFINITY;
          row_d[tid] = 0.f;
        }
        last_bad = i0 + 31 - __builtin_clz(bad);
        __syncthreads();
      }
    }
    if (i0 + 32 < S) {
      tq.load(qb + (size_t)(i0 + 32) * io.ldq, io.ldq, S - i0 - 32, a.dk, tid);
      td.load(db + (size_t)(i0 + 32) * I, I, S - i0 - 32, a.dk, tid);
      load_consts(i0 + 32);
    }
    if (CAUSAL && i0 + 31 < jw) continue;  // every query of the tile comes before this wavefront's keys
    f32x16 s, dp;
    clear(s);
    clear(dp);
    mul_rows<DKP, LD>(s, Qt, k, lane);
    mul_rows<DKP, LD>(dp, Dt, v, lane);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int il = ((r >> 2) << 3) + (g << 2) + (r & 3), i = i0 + il;
      const bool ok = i < S && j < Sk && !(CAUSAL && j > i);
      const float p = ok ? __builtin_amdgcn_exp2f((fmaf(s[r], a.scale, bias[r]) - row_l[il]) * kLog2e) : 0.f;
      float mk = 1.f;
      if (a.drop.on) mk = drop_keep16(a.drop, row_k[il] ^ (uint32_t)j) ? a.drop.scale : 0.f;
      s[r] = p * mk;
      dp[r] = ok ? p * (dp[r] * mk - row_d[il]) : 0.f;
    }
    mul_cols<CT, LD>(dv, Dt, s, lane);
    mul_cols<CT, LD>(dk, Qt, dp, lane);
  }
  if (j < Sk) {
    const float f = CAUSAL && j <= last_bad ? __builtin_nanf("") : 1.f;
    store_cols<CT, VEC>((float*)io.dk + ((size_t)b * Sk + j) * io.lddkv + h * a.dk, dk, a.scale * f, a.dk, g);
    store_cols<CT, VEC>((float*)io.dv + ((size_t)b * Sk + j) * io.lddkv + h * a.dk, dv, f, a.dk, g);
  }
}

bool vec_ok(const AttnIO& io, const AttnDims& a, const void* c, const void* dc) {
  const uintptr_t all = (uintptr_t)io.q | (uintptr_t)io.k | (uintptr_t)io.v | (uintptr_t)io.dq | (uintptr_t)io.dk |
                        (uintptr_t)io.dv | (uintptr_t)c | (uintptr_t)dc;
  return (all & 15) == 0 && a.dk % 4 == 0 && io.ldq % 4 == 0 && io.ldkv % 4 == 0 && io.lddq % 4 == 0 && io.lddkv % 4 == 0;
}

// Channels are rounded up to 32, 64 or 128, with float4 loads (VEC) or element loads.  Against the row-at-a-time kernels,
// forward + backward at 12 x 250 tokens, 6 heads: 5 channels 373 -> 147 us, 18 836 -> 150, 50 2003 -> 197, 66 2743 -> 332 (5
// channels in the 128-channel tiles: 438).  Those kernels stay ahead only with 5 to 18 channels and some 100 rows in all
// (2 x 33 tokens), by up to 5 us in the backward.
//
// Wavefronts per workgroup, which share each K/V (or Q/dO) tile: one where a sequence has no more than 32 rows, two up to
// 64, then four: the second workgroup of two wavefronts on a compute unit may land on the SIMDs of the first and leave the
// other two idle.  Forward, 16 x 250 tokens, 6 heads of 64: 48 us with two, 32 with four; 12 heads 53 and 51.  Backward at
// 8 x 500, 12 heads: 421 us with two in dk/dv, 380 with four.  dq adds into one window in LDS, where four wavefronts get
// into each other's way (1 x 250, 6 heads: backward 109 us with two in dq, 130 with four; 8 x 500, 12 heads 375 and 417),
// so it takes four only where two would make between one and two workgroups a unit (16 x 250, 6 heads: 151 and 135;
// 8 heads 153 and 137).
//
// Registers: with two wavefronts per SIMD asked for, the accumulators stay out of the accumulation registers, from which
// the element loops would copy them (8 x 500, causal: backward 398 -> 344 us).
template <int DKP, bool VEC, bool CAUSAL>
hipError_t launch_fwd_form(const AttnIO& io, const float* diag, float* c, float* lse, const AttnDims& a, hipStream_t st) {
  const int bh = a.B * a.H, nt = ceil_div(a.S, 128);
  if (a.S <= 32) attn_fwd_f32_kernel<DKP, 1, VEC, CAUSAL><<<bh, 64, 0, st>>>(io, diag, c, lse, a, 1);
  else if (a.S <= 64) attn_fwd_f32_kernel<DKP, 2, VEC, CAUSAL><<<bh, 128, 0, st>>>(io, diag, c, lse, a, 1);
  else attn_fwd_f32_kernel<DKP, 4, VEC, CAUSAL><<<nt * bh, 256, 0, st>>>(io, diag, c, lse, a, nt);
  return hipGetLastError();
}
template <int DKP, bool VEC>
hipError_t launch_fwd(const AttnIO& io, const float* diag, float* c, float* lse, const AttnDims& a, hipStream_t st) {
  return a.causal ? launch_fwd_form<DKP, VEC, true>(io, diag, c, lse, a, st)
                  : launch_fwd_form<DKP, VEC, false>(io, diag, c, lse, a, st);
}
template <int DKP, bool VEC, bool CAUSAL>
hipError_t launch_dkv_form(const AttnIO& io, const float* dc, const float* diag, const float* lse, const float* dvec,
                           const AttnDims& a, hipStream_t st) {
  const int bh = a.B * a.H, nt = ceil_div(a.Sk, 128);
  if (a.Sk <= 32) attn_bwd_dkv_f32_kernel<DKP, 1, VEC, CAUSAL><<<bh, 64, 0, st>>>(io, dc, diag, lse, dvec, a, 1);
  else if (a.Sk <= 64) attn_bwd_dkv_f32_kernel<DKP, 2, VEC, CAUSAL><<<bh, 128, 0, st>>>(io, dc, diag, lse, dvec, a, 1);
  else attn_bwd_dkv_f32_kernel<DKP, 4, VEC, CAUSAL><<<nt * bh, 256, 0, st>>>(io, dc, diag, lse, dvec, a, nt);
  return hipGetLastError();
}
template <int DKP, bool VEC>
hipError_t launch_bwd(const AttnIO& io, const float* c, const float* dc, const float* diag, const float* lse, float* dvec,
                      float* ddiag, const AttnDims& a, hipStream_t st) {
  const int bh = a.B * a.H, nt = ceil_div(a.S, 64);
  auto dq = [&](auto kern, int tiles, int waves) {
    const int lds = a.bias ? (a.S + waves * 32 - 1) * 4 : 0;
    kern<<<tiles * bh, waves * 64, lds, st>>>(io, c, dc, diag, lse, dvec, ddiag, a, tiles);
  };
  if (a.S <= 32) dq(attn_bwd_dq_f32_kernel<DKP, 1, VEC>, 1, 1);
  else if (a.S > 64 && nt * bh > 256 && nt * bh <= 512) dq(attn_bwd_dq_f32_kernel<DKP, 4, VEC>, ceil_div(a.S, 128), 4);
  else dq(attn_bwd_dq_f32_kernel<DKP, 2, VEC>, nt, 2);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  return a.causal ? launch_dkv_form<DKP, VEC, true>(io, dc, diag, lse, dvec, a, st)
                  : launch_dkv_form<DKP, VEC, false>(io, dc, diag, lse, dvec, a, st);
}

}  // namespace

bool attn_f32_supported(const AttnDims& a) {
  const int64_t tiles = ceil_div(a.S > a.Sk ? a.S : a.Sk, 64);
  // static tiles (up to 34 KB) + the diagonals of a workgroup in 64 KB of LDS
  return a.dk <= 128 && a.S <= 4096 && tiles * a.B * a.H < ((int64_t)1 << 31);
}

hipError_t launch_attn_fwd_f32(const AttnIO& io, const float* diag, float* c, float* lse, const AttnDims& a, hipStream_t st) {
  const bool vec = vec_ok(io, a, c, nullptr);
  if (a.dk <= 32) return vec ? launch_fwd<32, true>(io, diag, c, lse, a, st) : launch_fwd<32, false>(io, diag, c, lse, a, st);
  if (a.dk <= 64) return vec ? launch_fwd<64, true>(io, diag, c, lse, a, st) : launch_fwd<64, false>(io, diag, c, lse, a, st);
  return vec ? launch_fwd<128, true>(io, diag, c, lse, a, st) : launch_fwd<128, false>(io, diag, c, lse, a, st);
}

hipError_t launch_attn_bwd_f32(const AttnIO& io, const float* c, const float* dc, const float* diag, const float* lse,
                               float* dvec, float* ddiag, const AttnDims& a, hipStream_t st) {
  const bool vec = vec_ok(io, a, c, dc);
  auto run = [&](auto fn) { return fn(io, c, dc, diag, lse, dvec, ddiag, a, st); };
  if (a.dk <= 32) return run(vec ? launch_bwd<32, true> : launch_bwd<32, false>);
  if (a.dk <= 64) return run(vec ? launch_bwd<64, true> : launch_bwd<64, false>);
  return run(vec ? launch_bwd<128, true> : launch_bwd<128, false>);
}

}  // namespace t5mi
