// Adafactor with factored second moments and update clipping (the optimizer of the T5 models in
// paper Sec. 4).  HBM-bound: float32, 16-byte loads, wave reductions, deterministic two-stage sums.
//
// Factored tensor [R,C], tiles of 64 rows x 256 columns:
//   stats     : per-tile row sums and column sums of G*G          -> rowpart[tc][R], colpart[tr][C]
//   finalize  : v_row, v_col EMA; cfac_j = rsqrt(v_col_j); consumers form rsqrt(v_row_i / mean v_row)
//   norms     : per-tile sums of U*U (U = G rfac cfac) and of W*W -> part[2][tiles]
//   coef      : coef = lr * max(eps2, RMS(W)) / max(1, RMS(U)/clip)
//   apply     : W -= coef * U   (+ optional bf16 copy)
// Unfactored tensors use the same skeleton with v_full updated elementwise in the first pass.
//
// Every kernel works on a batch of up to 16 tensors at once (descriptor table passed by value, a
// workgroup finds its tensor from a prefix table of tile counts): a whole block's optimizer step is
// five launches, not five per tensor -- at T5.1.1-Base sizes the per-tensor launches cost more than
// the memory traffic.
#include "kernels.h"
#include <cmath>
#include <cstring>

namespace t5mi {

namespace {

constexpr int TR = 64;   // tile rows
constexpr int TC = 256;  // tile columns, four to a lane
// A tile's workgroup has sixteen wavefronts of four rows, whose loads are all in flight at once.  (With four wavefronts of sixteen
// rows eight workgroups shared a compute unit: the 2961 tiles of a d 2048 layer were 1.45 rounds, the second half empty; stats
// 57 -> 52 us, norms 83 -> 81, apply 121 -> 106.)
constexpr int NWV = 16, NT = NWV * 64, RPW = TR / NWV;

struct AfWs {
  float* rowpart;  // [ntc][R]
  float* colpart;  // [ntr][C]
  float* part_u;   // [ntiles]
  float* part_w;   // [ntiles]
  float* rsum;     // [ceil(R / 256)] sums of v_row over 256 rows (room for R)
  float* cfac;     // [C]
  float* scal;     // [4]: 0 = coef
};

// A lane's four columns: neighbours, read and written as 16 bytes, where rows are a multiple of 16 bytes (V4), else 64 apart, so
// that an instruction still covers 256 bytes of a row.  (Of rows that are no such multiple a tile had one column to a lane: a
// quarter of the work for the same sixteen wavefronts, 4097 x 4095 147 -> 93 us, 32128 x 769 230 -> 162.)
template <bool V4>
struct AfCols {
  int c0, n;  // first column of the lane, columns of the tensor
  __device__ __forceinline__ AfCols(int bx, int lane, int64_t C) : c0(bx * TC + (V4 ? lane * 4 : lane)), n((int)C) {}
  __device__ __forceinline__ bool any() const { return c0 < n; }
  __device__ __forceinline__ bool has(int i) const { return V4 || c0 + 64 * i < n; }  // (where there are any)
  // (past the end: the last column again, so that a row's loads are one block)
  __device__ __forceinline__ uint32_t at(int i) const { return V4 ? c0 + i : min(c0 + 64 * i, n - 1); }
  __device__ __forceinline__ static int slot(int lane, int i) { return V4 ? lane * 4 + i : lane + 64 * i; }  // in the tile
  // row: the same in the whole wavefront
  __device__ __forceinline__ void load(const float* __restrict__ row, float (&v)[4]) const {
    if constexpr (V4) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(row + at(0));
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = t[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = row[at(i)];
    }
  }
  __device__ __forceinline__ void store(float* __restrict__ row, const float (&v)[4]) const {
    if constexpr (V4) {
      f32x4 t;
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = v[i];
      *reinterpret_cast<f32x4*>(row + at(0)) = t;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (has(i)) row[at(i)] = v[i];
    }
  }
};

struct AfItem {
  float* w;
  const float* g;
  float* v_row;
  float* v_col;
  float* v_full;
  bf16* lp;
  float* m;  // momentum (nullable)
  int64_t R, C;
  AfWs ws;
  int v4, ntc, ntr, factored;
};
struct AfBatch {
  AfItem it[AF_MAX_TENSORS];
  int tile_start[AF_MAX_TENSORS + 1];  // prefix sums of ntc * ntr
  int fin_start[AF_MAX_TENSORS + 1];   // prefix sums of ceil((R + C) / 256) over factored tensors
  int count;
  float beta2, eps1;
  float beta1, decay;  // momentum coefficient; lr * weight_decay
};

// Tensor that owns 1-D block `b` under prefix table `start` (wave-uniform; entries past the last tensor hold the total).  All
// entries are compared, in scalar registers: a search would wait for one after the other before the first load of a tile.
__device__ __forceinline__ int af_find(const int* start, int b) {
  int t = 0;
#pragma unroll
  for (int i = 1; i < AF_MAX_TENSORS; ++i) t += b >= start[i] ? 1 : 0;
  return t;
}

// Wave w takes rows w, w + 16, ... of the tile; lanes span the columns.
template <bool V4>
__device__ __forceinline__ void af_stats_tile(const AfItem& it, int bx, int by, float (*colred)[256]) {
  const float* __restrict__ g = it.g;
  const int64_t R = it.R, C = it.C;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const AfCols<V4> cols(bx, lane, C);
  const int64_t r0 = (int64_t)by * TR + wave;
  float csum[4], v[RPW][4], rs[RPW];
#pragma unroll
  for (int i = 0; i < 4; ++i) csum[i] = 0.f;
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int64_t r = r0 + NWV * q;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[q][i] = 0.f;
    if (cols.any() && r < R) cols.load(g + r * C, v[q]);
  }
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    rs[q] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = cols.has(i) ? v[q][i] * v[q][i] : 0.f;
      csum[i] += x;
      rs[q] += x;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < RPW; ++q) rs[q] += __shfl_xor(rs[q], off, 64);
  if (lane < RPW) {
    const int64_t r = r0 + NWV * lane;
    if (r < R) it.ws.rowpart[(int64_t)bx * R + r] = lane == 0 ? rs[0] : lane == 1 ? rs[1] : lane == 2 ? rs[2] : rs[3];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) colred[wave][cols.slot(lane, i)] = csum[i];
  __syncthreads();
  for (int t = threadIdx.x; t < TC; t += NT) {
    const int64_t c = (int64_t)bx * TC + t;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) s += colred[w][t];
    if (c < C) it.ws.colpart[(int64_t)by * C + c] = s;
  }
}

__global__ __launch_bounds__(NT, 8) void af_stats_kernel(AfBatch b) {
  __shared__ float colred[NWV][256];
  const int ti = af_find(b.tile_start, blockIdx.x);
  const AfItem& it = b.it[ti];
  if (!it.factored) return;
  const int local = blockIdx.x - b.tile_start[ti];
  const int bx = local % it.ntc, by = local / it.ntc;
  if (it.v4) af_stats_tile<true>(it, bx, by, colred);
  else af_stats_tile<false>(it, bx, by, colred);
}

// One thread per row and per column: folds the tile partials into the second-moment vectors.
// cfac_j = rsqrt(v_col_j); the row factor needs mean(v_row) and is formed by the consumers, from the workgroups' sums.
__global__ __launch_bounds__(256) void af_finalize_kernel(AfBatch b) {
  __shared__ float red[4];
  const int ti = af_find(b.fin_start, blockIdx.x);
  const AfItem& it = b.it[ti];
  if (!it.factored) return;
  const int64_t R = it.R, C = it.C;
  const float beta2 = b.beta2, eps1 = b.eps1;
  const int64_t blk = blockIdx.x - b.fin_start[ti], idx = blk * 256 + threadIdx.x;
  float vr = 0.f;
  if (idx < R) {
    float s = 0.f;
#pragma unroll 8
    for (int t = 0; t < it.ntc; ++t) s += it.ws.rowpart[(int64_t)t * R + idx];  // (eight loads in flight, summed in order)
    vr = beta2 * it.v_row[idx] + (1.f - beta2) * (s / (float)C + eps1);
    it.v_row[idx] = vr;
  } else if (idx < R + C) {
    const int64_t j = idx - R;
    float s = 0.f;
#pragma unroll 8
    for (int t = 0; t < it.ntr; ++t) s += it.ws.colpart[(int64_t)t * C + j];
    const float vc = beta2 * it.v_col[j] + (1.f - beta2) * (s / (float)R + eps1);
    it.v_col[j] = vc;
    it.ws.cfac[j] = rsqrtf(vc);
  }
  if (blk * 256 < R) {
    vr = block_sum<4>(vr, red);
    if (threadIdx.x == 0) it.ws.rsum[blk] = vr;
  }
}

// mean(v_row) in a fixed order, by a wavefront (all get the same value).
__device__ __forceinline__ float af_mean_vrow(const float* __restrict__ rsum, int64_t R) {
  float s = 0.f;
  for (int64_t i = threadIdx.x & 63; i < (R + 255) / 256; i += 64) s += rsum[i];
  return wave_sum(s) / (float)R;
}

// Per-tile sums of U*U and W*W.  FACT: U = g rfac cfac.  !FACT: updates v_full and U = g rsqrt(v).
template <bool V4, bool FACT>
__device__ __forceinline__ void af_norms_tile(const AfItem& it, int bx, int by, int tile, float beta2, float eps1,
                                              float* red) {
  const float* __restrict__ g = it.g;
  const float* __restrict__ w = it.w;
  float* __restrict__ v_full = it.v_full;
  const float* __restrict__ v_row = it.v_row;
  const int64_t R = it.R, C = it.C;
  const AfWs& ws = it.ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const AfCols<V4> cols(bx, lane, C);
  const int64_t r0 = (int64_t)by * TR + wave;
  float gv[RPW][4], wv[RPW][4];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int64_t r = r0 + NWV * q;
#pragma unroll
    for (int i = 0; i < 4; ++i) gv[q][i] = wv[q][i] = 0.f;
    if (cols.any() && r < R) {
      cols.load(g + r * C, gv[q]);
      cols.load(w + r * C, wv[q]);
    }
  }
  float inv_mean = 1.f;
  if constexpr (FACT) {
    const float mean_vr = af_mean_vrow(ws.rsum, R);
    inv_mean = 1.f / mean_vr;
    if (tile == 0 && threadIdx.x == 0) ws.scal[1] = inv_mean;
  }
  float su = 0.f, sw = 0.f;
  if (cols.any()) {
    float cf[4];
    if constexpr (FACT) cols.load(ws.cfac, cf);
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      const int64_t r = r0 + NWV * q;
      if (r >= R) break;
      if constexpr (FACT) {
        const float rf = rsqrtf(v_row[r] * inv_mean);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float u = gv[q][i] * rf * cf[i];
          su += cols.has(i) ? u * u : 0.f;
          sw += cols.has(i) ? wv[q][i] * wv[q][i] : 0.f;
        }
      } else {
        float vv[4];
        cols.load(v_full + r * C, vv);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          vv[i] = beta2 * vv[i] + (1.f - beta2) * (gv[q][i] * gv[q][i] + eps1);
          const float u = gv[q][i] * rsqrtf(vv[i]);
          su += cols.has(i) ? u * u : 0.f;
          sw += cols.has(i) ? wv[q][i] * wv[q][i] : 0.f;
        }
        cols.store(v_full + r * C, vv);
      }
    }
  }
  su = block_sum<NWV>(su, red);
  sw = block_sum<NWV>(sw, red + NWV);
  if (threadIdx.x == 0) {
    ws.part_u[tile] = su;
    ws.part_w[tile] = sw;
  }
}

__global__ __launch_bounds__(NT, 8) void af_norms_kernel(AfBatch b) {
  __shared__ float red[2 * NWV];
  const int ti = af_find(b.tile_start, blockIdx.x);
  const AfItem& it = b.it[ti];
  const int local = blockIdx.x - b.tile_start[ti];
  const int bx = local % it.ntc, by = local / it.ntc;
  if (it.v4) {
    if (it.factored) af_norms_tile<true, true>(it, bx, by, local, b.beta2, b.eps1, red);
    else af_norms_tile<true, false>(it, bx, by, local, b.beta2, b.eps1, red);
  } else {
    if (it.factored) af_norms_tile<false, true>(it, bx, by, local, b.beta2, b.eps1, red);
    else af_norms_tile<false, false>(it, bx, by, local, b.beta2, b.eps1, red);
  }
}

// One workgroup per tensor.
__global__ __launch_bounds__(1024) void af_coef_kernel(AfBatch b, adafactor_cfg c) {
  __shared__ float red[32];
  const AfItem& it = b.it[blockIdx.x];
  const int64_t ntiles = (int64_t)it.ntc * it.ntr;
  float su = 0.f, sw = 0.f;
  for (int64_t i = threadIdx.x; i < ntiles; i += 1024) {
    su += it.ws.part_u[i];
    sw += it.ws.part_w[i];
  }
  su = block_sum<16>(su, red);
  sw = block_sum<16>(sw, red + 16);
  if (threadIdx.x == 0) {
    const double count = (double)it.R * (double)it.C;
    const float rms_u = sqrtf(su / (float)count), rms_w = sqrtf(sw / (float)count);
    float alpha = c.lr;
    if (c.scale_by_param) alpha *= fmaxf(c.eps2, rms_w);
    it.ws.scal[0] = alpha / fmaxf(1.f, rms_u / c.clip);
  }
}

// W <- W - D - decay W,  D = alpha U, or with momentum m <- beta1 m + (1 - beta1) alpha U, D = m
template <bool V4, bool FACT>
__device__ __forceinline__ void af_apply_tile(const AfItem& it, int bx, int by, float beta1, float decay) {
  float* __restrict__ w = it.w;
  const float* __restrict__ g = it.g;
  const float* __restrict__ v_full = it.v_full;
  const float* __restrict__ v_row = it.v_row;
  bf16* __restrict__ lp = it.lp;
  float* __restrict__ mom = it.m;
  const int64_t R = it.R, C = it.C;
  const AfWs& ws = it.ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const AfCols<V4> cols(bx, lane, C);
  const int64_t r0 = (int64_t)by * TR + wave;
  if (!cols.any()) return;
  float gv[RPW][4], wv[RPW][4];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int64_t r = r0 + NWV * q;
    if (r < R) {
      cols.load(g + r * C, gv[q]);
      cols.load(w + r * C, wv[q]);
    }
  }
  const float coef = ws.scal[0];
  float cf[4];
  if constexpr (FACT) cols.load(ws.cfac, cf);
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int64_t r = r0 + NWV * q;
    if (r >= R) break;
    float dv[4];
    if constexpr (FACT) {
      const float rf = rsqrtf(v_row[r] * ws.scal[1]) * coef;
#pragma unroll
      for (int i = 0; i < 4; ++i) dv[i] = gv[q][i] * rf * cf[i];
    } else {
      float vv[4];
      cols.load(v_full + r * C, vv);
#pragma unroll
      for (int i = 0; i < 4; ++i) dv[i] = coef * gv[q][i] * rsqrtf(vv[i]);
    }
    if (mom) {
      float mv[4];
      cols.load(mom + r * C, mv);
#pragma unroll
      for (int i = 0; i < 4; ++i) { mv[i] = beta1 * mv[i] + (1.f - beta1) * dv[i]; dv[i] = mv[i]; }
      cols.store(mom + r * C, mv);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) wv[q][i] = wv[q][i] - dv[i] - decay * wv[q][i];
    cols.store(w + r * C, wv[q]);
    if (lp) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (cols.has(i)) (lp + r * C)[cols.at(i)] = (bf16)wv[q][i];
    }
  }
}

__global__ __launch_bounds__(NT, 8) void af_apply_kernel(AfBatch b) {
  const int ti = af_find(b.tile_start, blockIdx.x);
  const AfItem& it = b.it[ti];
  const int local = blockIdx.x - b.tile_start[ti];
  const int bx = local % it.ntc, by = local / it.ntc;
  if (it.v4) {
    if (it.factored) af_apply_tile<true, true>(it, bx, by, b.beta1, b.decay);
    else af_apply_tile<true, false>(it, bx, by, b.beta1, b.decay);
  } else {
    if (it.factored) af_apply_tile<false, true>(it, bx, by, b.beta1, b.decay);
    else af_apply_tile<false, false>(it, bx, by, b.beta1, b.decay);
  }
}

struct AfGeom {
  int ntc, ntr;
  int64_t ntiles;
};
AfGeom geom(int64_t R, int64_t C) {
  AfGeom g;
  g.ntc = ceil_div(C, TC);
  g.ntr = ceil_div(R, TR);
  g.ntiles = (int64_t)g.ntc * g.ntr;
  return g;
}
AfWs carve(void* ws, int64_t R, int64_t C, const AfGeom& g) {
  char* p = (char*)ws;
  AfWs w;
  auto take = [&](size_t n) { float* r = (float*)p; p += align_up(n * sizeof(float)); return r; };
  w.rowpart = take((size_t)g.ntc * R);
  w.colpart = take((size_t)g.ntr * C);
  w.part_u = take(g.ntiles);
  w.part_w = take(g.ntiles);
  w.rsum = take(R);
  w.cfac = take(C);
  w.scal = take(4);
  return w;
}

}  // namespace

size_t adafactor_ws_bytes(int64_t R, int64_t C, int factored) {
  (void)factored;
  AfGeom g = geom(R, C);
  if (C % 4) {  // (the size callers know for such rows: room for tiles of 64 columns)
    g.ntc = ceil_div(C, 64);
    g.ntiles = (int64_t)g.ntc * g.ntr;
  }
  size_t n = 0;
  n += align_up((size_t)g.ntc * R * 4) + align_up((size_t)g.ntr * C * 4);
  n += 2 * align_up((size_t)g.ntiles * 4) + align_up(R * 4) + align_up(C * 4) + align_up(16);
  return n;
}

hipError_t launch_adafactor_multi(const AfTensor* t, int n, const adafactor_cfg& c, void* wsp, hipStream_t st) {
  if (n < 1 || n > AF_MAX_TENSORS) return hipErrorInvalidValue;
  AfBatch b;
  std::memset(&b, 0, sizeof(b));
  b.count = n;
  b.beta2 = (float)(1.0 - pow((double)c.step, -(double)c.decay_pow));
  b.eps1 = c.eps1;
  b.beta1 = c.beta1;
  b.decay = c.lr * c.weight_decay;
  char* wp = (char*)wsp;
  int64_t tiles = 0, fins = 0;
  bool any_factored = false;
  for (int i = 0; i < n; ++i) {
    const AfGeom g = geom(t[i].rows, t[i].cols);
    AfItem& it = b.it[i];
    it.w = t[i].param; it.g = t[i].grad; it.v_row = t[i].v_row; it.v_col = t[i].v_col; it.v_full = t[i].v_full;
    it.lp = (bf16*)t[i].bf16_out;
    it.m = c.beta1 > 0.f ? t[i].m : nullptr;
    it.R = t[i].rows; it.C = t[i].cols;
    it.ws = carve(wp, it.R, it.C, g);
    wp += adafactor_ws_bytes(it.R, it.C, t[i].factored);
    it.v4 = it.C % 4 == 0; it.ntc = g.ntc; it.ntr = g.ntr; it.factored = t[i].factored ? 1 : 0;
    b.tile_start[i] = (int)tiles;
    b.fin_start[i] = (int)fins;
    tiles += g.ntiles;
    if (it.factored) { fins += ceil_div(it.R + it.C, (int64_t)256); any_factored = true; }
    if (tiles > (int64_t)1 << 30 || fins > (int64_t)1 << 30) return hipErrorInvalidValue;
  }
  for (int i = n; i <= AF_MAX_TENSORS; ++i) { b.tile_start[i] = (int)tiles; b.fin_start[i] = (int)fins; }
  hipError_t e;
  if (any_factored) {
    af_stats_kernel<<<(unsigned)tiles, NT, 0, st>>>(b);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    af_finalize_kernel<<<(unsigned)fins, 256, 0, st>>>(b);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  af_norms_kernel<<<(unsigned)tiles, NT, 0, st>>>(b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  af_coef_kernel<<<n, 1024, 0, st>>>(b, c);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  af_apply_kernel<<<(unsigned)tiles, NT, 0, st>>>(b);
  return hipGetLastError();
}

hipError_t launch_adafactor(float* param, const float* grad, float* v_row, float* v_col, float* v_full,
                            int64_t R, int64_t C, int factored, const adafactor_cfg& c, void* bf16_out,
                            void* wsp, hipStream_t st) {
  AfTensor t{param, grad, v_row, v_col, v_full, R, C, factored, bf16_out, nullptr};
  return launch_adafactor_multi(&t, 1, c, wsp, st);
}

}  // namespace t5mi

// ------------------------------------------------------------------------------------------------
// adafactor_step_static: the single-tensor update for callers that cannot allocate.  Its scratch
// (the tile partial sums and factors that adafactor_step takes from the caller's workspace) is this
// file-scope device array; every GPU holds its own copy at its own address, looked up once per device.
// ------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[ADAFACTOR_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU, set on first use there
}  // namespace

extern "C" int adafactor_step_static(float* param, const float* grad, float* v_row, float* v_col, float* v_full,
                                     int64_t rows, int64_t cols, int factored, const adafactor_cfg* cfg,
                                     void* bf16_copy_out, void* stream) {
  using namespace t5mi;
  if (!cfg) return T5_ERR_NULL;
  if (rows < 1 || cols < 1 || cfg->step < 1 || !(cfg->clip > 0.f) || !(cfg->eps1 >= 0.f)) return T5_ERR_SHAPE;
  if (!(cfg->beta1 >= 0.f && cfg->beta1 < 1.f) || !(cfg->weight_decay >= 0.f)) return T5_ERR_SHAPE;
  if (cfg->beta1 > 0.f) return T5_ERR_UNSUPPORTED;
  if (rows > (1 << 24) || cols > (1 << 24)) return T5_ERR_UNSUPPORTED;
  if (!param || !grad) return T5_ERR_NULL;
  if (factored ? (!v_row || !v_col) : !v_full) return T5_ERR_NULL;
  if (adafactor_ws_bytes(rows, cols, factored) > (size_t)ADAFACTOR_STATIC_SCRATCH_BYTES) return T5_ERR_WORKSPACE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return T5_ERR_DEVICE;
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return T5_ERR_DEVICE;
    g_scratch_ptr[dev] = p;
  }
  // Nothing in the scratch has to start at zero: every partial sum, factor and scalar a kernel of this
  // update reads was written by an earlier kernel of the same update.
  if (launch_adafactor(param, grad, v_row, v_col, v_full, rows, cols, factored, *cfg, bf16_copy_out,
                       g_scratch_ptr[dev], (hipStream_t)stream) != hipSuccess)
    return T5_ERR_DEVICE;
  return T5_OK;
}

