// Reference-grade GEMM for bf16 shapes the MFMA kernel does not take (and float32 problems beyond its grid):
// 64x64 output tile, 16-deep LDS stages, float32 FMA, any shape and either operand orientation.
// Also: the elementwise gated-GELU of the unfused path and the bf16 weight transpose-pack.
#include "kernels.h"
#include <algorithm>

namespace t5mi {

namespace {

constexpr int SB = 64;  // tile edge
constexpr int SK = 16;  // k depth per stage

__device__ __forceinline__ float ld_elem(const void* p, size_t idx, int type) {
  return type == IN_BF16 ? (float)((const bf16*)p)[idx] : ((const float*)p)[idx];
}
__device__ __forceinline__ void st_elem(void* p, size_t idx, int type, float v) {
  if (type == IN_BF16) ((bf16*)p)[idx] = (bf16)v; else ((float*)p)[idx] = v;
}

__global__ __launch_bounds__(256) void gemm_simple_kernel(GemmDesc g, GemmEpi e) {
  __shared__ float As[SK][SB + 1];
  __shared__ float Bs[SK][SB + 1];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int m0 = blockIdx.y * SB, n0 = blockIdx.x * SB;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int s = 0; s < g.nseg; ++s) {
    const GemmSeg sg = g.seg[s];
    for (int k0 = 0; k0 < sg.K; k0 += SK) {
      // 64x16 elements per operand, 256 threads -> 4 each
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int idx = tid + i * 256;
        int mm, kk;
        if (g.a_kc) { kk = idx % SK; mm = idx / SK; } else { mm = idx % SB; kk = idx / SB; }
        float v = 0.f;
        if (m0 + mm < g.M && k0 + kk < sg.K) {
          const size_t off = g.a_kc ? (size_t)(m0 + mm) * sg.lda + (k0 + kk)
                                    : (size_t)(k0 + kk) * sg.lda + (m0 + mm);
          v = ld_elem(sg.A, off, g.in_type);
        }
        As[kk][mm] = v;
        int nn, kb;
        if (g.b_kc) { kb = idx % SK; nn = idx / SK; } else { nn = idx % SB; kb = idx / SB; }
        float u = 0.f;
        if (n0 + nn < g.N && k0 + kb < sg.K) {
          const size_t off = g.b_kc ? (size_t)(n0 + nn) * sg.ldb + (k0 + kb)
                                    : (size_t)(k0 + kb) * sg.ldb + (n0 + nn);
          u = ld_elem(sg.B, off, g.in_type);
        }
        Bs[kb][nn] = u;
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < SK; ++kk) {
        float a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= g.N) continue;
      const float v = acc[i][j];
      const size_t o = (size_t)m * e.ld0 + n;
      const float mk = e.drop.on ? drop_mult(e.drop, drop_row_key(e.drop, (uint32_t)m), (uint32_t)n) : 1.f;
      switch (e.kind) {
        case EPI_STORE:
          st_elem(e.out0, o, e.out_type, (e.act == ACT_RELU ? fmaxf(v, 0.f) : v) * mk);
          break;
        case EPI_RESID: {
          const float a = ld_elem(e.aux0, (size_t)m * (e.ld_aux ? e.ld_aux : e.ld0) + n, e.aux_type);
          const float sc = e.drop.on ? e.drop.scale : 1.f;
          st_elem(e.out0, o, e.out_type, e.aux_mask ? (a > 0.f ? v * sc : 0.f) : v * mk + a);
          break;
        }
        case EPI_GEGLU_BWD: {
          const size_t oa = (size_t)m * (e.ld_aux ? e.ld_aux : e.ld0) + n;
          const float gp = ld_elem(e.aux0, oa, e.aux_type), gl = ld_elem(e.aux1, oa, e.aux_type);
          st_elem(e.out0, o, e.out_type, v * gp);
          st_elem(e.out1, o, e.out_type, v * gl);
          break;
        }
        case EPI_SPLIT_F32: {
          const int which = n / e.split_n, nn = n % e.split_n;
          float* dst = (float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2);
          const size_t oo = (size_t)m * e.ld0 + nn;
          dst[oo] = e.accumulate ? dst[oo] + v : v;
          break;
        }
        default:
          break;
      }
    }
  }
}

template <typename T>
__global__ void geglu_fwd_kernel(T* __restrict__ u, T* __restrict__ w, T* __restrict__ a, int64_t n, int act,
                                 DropSite drop, int cols) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    const float uu = to_f32(u[i]), ww = to_f32(w[i]);
    float gl, dgl;
    gelu_both(act, uu, gl, dgl);
    // the saved factors carry the dropout multiplier of the hidden activation, for the backward
    const float mk = drop.on ? drop_mult(drop, drop_row_key(drop, (uint32_t)(i / cols)), (uint32_t)(i % cols)) : 1.f;
    a[i] = from_f32<T>(gl * ww * mk);
    u[i] = from_f32<T>(ww * dgl * mk);
    w[i] = from_f32<T>(gl * mk);
  }
}

// dst[n][k] for a 64x64 tile staged through LDS; see launch_pack_transpose_multi.  A workgroup finds its job and tile in the
// jobs' first workgroups.  (With one grid plane per job, each as large as the largest, five of six workgroups found nothing
// to do: 13.4 us at d 768, 46.3 at d 2048 against 11.7 and 45.1 like this.)
// Bound: bytes (28 MB for the weights of a d 768 layer, 6 us at the copy rate).  A thread reads 16 bytes of two rows, pairs the rows'
// elements into words (k, k + 1) of its 8 columns, and the tile leaves LDS as 16-byte runs along k.
// LDS: word (n, k/2) of the tile at n * 32 + ((k/2) ^ swz(n)), the 16-byte groups of a row swizzled so that the writes of
// a wavefront (8 columns of 8 row pairs at a time) and its 16-byte reads spread over the banks.
struct PackArgs {
  PackJobs jobs;
  int first[9];  // first workgroup of each job, then that of the bias diagonals
};
__global__ __launch_bounds__(256) void pack_transpose_kernel(PackArgs args) {
  __shared__ __attribute__((aligned(16))) uint32_t tile[64 * 32];
  const PackJobs& jobs = args.jobs;
  int job = 0;
  while (job < jobs.count && (int)blockIdx.x >= args.first[job + 1]) ++job;
  const int blk = (int)blockIdx.x - args.first[job];
  if (job == jobs.count) {  // the layer's bias diagonals (see launch_relpos_diag): a launch of their own costs 4.5 us
    const int w = 2 * jobs.S - 1, i = blk * 256 + (int)threadIdx.x;
    if (i >= w) return;
    const int b = relpos_bucket_dev(i - (jobs.S - 1), jobs.lut);
    for (int h = 0; h < jobs.H; ++h) jobs.diag[(size_t)h * w + i] = (float)((const bf16*)jobs.table)[b * jobs.H + h];
    return;
  }
  const PackJob& jb = jobs.j[job];
  const int nsrc = jb.nsrc, K = jb.K, n_each = jb.n_each, interleave = jb.interleave;
  const int n_total = nsrc * n_each;
  const int tiles_n = (n_total + 63) / 64;
  const int n0 = blk % tiles_n * 64, k0 = blk / tiles_n * 64;
  // interleave and n_each are multiples of 32 (or interleave == 0), so each 32-wide half of the tile's packed
  // rows comes from one source and 32 consecutive source columns; a thread's 8 columns lie inside one half.
  const int c = (threadIdx.x & 7) * 8, kp = threadIdx.x >> 3, nh = n0 + (c & 32);  // columns c .. c+7, rows 2 kp and 2 kp + 1
  int which, col0;
  if (interleave > 0) {
    which = (nh / interleave) % nsrc;
    col0 = (nh / (interleave * nsrc)) * interleave + nh % interleave;
  } else {
    which = nh / n_each;
    col0 = nh % n_each;
  }
  const bool in_n = nh < n_total;
  const bf16* src = (const bf16*)jb.src[in_n ? which : 0] + (in_n ? col0 + (c & 31) : 0);
  const int k = k0 + 2 * kp;
  u32x4 lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
  if (in_n && k < K) {  // K is even: the two rows are inside or outside together
    const bf16 *r0 = src + (size_t)k * n_each, *r1 = r0 + n_each;
    if (((uintptr_t)src & 15) == 0) {  // (uniform over the 32 columns of a source: n_each is a multiple of 32)
      lo = *reinterpret_cast<const u32x4*>(r0);
      hi = *reinterpret_cast<const u32x4*>(r1);
    } else {  // a weight that does not start on 16 bytes
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        lo[q] = __builtin_bit_cast(uint16_t, r0[2 * q]) | ((uint32_t)__builtin_bit_cast(uint16_t, r0[2 * q + 1]) << 16);
        hi[q] = __builtin_bit_cast(uint16_t, r1[2 * q]) | ((uint32_t)__builtin_bit_cast(uint16_t, r1[2 * q + 1]) << 16);
      }
    }
  }
  auto swz = [](int n) { return ((n ^ (n >> 3)) & 7) << 2; };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = c + 2 * q;
    tile[n * 32 + (kp ^ swz(n))] = (lo[q] & 0xFFFFu) | (hi[q] << 16);
    tile[(n + 1) * 32 + (kp ^ swz(n + 1))] = (lo[q] >> 16) | (hi[q] & 0xFFFF0000u);
  }
  __syncthreads();
  bf16* dst = (bf16*)jb.dst;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int n = it * 32 + (threadIdx.x >> 3), k8 = threadIdx.x & 7;  // 16 bytes: k0 + 8 k8 .. + 7 of packed row n0 + n
    const u32x4 v = *reinterpret_cast<const u32x4*>(tile + n * 32 + ((k8 * 4) ^ swz(n)));
    if (n0 + n >= n_total) continue;
    bf16* d = dst + (size_t)(n0 + n) * K + k0 + k8 * 8;
    if (k0 + k8 * 8 + 8 <= K && K % 8 == 0 && ((uintptr_t)dst & 15) == 0) {
      *reinterpret_cast<u32x4*>(d) = v;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (k0 + k8 * 8 + 2 * q < K) reinterpret_cast<uint32_t*>(d)[q] = v[q];
    }
  }
}

}  // namespace

hipError_t launch_gemm_simple(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  if (e.kind == EPI_GEGLU_FWD) return hipErrorInvalidValue;
  dim3 grid(ceil_div(g.N, SB), ceil_div(g.M, SB));
  gemm_simple_kernel<<<grid, 256, 0, st>>>(g, e);
  return hipGetLastError();
}

__global__ void zero_f32_kernel(ZeroList z) {
  const int a = blockIdx.y;
  float* p = z.p[a];
  const int64_t n = z.n[a];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
}

hipError_t launch_zero_f32(const ZeroList& z, hipStream_t st) {
  if (z.count <= 0) return hipSuccess;
  int64_t mx = 0;
  for (int a = 0; a < z.count; ++a) mx = z.n[a] > mx ? z.n[a] : mx;
  const int64_t blocks = std::min<int64_t>((mx + 255) / 256, 1024);
  zero_f32_kernel<<<dim3((unsigned)std::max<int64_t>(blocks, 1), (unsigned)z.count), 256, 0, st>>>(z);
  return hipGetLastError();
}

hipError_t launch_geglu_fwd(void* u, void* w, void* a, int type, int64_t n, int act, const DropSite& drop, int cols,
                            hipStream_t st) {
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (type == IN_BF16)
    geglu_fwd_kernel<bf16><<<(int)blocks, 256, 0, st>>>((bf16*)u, (bf16*)w, (bf16*)a, n, act, drop, cols);
  else
    geglu_fwd_kernel<float><<<(int)blocks, 256, 0, st>>>((float*)u, (float*)w, (float*)a, n, act, drop, cols);
  return hipGetLastError();
}

hipError_t launch_pack_transpose_multi(const PackJobs& jobs, hipStream_t st) {
  if (jobs.count < 1 || jobs.count > 8) return hipErrorInvalidValue;
  PackArgs args;
  args.jobs = jobs;
  int blocks = 0;
  for (int q = 0; q < 9; ++q) args.first[q] = 0;
  for (int q = 0; q < jobs.count; ++q) {
    const PackJob& jb = jobs.j[q];
    if (jb.nsrc < 1 || jb.nsrc > 3 || jb.n_each % 32 != 0 || (jb.interleave > 0 && jb.interleave % 32 != 0) ||
        jb.K % 2 != 0)
      return hipErrorInvalidValue;
    args.first[q] = blocks;
    blocks += ceil_div((int64_t)jb.nsrc * jb.n_each, 64) * ceil_div(jb.K, 64);
  }
  args.first[jobs.count] = blocks;
  if (jobs.diag) blocks += ceil_div(2 * (int64_t)jobs.S - 1, 256);
  pack_transpose_kernel<<<blocks, 256, 0, st>>>(args);
  return hipGetLastError();
}

}  // namespace t5mi
