// Host side of the bf16 MFMA GEMM: what it takes, sizes, dispatch to the epilogue families (gemm_mfma_*.hip), and the
// pointer tables of grouped launches.
#include "gemm_mfma.h"

namespace t5mi {

namespace {

struct PtrChunk { const void* p[64]; };
__global__ void fill_ptrs_kernel(PtrChunk c, int n, const void** dst) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = c.p[threadIdx.x];
}

__global__ void zero_split_kernel(GemmEpi e, int M, int N) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)M * N) return;
  const int m = (int)(idx / N), n = (int)(idx % N);
  const int which = n / e.split_n, nn = n - which * e.split_n;
  float* dst = (float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2);
  dst[(size_t)m * e.ld0 + nn] = 0.f;
}

// out[m][n] (+)= partials[0][m][n] + partials[1][m][n] + ... in that order; out as in EPI_SPLIT_F32.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmEpi e, int M, int N, int slices) {
  const int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;  // N % 4 == 0 (checked by the launcher)
  if (idx >= (int64_t)M * N) return;
  const size_t mn = (size_t)M * N;
  const float* partials = (const float*)e.aux0;
  f32x4 acc = *reinterpret_cast<const f32x4*>(partials + idx);
  for (int s = 1; s < slices; ++s) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(partials + (size_t)s * mn + idx);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] += v[q];
  }
  const int m = (int)(idx / N), n = (int)(idx % N);
  const int which = n / e.split_n, nn = n - which * e.split_n;  // split_n % 4 == 0: the four columns share an output
  float* dst = (float*)(which == 0 ? e.out0 : which == 1 ? e.out1 : e.out2) + (size_t)m * e.ld0 + nn;
  if (e.accumulate) {
    const f32x4 old = *reinterpret_cast<const f32x4*>(dst);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] += old[q];
  }
  *reinterpret_cast<f32x4*>(dst) = acc;
}

}  // namespace

hipError_t launch_zero_split(const GemmEpi& e, int M, int N, hipStream_t st) {
  zero_split_kernel<<<ceil_div((int64_t)M * N, 256), 256, 0, st>>>(e, M, N);
  return hipGetLastError();
}
hipError_t launch_splitk_reduce(const GemmEpi& e, int M, int N, int slices, hipStream_t st) {
  splitk_reduce_kernel<<<ceil_div((int64_t)M * N / 4, 256), 256, 0, st>>>(e, M, N, slices);
  return hipGetLastError();
}

bool gemm_mfma_supported(const GemmDesc& g, const GemmEpi& e) {
  if (g.in_type != IN_BF16) return false;
  if (g.nseg < 1 || g.nseg > 3) return false;
  if (g.a_kc != g.b_kc) return false;  // implemented: both k-contiguous, or both m/n-contiguous
  for (int s = 0; s < g.nseg; ++s) {
    const GemmSeg& sg = g.seg[s];
    if (g.a_kc ? (sg.K < KQ || sg.K % KQ != 0) : sg.K < 1) return false;
    if (sg.lda % 8 != 0 || sg.ldb % 8 != 0) return false;
    if (sg.lda != g.seg[0].lda || sg.ldb != g.seg[0].ldb) return false;
    if (((uintptr_t)sg.A | (uintptr_t)sg.B) & 15) return false;
  }
  if (g.M < 8 || g.N < 8) return false;
  // per-lane byte offsets are 32-bit
  if ((uint64_t)(g.a_kc ? g.M : KQ) * g.seg[0].lda * 2 >= (1ull << 32)) return false;
  if ((uint64_t)(g.b_kc ? g.N : KQ) * g.seg[0].ldb * 2 >= (1ull << 32)) return false;
  if (!g.a_kc && (g.M % 8 != 0 || g.N % 8 != 0)) return false;
  switch (e.kind) {
    case EPI_STORE: case EPI_RESID: case EPI_GEGLU_BWD:
      return g.a_kc == 1;
    case EPI_GEGLU_FWD:
      return g.a_kc == 1 && g.N % 64 == 0 && e.out_type == IN_BF16;
    case EPI_SPLIT_F32:
      if (g.ngroups > 1 && (!g.groups || !e.accumulate)) return false;
      return g.a_kc == 0 && g.nseg == 1;  // k may be split into slices: one segment only
    default:
      return false;
  }
}

int gemm_wgrad_slices(const GemmDesc& g, const GemmEpi& e) {
  bool big;
  int split_k;
  wgrad_plan(g, e, 1, big, split_k);
  return split_k;
}

size_t gemm_split_partials_bytes(const GemmDesc& g, const GemmEpi& e) {
  if (e.kind != EPI_SPLIT_F32 || g.ngroups > 1) return 0;
  bool big;
  int split_k;
  wgrad_plan(g, e, 1, big, split_k);
  return split_k > 1 ? (size_t)split_k * (size_t)g.M * (size_t)g.N * sizeof(float) : 0;
}

hipError_t launch_fill_ptrs(const void* const* ptrs, int n, const void** dst, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += 64) {
    PtrChunk c;
    const int m = n - i0 < 64 ? n - i0 : 64;
    for (int i = 0; i < 64; ++i) c.p[i] = i < m ? ptrs[i0 + i] : nullptr;
    fill_ptrs_kernel<<<1, 64, 0, st>>>(c, m, dst + i0);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

hipError_t launch_gemm_mfma(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  switch (e.kind) {
    case EPI_STORE: return launch_gemm_mfma_store(g, e, st);
    case EPI_RESID: return launch_gemm_mfma_resid(g, e, st);
    case EPI_GEGLU_FWD: return launch_gemm_mfma_geglu_fwd(g, e, st);
    case EPI_GEGLU_BWD: return launch_gemm_mfma_geglu_bwd(g, e, st);
    case EPI_SPLIT_F32: return g.ngroups > 1 ? launch_gemm_mfma_split_grouped(g, e, st) : launch_gemm_mfma_split(g, e, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace t5mi
