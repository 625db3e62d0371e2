// Fused attention for gfx950 (bf16 MFMA 32x32x16, float32 online softmax): self-attention with the
// T5 relative-position bias (BIAS, optionally CAUSAL), or cross-attention of S queries over Sk keys
// of another sequence without bias or mask.  The S x Sk scores never leave registers.
//
// Forward and the dq kernel give each lane one query: scores are computed transposed,
// S^T = K Q^T, so the MFMA result layout puts a query in lane%32 and 16 keys of a 32-key tile in
// the lane's registers.  Row maxima and sums are then register reductions plus one exchange between
// the two lane halves, and the probabilities feed the second matmul (O^T = V^T P^T) straight from
// the result registers: the contraction index of an MFMA may be permuted freely as long as both
// operands use the same permutation, and the V^T operand is fetched with that permutation by the
// LDS transpose load.  The dk/dv kernel mirrors this with one key per lane (S = Q K^T).
//
// Dropout of the probabilities (DROP): the keep decision of element ((b*H + h)*S + i, j) comes from the counter-based
// generator in the forward, which leaves it as a bit for the backward (AttnDims::keep; 1/16 of the bytes of a bf16 score):
// one more instruction an element in the forward, two or three instead of nine in each kernel of the backward.  128 x 512
// tokens, 12 heads: forward 242 -> 250 us, dq 399 -> 352, dk/dv 371 -> 318.  A lane of the forward and of dq owns a query and
// 32 keys of a 64-key tile: one word a tile, which dq loads a tile ahead; the dk/dv kernel stages the words of its two key
// tiles and a query tile in LDS by DMA.  The factor 1/(1 - rate) of the kept probabilities is applied to the finished O and
// dV accumulators, and to dP before dvec is subtracted.
//
// Sequence lengths need not be multiples of the tile sizes: tiles are rounded up, rows past the end are
// fetched from the last valid row, keys past the end are masked like causal ones, and queries past the end
// are neither stored nor counted in the bias gradient.
//
// The bias is Toeplitz: bias[h,i,j] = diag[h][j - i + S - 1], and constant from the first distance of the last bucket
// on.  Each workgroup stages the diagonals up to there in LDS (BiasWin), or, where that window would be long, the
// slice of the per-head diagonal vector it can touch (S + tile - 1 floats).
#include <algorithm>
#include <type_traits>
#include "kernels.h"

namespace t5mi {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef __attribute__((address_space(3))) short4v lds_short4;
typedef __attribute__((ext_vector_type(8))) short short8v;

// Row-dependent XOR applied to the 16-byte chunk index of a [rows][DK] bf16 tile.  Chosen so that
// both access patterns are bank-conflict free: 16 consecutive rows x one chunk (ds_read_b128
// operand reads) and 4 consecutive rows x 4 consecutive chunks (transpose reads).
template <int DK>
__device__ __forceinline__ int row_swz(int row) {
  if constexpr (DK == 64)
    return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1);
  else
    return ((row & 1) << 2) | (((row >> 1) & 1) << 3) | ((row >> 2) & 1) | (((row >> 3) & 1) << 1);
}
template <int DK>
__device__ __forceinline__ int tile_off(int row, int chunk) {
  return row * (DK * 2) + ((chunk ^ row_swz<DK>(row)) << 4);
}

// Cooperative copy of `rows` rows of DK bf16 (row r at src + r*ld) into a swizzled LDS tile.
// Rows at or beyond `valid` are clamped to the last valid row (their results are never used).
template <int DK, int NT>
__device__ __forceinline__ void load_tile(char* dst, const bf16* __restrict__ src, size_t ld, int rows,
                                          int valid, int tid) {
  constexpr int CPR = DK / 8;
  for (int q = tid; q < rows * CPR; q += NT) {
    const int row = q / CPR, ch = q % CPR;
    const int rs = row < valid ? row : valid - 1;
    *reinterpret_cast<u32x4*>(dst + tile_off<DK>(row, ch)) =
        *reinterpret_cast<const u32x4*>(src + (size_t)rs * ld + ch * 8);
  }
}

// DMA descriptor of one [ROWS][DK] bf16 tile for a 4-wave workgroup: the tile is ROWS*DK*2/1024
// blocks of 1 KB, wave w copies blocks w, w+4, ...  The swizzle of tile_off() is applied on the
// global side: the lane that owns LDS slot (row, physical chunk) fetches the logical chunk.
template <int DK, int ROWS>
struct TileDma {
  static constexpr int PER_WAVE = ROWS * DK * 2 / 1024 / 4;
  uint32_t voff[PER_WAVE];
  // valid: rows of the tile that exist; the others fetch the last valid row again (their values are masked
  // or never stored), so that a ragged last tile reads nothing outside the operand
  __device__ __forceinline__ void init(int wave, int lane, size_t ld_elems, int valid = ROWS) {
    constexpr int CPR = DK / 8;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int slot = (wave + i * 4) * 64 + lane;
      const int row = slot / CPR, pch = slot % CPR;
      const int src = row < valid ? row : valid - 1;
      voff[i] = (uint32_t)(src * ld_elems * 2) + (uint32_t)((pch ^ row_swz<DK>(row)) << 4);
    }
  }
  __device__ __forceinline__ void issue(uint32_t lds_addr, const void* sbase, int wave) const {
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) dma_1k(lds_addr + (wave + i * 4) * 1024, sbase, voff[i]);
  }
};

// All DMA issued so far has landed, this wave's LDS traffic is complete, and every wave is here.
// 64 floats global -> LDS, one per lane (global_load_lds_dword): lane L fetches 4 bytes at sbase + voff and they
// land at LDS address lds_addr + 4*L.  Same ordering rules as the 1 KB form.
__device__ __forceinline__ void dma_64f(uint32_t lds_addr, const void* sbase, uint32_t voff) {
  lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase));
}

__device__ __forceinline__ void dma_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Operand with 8 consecutive channels of row (base + lane%32): k-step kk covers channels kk*16..+15.
template <int DK>
__device__ __forceinline__ bf16x8 frag_rows(const char* tile, int base, int kk, int lane) {
  return *reinterpret_cast<const bf16x8*>(tile + tile_off<DK>(base + (lane & 31), kk * 2 + (lane >> 5)));
}

// Transposed operand: MFMA row = channel (cbase + lane%32), contraction over tile rows.  Slot jj of
// lane half g holds tile row  rbase + 8*(jj/4) + 4*g + jj%4  -- the order in which the 32x32 result
// layout keeps rows 8*(r/4) + 4*g + r%4 in consecutive registers.
template <int DK>
__device__ __forceinline__ bf16x8 frag_cols_tr(const char* tile, int rbase, int cbase, int lane) {
  const int i16 = lane & 15;
  const int ch_e = cbase + (((lane >> 4) & 1) << 4) + ((i16 & 3) << 2);  // first of 4 channels addressed
  const int row0 = rbase + ((lane >> 5) << 2) + (i16 >> 2);
  const int row1 = row0 + 8;
  const int o0 = tile_off<DK>(row0, ch_e >> 3) + ((ch_e & 7) << 1);
  const int o1 = tile_off<DK>(row1, ch_e >> 3) + ((ch_e & 7) << 1);
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(tile + o0));
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(tile + o1));
  short8v r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int first) {
  bf16x8 o;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (bf16)v[first + i];
  return o;
}

// A wavefront's 32 result rows (row = lane%32, channels in registers), times f, to global rows of DK bf16 (row r at
// dst + r*ld, the first `valid` of them).  The registers of a lane are 8-byte pieces of a row: stored as they are, an
// instruction touches 32 rows with 16 bytes each and the address path takes a cycle or two per row.  They go through
// LDS (32 rows of DK*2 + 16 bytes per wavefront, in the tile stages, free by now) and leave as whole rows.  Measured
// (before -> now): cross-attention dk/dv at 128 x (114 over 512) tokens, 12 heads, which stores half of all it moves,
// 149 -> 108 us; dk/dv at 32 x 1024, 32 heads, 633 -> 597; forward 379 -> 371; at 64 x 512, 6 heads, 75 -> 69 and 51 -> 48.
template <int DK, int CT>
__device__ __forceinline__ void store_rows(char* lds, const f32x16 (&acc)[CT], float f, bf16* dst, size_t ld, int valid,
                                           int lane) {
  constexpr int RB = DK * 2 + 16, LPR = DK / 8, RPI = 64 / LPR;
  const int row = lane & 31, g = lane >> 5;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)(acc[ct][rq * 4 + e] * f);
      *reinterpret_cast<bf16x4*>(lds + row * RB + (ct * 32 + rq * 8 + g * 4) * 2) = o;
    }
  // (the wavefront's own rows: LDS operations of one wavefront complete in order)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + lane / LPR, ch = lane % LPR;
    const u32x4 v = *reinterpret_cast<const u32x4*>(lds + r * RB + ch * 16);
    if (r < valid) *reinterpret_cast<u32x4*>(dst + (size_t)r * ld + ch * 8) = v;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Workgroup -> (tile, head, batch).  Workgroup ids are dealt round-robin to the 8 XCDs; the tiles of
// one (batch, head) share its K/V (or Q/dO) stream, so they are given ids that are congruent mod 8
// and adjacent in dispatch order: they run on one XCD at about the same time and share its L2.
__device__ __forceinline__ void decode_block(int n_tiles, int H, int B, int& tile, int& h, int& b) {
  const int bh_total = H * B;
  const int id = blockIdx.x;
  int bh;
  if ((bh_total & 7) == 0) {
    const int xcd = id & 7, j = id >> 3;
    bh = (j / n_tiles) * 8 + xcd;
    tile = j % n_tiles;
  } else {
    bh = id / n_tiles;
    tile = id % n_tiles;
  }
  h = bh % H;
  b = bh / H;
}

// dg[t] = src[idx_of(t)] * log2(e) for t in [0, n): 256 threads, four independent loads in flight per
// thread (the slice is short, so its load latency is all there is to hide).
template <typename F>
__device__ __forceinline__ void fill_bias_slice(float* dg, const float* __restrict__ src, int n, int tid, F idx_of) {
  for (int t0 = tid; t0 < n; t0 += 4 * 256) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * 256;
      v[q] = src[idx_of(t < n ? t : n - 1)];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * 256;
      if (t < n) dg[t] = v[q] * kLog2e;
    }
  }
}

// Window of diagonals (WIN).  A 32x32 sub-tile of scores whose first key lies m after its first query (m a multiple of
// 32) touches the diagonals m - 31 .. m + 31; from |m| = M on they all have the bias of the last bucket, so m is clamped
// to [-M, M] and a window of 2M + 63 values serves any length.  Causal: the diagonals of later keys hold -infinity, which
// is the mask, and m = 32 stands for all sub-tiles that are masked whole.  The window is held four times, copy c shifted
// by c values: whatever the lane's diagonal modulo 4, the bias of four neighbouring diagonals is then one aligned 16-byte
// read.  (An LDS instruction takes the same 4-5 cycles for 4 and for 16 bytes a lane; read one by one the bias values were
// half of the forward's LDS instructions, a third of the others'.)  The copies are 16 banks apart, so that 16 neighbouring
// lanes (4 copies x 4 positions) meet no bank twice.
// Against the slice of S + 127 diagonals with mask instructions, us: dq 16 x 2048 causal, 16 heads of 128 channels 911 -> 622
// (80 instead of 84 KB: two workgroups on a compute unit), 1 x 4096, 32 heads of 64 channels 285 -> 256; causal forward
// 32 x 512, 12 heads 46 -> 40, 8 x 2048 111 -> 98 (no mask to compute: 126 registers instead of 167); the others 1-3 %.
// A masked score that is infinite or NaN would pass that bias, so where the diagonal cuts a sub-tile the kernels also choose:
// queries and keys, finite or not, add nothing through a masked score.
struct BiasWin {
  int M, top, stride;  // top: largest m that is told apart
  __host__ __device__ BiasWin(int S, int far, bool causal) {
    M = ((far < S ? far : S) + 31 + 31) / 32 * 32;
    top = causal ? 32 : M;
    stride = (M + top + 63 - 16 + 63) / 64 * 64 + 16;
  }
  __host__ __device__ int floats() const { return 4 * stride; }
  // offset in a copy that belongs to a sub-tile
  __device__ __forceinline__ int at(int m) const { return (m < -M ? -M : m > top ? top : m) + M; }
  // 256 threads; in log2 units
  template <bool CAUSAL>
  __device__ __forceinline__ void fill(float* win, const float* __restrict__ diag_h, int S, int tid) const {
    for (int t = tid; t < M + top + 63; t += 256) {
      const int delta = t - M - 31;
      int idx = delta + S - 1;
      idx = idx < 0 ? 0 : idx > 2 * S - 2 ? 2 * S - 2 : idx;  // (past the ends: masked, or constant)
      const float v = CAUSAL && delta > 0 ? -INFINITY : diag_h[idx] * kLog2e;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (t >= c) win[c * stride + t - c] = v;
    }
  }
  // a lane's base: the diagonals u .. u + 3 of the window of a sub-tile are the four values from lane(win, u) + at(m) on
  __device__ __forceinline__ const float* lane(const float* win, int u) const { return win + (u & 3) * stride + (u & ~3); }
};
// Registers R.. of a 32x32 ds sub-tile (S^T layout), each rotated across the 32 lanes of its half by
// its key offset, summed into `tot`; `lo` gets the part whose source query did not wrap around
// (lp = 31 - query index of the receiving lane).  The rotation amount must be an immediate.
// The rotations are issued in groups of eight before any of their results is used: one at a time, each
// is followed by a wait for its trip through the LDS crossbar.
template <int R>
__device__ __forceinline__ float diag_rot(const f32x16& ds) {
  constexpr int kj0 = ((R >> 2) << 3) + (R & 3);  // key offset of register R (without the half's + 4)
  const float x = ds[R];  // (a plain float first: bit-casting the vector element itself picks element 0)
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), 0xC000 | (kj0 << 5)));
}
template <int R0>
__device__ __forceinline__ void diag_accum8(const f32x16& ds, int lp, float& lo, float& tot) {
  const float v0 = diag_rot<R0>(ds), v1 = diag_rot<R0 + 1>(ds), v2 = diag_rot<R0 + 2>(ds), v3 = diag_rot<R0 + 3>(ds);
  const float v4 = diag_rot<R0 + 4>(ds), v5 = diag_rot<R0 + 5>(ds), v6 = diag_rot<R0 + 6>(ds), v7 = diag_rot<R0 + 7>(ds);
  __builtin_amdgcn_sched_barrier(0);
  const float v[8] = {v0, v1, v2, v3, v4, v5, v6, v7};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int r = R0 + q;
    const int kj0 = ((r >> 2) << 3) + (r & 3);
    lo += lp >= kj0 ? v[q] : 0.f;
    tot += v[q];
  }
}
__device__ __forceinline__ void diag_accum(const f32x16& ds, int lp, float& lo, float& tot) {
  diag_accum8<0>(ds, lp, lo, tot);
  diag_accum8<8>(ds, lp, lo, tot);
}

// Number of 32-key blocks on each side of a wave's queries whose diagonals are resolved one by one in
// the dq kernel: offsets up to far + 30 can fall into a sub-tile that is not entirely saturated.
__host__ __device__ inline int attn_dq_window_blocks(int S, int far) {
  const int nb = (far + 30) / 32, cap = (S + 31) / 32 - 1;
  return nb < cap ? nb : cap;
}
// Floats per workgroup row of the reproducible bias-gradient buffer: a window is at most 64 * ceil(S / 32)
// entries wide (+ 4 for the upper lane half) and two sums of the saturated buckets follow it.
__host__ __device__ inline int attn_ddiag_part_stride(int S) { return 64 * ((S + 31) / 32) + 8; }
// words between two key tiles of AttnDims::keep: two lane halves of a row of queries each
__host__ __device__ inline size_t attn_keep_stride(int S) { return (size_t)2 * ((S + 127) / 128 * 128); }
// the words of a key tile and lane half, one per query
__device__ __forceinline__ uint32_t* keep_row(const AttnDims& a, size_t bh, int tile, int half) {
  const size_t stride = attn_keep_stride(a.S);
  return a.keep + (bh * ((a.Sk + 63) / 64) + tile) * stride + half * (stride / 2);
}
// Whether `here` holds in any lane of a workgroup of four wavefronts.  flags: 16 bytes of LDS that no wavefront uses.
__device__ __forceinline__ bool any_in_workgroup(bool here, char* flags, int wave, int lane) {
  const bool mine = __builtin_amdgcn_ballot_w64(here) != 0;
  if (lane == 0) reinterpret_cast<int*>(flags)[wave] = mine;
  __syncthreads();
  const int4 f = *reinterpret_cast<const int4*>(flags);
  return __builtin_amdgcn_readfirstlane(f.x | f.y | f.z | f.w) != 0;
}
// word << 4 | this lane's bits of four of the wave's masks, each as one add with carry.  A vector instruction that reads a scalar
// register as a mask needs two wait states after the vector instruction that wrote it, and the compiler does not count them
// into an asm block: they stand at its head, once for the four.
__device__ __forceinline__ uint32_t shift_in4(uint32_t word, const uint64_t (&mask)[4]) {
  uint64_t carry_out;
  asm("s_nop 1\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %2\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %3\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %4\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %5"
      : "+v"(word), "=&s"(carry_out)
      : "s"(mask[0]), "s"(mask[1]), "s"(mask[2]), "s"(mask[3]));
  return word;
}
// all ones where bit 31 - n of the word is set, else 0 (the builtin: a shift and a test become a comparison and selects)
__device__ __forceinline__ int keep_mask(uint32_t word, int n) { return __builtin_amdgcn_sbfe(word, 31 - n, 1); }
__device__ __forceinline__ float keep_if(int mask, float x) { return __builtin_bit_cast(float, mask & __builtin_bit_cast(int, x)); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// max(x of this lane, x of the lane 32 away).  v_permlane32_swap exchanges lanes 32..63 of its first operand with
// lanes 0..31 of its second: started from two copies of x, every lane then holds its own value in one of the two
// registers and its partner's in the other.  One vector instruction through no memory, where the generic shuffle
// is an LDS round trip (ds_bpermute) on the dependent chain of every key tile.  (The s_nop covers the wait states
// between a vector write of the operands and the swap; the compiler's builtin for this instruction returned the
// same half in both results when tried here, hence the assembly.)
__device__ __forceinline__ float max_across_halves(float x) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}

// ------------------------------------------------------------------------------------------------
// Forward.  grid (ceil(S/128), H, B), 256 threads; wave w owns queries i0 + 32w + lane%32.
// ------------------------------------------------------------------------------------------------
template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN>
__global__ __launch_bounds__(256, 2) void attn_fwd_mfma_kernel(AttnIO io, const float* __restrict__ diag,
                                                            bf16* __restrict__ c, float* __restrict__ lse,
                                                            AttnDims a) {
  constexpr int BR = 128, BC = 64, KS = DK / 16, CT = DK / 32;
  constexpr int TILE = BC * DK * 2, STG = 2 * TILE;  // a stage holds a K tile then a V tile
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  float* dg = reinterpret_cast<float*>(smem + 2 * STG);  // window, or [S + BR - 1], log2 units (BIAS only)

  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.S, Sk = a.Sk, I = a.H * DK;
  const size_t ldq = (size_t)io.ldq, ld = (size_t)io.ldkv;
  int qt, h, b;
  decode_block((S + BR - 1) / BR, a.H, a.B, qt, h, b);
  if (CAUSAL) qt = (S + BR - 1) / BR - 1 - qt;  // heavy causal tiles first
  const int i0 = qt * BR;
  const int i_loc = wave * 32 + (lane & 31);
  const int i = i0 + i_loc;
  const int i_ld = i < S ? i : S - 1;
  const bf16* kbase = (const bf16*)io.k + (size_t)b * Sk * ld + h * DK;
  const bf16* vbase = (const bf16*)io.v + (size_t)b * Sk * ld + h * DK;

  bf16x8 qf[KS];
  {
    const bf16* qrow = (const bf16*)io.q + ((size_t)b * S + i_ld) * ldq + h * DK;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16 + g * 8);
    // (an empty use: the wait for these loads belongs here, not at their first use inside the loop, where it
    // would also wait for the tile DMA of every iteration -- see the dk/dv kernel)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" ::"v"(qf[kk]));
  }
  const BiasWin win(S, a.far, CAUSAL);
  if constexpr (WIN) {
    win.fill<CAUSAL>(dg, diag + (size_t)h * (2 * S - 1), S, tid);
  } else if constexpr (BIAS) {
    const float* dgh = diag + (size_t)h * (2 * S - 1);
    fill_bias_slice(dg, dgh, S + BR - 1, tid, [&](int t) {
      const int idx = t - (i0 + BR - 1) + (S - 1);  // delta + S - 1
      return idx < 0 ? 0 : idx;                     // only reachable by clamped (unused) queries
    });
  }
  const int i_w0 = i0 + wave * 32;                               // first query of this wave
  const float* dgw = win.lane(dg, 31 - (lane & 31) + (g << 2));  // (WIN)
  const float sc = a.scale * kLog2e;
  const int dg_base = BR - 1 - i_loc;  // dg[dg_base + j] = bias(j - i)
  uint32_t k1 = 0;  // dropout row key of this lane's query
  if constexpr (DROP) k1 = drop_row_pre(drop_row_key(a.drop, (uint32_t)(((size_t)b * a.H + h) * S + i_ld)));
  // this lane's words (rows of queries are padded to whole workgroups)
  uint32_t* keep_q = DROP ? keep_row(a, (size_t)b * a.H + h, 0, g) + i : nullptr;

  f32x16 oT[CT];
  float m, l;

  int n_kv = (Sk + BC - 1) / BC;
  if (CAUSAL) {
    const int last = (i0 + BR < S ? i0 + BR : S);
    n_kv = (last + BC - 1) / BC;
  }
  // K/V tiles are double buffered: tile jt+1 is in flight (DMA) while tile jt is used.  td_tail fetches the
  // last tile of a key sequence whose length is not a multiple of the tile.
  TileDma<DK, BC> td, td_tail;
  td.init(wave, lane, ld);
  td_tail.init(wave, lane, ld, Sk % BC ? Sk % BC : BC);
  const int jt_tail = Sk % BC ? Sk / BC : -1;  // index of the ragged tile, if there is one
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
  // select: masked scores count as zero before the window's -infinity is added.  Without dropout the tiles are gone through
  // without it, and only a workgroup that finds a NaN in its sums (which a masked score that is not finite leaves there) takes
  // them a second time: the branch around the select cuts the loop's block in two (64 channels, 1 x 1024 tokens, 12 heads 18
  // -> 21 us, 4 x 333 10 -> 11, 64 x 512, 6 heads 38.1 -> 40.4; like this 18, 10 and 38.4).  With dropout it costs nothing.
  constexpr bool TWICE = CAUSAL && WIN && !DROP;
#pragma unroll
  for (int select = CAUSAL && WIN && !TWICE; select < (CAUSAL && WIN ? 2 : 1); ++select) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) oT[ct][r] = 0.f;
    m = -INFINITY;
    l = 0.f;
    (jt_tail == 0 ? td_tail : td).issue(lds0, kbase, wave);
    (jt_tail == 0 ? td_tail : td).issue(lds0 + TILE, vbase, wave);
    for (int jt = 0; jt < n_kv; ++jt) {
      const int j0 = jt * BC;
      dma_wait_barrier();  // tile jt landed; every wave is done with the other stage
      if (jt + 1 < n_kv) {
        const uint32_t nxt = lds0 + ((jt + 1) & 1) * STG;
        const TileDma<DK, BC>& tn = jt + 1 == jt_tail ? td_tail : td;
        tn.issue(nxt, kbase + (size_t)(j0 + BC) * ld, wave);
        tn.issue(nxt + TILE, vbase + (size_t)(j0 + BC) * ld, wave);
      }
      const char* Kt = smem + (jt & 1) * STG;
      const char* Vt = Kt + TILE;

      f32x16 sT[BC / 32];
#pragma unroll
      for (int kt = 0; kt < BC / 32; ++kt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sT[kt][r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
          sT[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DK>(Kt, kt * 32, kk, lane), qf[kk], sT[kt],
                                                          0, 0, 0);
      }
      if constexpr (DK == 128) {
        // K operands requested two contraction steps ahead of the products that use them
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
        for (int q = 0; q + 3 < (BC / 32) * KS; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
      }
      float mx = -INFINITY;
      // only tiles that reach above the diagonal of this wave's queries pay for the mask (wave-uniform)
      // (and the tile that reaches past the last key)
      // (causal with the window: the mask is in the bias, and a key past the end comes after every query)
      const bool on_diag = CAUSAL && WIN ? false : (CAUSAL && j0 + BC - 1 > i_w0) || j0 + BC > Sk;
      const float* dgt[BC / 32];
#pragma unroll
      for (int kt = 0; kt < BC / 32; ++kt) dgt[kt] = dgw + win.at(j0 + kt * 32 - i_w0);
      if (select && j0 + BC - 1 > i_w0) {  // (wave-uniform)
#pragma unroll
        for (int kt = 0; kt < BC / 32; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (kt * 32 + ((r >> 2) << 3) + (r & 3) > i - j0 - (g << 2)) sT[kt][r] = 0.f;
      }
      if (on_diag) {
#pragma unroll
        for (int kt = 0; kt < BC / 32; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = j0 + kt * 32 + ((r >> 2) << 3) + (g << 2) + (r & 3);
            // (a masked key's bias slot may lie outside the slice: clamp the index, the value is discarded)
            const int jb = j < Sk ? j : Sk - 1;
            float s;
            if constexpr (WIN) s = fmaf(sT[kt][r], sc, (*reinterpret_cast<const f32x4*>(dgt[kt] + ((r >> 2) << 3)))[r & 3]);
            else s = BIAS ? fmaf(sT[kt][r], sc, dg[dg_base + jb]) : sT[kt][r] * sc;
            if ((CAUSAL && j > i) || j >= Sk) s = -INFINITY;
            sT[kt][r] = s;
            mx = fmaxf(mx, s);
          }
      } else {
#pragma unroll
        for (int kt = 0; kt < BC / 32; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = j0 + kt * 32 + ((r >> 2) << 3) + (g << 2) + (r & 3);
            float s;
            if constexpr (WIN) s = fmaf(sT[kt][r], sc, (*reinterpret_cast<const f32x4*>(dgt[kt] + ((r >> 2) << 3)))[r & 3]);
            else s = BIAS ? fmaf(sT[kt][r], sc, dg[dg_base + j]) : sT[kt][r] * sc;
            sT[kt][r] = s;
            mx = fmaxf(mx, s);
          }
      }
      mx = max_across_halves(mx);
      const float m_new = fmaxf(m, mx);
      // (a bias table may mask all keys so far, with -inf or with the lowest number: then there is no maximum yet)
      const float base = BIAS && m_new == -INFINITY ? 0.f : m_new;
      const float alpha = fast_exp2(m - base);
      m = m_new;
      float ls = 0.f;
      uint32_t kx = 0, kept = 0;
      uint64_t keeps[4];
      if constexpr (DROP) kx = k1 ^ (uint32_t)(j0 | (g << 2));
#pragma unroll
      for (int kt = 0; kt < BC / 32; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = fast_exp2(sT[kt][r] - base);
          ls += p;  // the normaliser is that of the undropped probabilities
          if constexpr (DROP) {
            // (key index = tile start | lane half << 2 | constant of the register, disjoint bits)
            const uint32_t c = (uint32_t)(kt * 32 + ((r >> 2) << 3) + (r & 3));
            const bool keep = drop_keep16(a.drop, kx ^ c);
            keeps[r & 3] = __builtin_amdgcn_ballot_w64(keep);
            if ((r & 3) == 3) kept = shift_in4(kept, keeps);
            float pk = keep ? p : 0.f;
            asm("" : "+v"(pk));  // (a select of the bf16 values instead would cost a conversion and a permute each)
            sT[kt][r] = pk;
          } else {
            sT[kt][r] = p;
          }
        }
      if constexpr (DROP) keep_q[jt * attn_keep_stride(S)] = kept;
      l = l * alpha + ls;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) oT[ct][r] *= alpha;
#pragma unroll
      for (int kt = 0; kt < BC / 32; ++kt)
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          const bf16x8 pf = pack8(sT[kt], mm * 8);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            oT[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_tr<DK>(Vt, kt * 32 + mm * 16, ct * 32, lane),
                                                            pf, oT[ct], 0, 0, 0);
        }
    }
    __syncthreads();  // every wave is done with the tiles
    if (TWICE && !select && !any_in_workgroup(__builtin_isnan(l), smem + 2 * STG - 16, wave, lane)) break;
  }
  const float l_tot = l + __shfl_xor(l, 32, 64);
  store_rows<DK>(smem + wave * 32 * (DK * 2 + 16), oT, (DROP ? a.drop.scale : 1.f) / l_tot,
                 c + ((size_t)b * S + i0 + wave * 32) * I + h * DK, (size_t)I, S - i0 - wave * 32, lane);
  if (i < S) {
    if (g == 0) lse[((size_t)b * a.H + h) * S + i] = (m + __builtin_amdgcn_logf(l_tot)) * kLn2;
  }
}

// ------------------------------------------------------------------------------------------------
// dq and the per-diagonal bias gradient.  Same ownership as the forward (lane = query).  The kernel also
// forms dvec[b,h,i] = sum_c dO[b,i,h,c] * O[b,i,h,c] for its query -- the two lane halves hold the two halves
// of the dO row as MFMA operands already, so it costs one read of the O row -- and writes it for the
// dk/dv kernel, which runs after this one.
//
// Bias gradient: ddiag[delta] = sum over (b, i) of ds[i, i + delta].  In the MFMA result layout a
// register holds one key offset for 32 queries, i.e. 32 consecutive diagonals, and a different
// register holds the same diagonals shifted by its key offset.  Rotating each register across the
// 32 lanes by its key offset (ds_swizzle rotate mode: a crossbar permute, no LDS memory) lines the
// diagonals up: after the rotation lane p holds, from every register, a value of diagonal slot
// 31 - p or 63 - p of the sub-tile's 63 diagonals.  Each lane therefore owns two slots per
// sub-tile, adds into them in a per-(wave, lane half) window in LDS with plain read-modify-write
// (the owner of a window entry never changes, so no synchronisation until the final flush), and the
// workgroup adds the eight windows up and issues one global atomic per diagonal.  Sub-tiles whose
// every offset lies in the saturated last bucket (|delta| >= far) skip all that and add into one
// scalar per lane; it is credited to the outermost diagonal, which is in the same bucket.
// ------------------------------------------------------------------------------------------------
template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN>
// (three waves per SIMD with 64 channels; with dropout only causal and with the window: the others would spill.  32 x 512
// tokens, 12 heads, causal 86 -> 75 us, 128 x 512 not causal 351 -> 393; slice, causal, 2 x 4096 253 us with either)
__global__ __launch_bounds__(256, DK == 64 && (!DROP || (CAUSAL && WIN)) ? 3 : 2) void attn_bwd_dq_mfma_kernel(AttnIO io,
                                                               const bf16* __restrict__ o,
                                                               const bf16* __restrict__ dout,
                                                               const float* __restrict__ diag,
                                                               const float* __restrict__ lse,
                                                               float* __restrict__ dvec,
                                                               float* __restrict__ ddiag,
                                                               float* __restrict__ ddiag_part,
                                                               AttnDims a) {
  constexpr int BR = 128, BC = 64, KS = DK / 16, CT = DK / 32;
  // The causal form with dropout has no register to spare for the third wave: the keep words by a uniform base and one 32-bit
  // offset, the ragged tile's offsets formed where it is fetched (with both kept, 6 registers with the window and 9 with the
  // slice were spilled, and reloaded between the tiles' DMA: slice, 2 x 4096 tokens, 12 heads 310 -> 253 us, 32 x 620 137 ->
  // 115; window, 1 x 4096 154 -> 144, 4 x 333 20.0 -> 17.7).
  constexpr bool LEAN = DK == 64 && DROP && CAUSAL;
  constexpr int TILE = BC * DK * 2, STG = 2 * TILE;  // a stage holds a K tile then a V tile
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int far = a.far;
  const BiasWin win(a.S, far, CAUSAL);
  float* dg = reinterpret_cast<float*>(smem + 2 * STG);  // bias, log2 units: window, or [S + BR - 1]
  // Diagonal windows [4 waves][2 lane halves][W].  A sub-tile at key offset j0s - i_w0 = 32 m from
  // the wave's queries is resolved per diagonal for |m| <= nb; its slot u (0..62) lives at
  // (m + nb) * 32 + u, which is diagonal delta = 32 m + u - 31 (+ 4 for the upper lane half).
  const int nb = BIAS ? attn_dq_window_blocks(a.S, far) : 0, W = 32 * (2 * nb + 2);
  float* ddg_all = dg + (WIN ? win.floats() : a.S + BR - 1);

  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.S, Sk = a.Sk, I = a.H * DK;
  const size_t ldq = (size_t)io.ldq, ld = (size_t)io.ldkv;
  int qt, h, b;
  decode_block((S + BR - 1) / BR, a.H, a.B, qt, h, b);
  if (CAUSAL) qt = (S + BR - 1) / BR - 1 - qt;
  const int i0 = qt * BR;
  const int i_w0 = i0 + wave * 32;         // first query of this wave
  const int i_lw = lane & 31;              // query index inside the wave
  const int i_loc = wave * 32 + i_lw;
  const int i = i0 + i_loc;
  const int i_ld = i < S ? i : S - 1;      // queries past the end read the last row; their ds is forced to zero
  const bool q_ok = i < S;
  const bf16* kbase = (const bf16*)io.k + (size_t)b * Sk * ld + h * DK;
  const bf16* vbase = (const bf16*)io.v + (size_t)b * Sk * ld + h * DK;
  float* ddgw = ddg_all + (wave * 2 + g) * W + (31 - i_lw);  // this lane's first slot of block m = -nb

  bf16x8 qf[KS], dof[KS];
  float dsum = 0.f;  // this lane half's share of sum_c dO * O
  {
    const bf16* qrow = (const bf16*)io.q + ((size_t)b * S + i_ld) * ldq + h * DK;
    const bf16* drow = dout + ((size_t)b * S + i_ld) * I + h * DK;
    const bf16* orow = o + ((size_t)b * S + i_ld) * I + h * DK;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16 + g * 8);
      dof[kk] = *reinterpret_cast<const bf16x8*>(drow + kk * 16 + g * 8);
      const bf16x8 of = *reinterpret_cast<const bf16x8*>(orow + kk * 16 + g * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) dsum = fmaf((float)of[e], (float)dof[kk][e], dsum);
    }
    // (an empty use: see the forward kernel)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" ::"v"(qf[kk]), "v"(dof[kk]));
  }
  dsum += __shfl_xor(dsum, 32, 64);
  const size_t srow = ((size_t)b * a.H + h) * S + i_ld;
  // for the dk/dv kernel, which stages them per query tile by DMA: -dvec, and behind it -lse / scale
  const float lse_q = lse[srow];
  if (g == 0 && q_ok) {
    dvec[srow] = -dsum;
    dvec[(size_t)a.B * a.H * S + srow] = lse_q * (-1.f / a.scale);
  }
  const float nlse2 = -lse_q * kLog2e, ndv = -dsum;
  // this lane's words of keep decisions, and that of the next key tile
  const uint32_t* keep_q = DROP ? keep_row(a, (size_t)b * a.H + h, 0, LEAN ? 0 : g) + (LEAN ? 0 : i) : nullptr;  // (+ keep_i)
  const uint32_t keep_i = LEAN ? (uint32_t)(g * (int)(attn_keep_stride(S) / 2) + i) : 0;
  uint32_t kept_next = DROP ? keep_q[keep_i] : 0;
  // dP of a kept probability carries the factor 1/(1 - rate); that of a dropped one is zero
  auto dp_masked = [&](float dp, uint32_t kept, int n) {
    if constexpr (DROP) {
      int mask = keep_mask(kept, n);
      asm("" : "+v"(mask));  // (a constant bit would become a test and a select)
      return keep_if(mask, dp * a.drop.scale);
    } else {
      return dp;
    }
  };
  if constexpr (BIAS) {
    const float* dgh = diag + (size_t)h * (2 * S - 1);
    if constexpr (WIN)
      win.fill<CAUSAL>(dg, dgh, S, tid);
    else
      fill_bias_slice(dg, dgh, S + BR - 1, tid, [&](int t) {
        const int idx = t - (i0 + BR - 1) + (S - 1);  // delta + S - 1
        return idx < 0 ? 0 : idx;                     // only reachable by queries past the end
      });
    for (int t = tid; t < 8 * W; t += 256) ddg_all[t] = 0.f;
  }
  const float* dgw = win.lane(dg, 31 - i_lw + (g << 2));  // (WIN)
  const float sc = a.scale * kLog2e;
  const int dg_base = BR - 1 - i_loc;
  float far_neg = 0.f, far_pos = 0.f;

  f32x16 dqT[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) dqT[ct][r] = 0.f;

  const int n_kv = ((CAUSAL && i0 + BR < Sk ? i0 + BR : Sk) + BC - 1) / BC;
  TileDma<DK, BC> td, td_tail;  // td_tail: the last tile of a key sequence that does not fill it
  td.init(wave, lane, ld);
  if constexpr (!LEAN) td_tail.init(wave, lane, ld, Sk % BC ? Sk % BC : BC);
  const int jt_tail = Sk % BC ? Sk / BC : -1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
  auto issue = [&](int jt) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + (jt & 1) * STG;
    const bf16 *kt = kbase + (size_t)(jt * BC) * ld, *vt = vbase + (size_t)(jt * BC) * ld;
    if (LEAN && jt == jt_tail) {
      int rows = Sk % BC;
      asm volatile("" : "+s"(rows));  // (opaque: its offsets stay out of the loop's registers)
      TileDma<DK, BC> tail;
      tail.init(wave, lane, ld, rows);
      tail.issue(dst, kt, wave);
      tail.issue(dst + TILE, vt, wave);
    } else {
      const TileDma<DK, BC>& t = !LEAN && jt == jt_tail ? td_tail : td;
      t.issue(dst, kt, wave);
      t.issue(dst + TILE, vt, wave);
    }
  };
  issue(0);
  for (int jt = 0; jt < n_kv; ++jt) {
    const int j0 = jt * BC;
    dma_wait_barrier();  // tile jt landed; every wave is done with the other stage
    // (an empty use: the compiler's wait for the word belongs here, before the next tile's DMA is on its way)
    const uint32_t kept = kept_next;
    if constexpr (DROP) asm volatile("" ::"v"(kept));
    if (jt + 1 < n_kv) {
      if constexpr (DROP) kept_next = (keep_q + (jt + 1) * attn_keep_stride(S))[keep_i];
      issue(jt + 1);
    }
    const char* Kt = smem + (jt & 1) * STG;
    const char* Vt = Kt + TILE;
#pragma unroll
    for (int kt = 0; kt < BC / 32; ++kt) {
      const int j0s = j0 + kt * 32;
      if (CAUSAL && j0s > i_w0 + 31) continue;  // whole sub-tile masked for this wave
      if (j0s >= Sk || i_w0 >= S) continue;     // whole sub-tile past the last key, or no query of this wave exists
      // The bias values are requested before the MFMAs (and the scheduler may not sink them): read at
      // first use, each one stalls the softmax arithmetic for an LDS round trip.  Prefetching the
      // MFMA operands as well, or seeding the accumulators with -lse and -dvec, costs more registers
      // than the third wave per SIMD they displace is worth (measured).
      float bias[16];
      if constexpr (WIN) {
        const float* bp = dgw + win.at(j0s - i_w0);
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const f32x4 b4 = *reinterpret_cast<const f32x4*>(bp + rq * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) bias[rq * 4 + e] = b4[e];
        }
        __builtin_amdgcn_sched_barrier(0);
      } else if constexpr (BIAS) {
        if (j0s + 32 <= Sk) {
          // every key of the sub-tile exists: one address per lane and sixteen constant offsets (with the
          // clamp below each value costs four address instructions, a third of the kernel's vector work)
          const float* bp = dg + (dg_base + j0s + (g << 2));
#pragma unroll
          for (int r = 0; r < 16; ++r) bias[r] = bp[((r >> 2) << 3) + (r & 3)];
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = j0s + ((r >> 2) << 3) + (g << 2) + (r & 3);
            bias[r] = dg[dg_base + (j < Sk ? j : Sk - 1)];  // (keys past the end are masked below)
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x16 sT, dpT;
#pragma unroll
      for (int r = 0; r < 16; ++r) { sT[r] = 0.f; dpT[r] = 0.f; }
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        sT = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DK>(Kt, kt * 32, kk, lane), qf[kk], sT, 0, 0, 0);
        dpT = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DK>(Vt, kt * 32, kk, lane), dof[kk], dpT, 0, 0, 0);
      }
      // the K / V operands of a contraction step are requested one step ahead of the products that use them
      // (left alone the compiler reads them right before, and every pair of products waits out an LDS round trip)
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int kk = 0; kk + 2 < KS; ++kk) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      // sub-tile reaches above the diagonal, past the last key, or this wave holds queries past the end
      // (all wave-uniform)
      if ((CAUSAL && j0s + 31 > i_w0) || j0s + 32 > Sk || i_w0 + 32 > S) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = j0s + ((r >> 2) << 3) + (g << 2) + (r & 3);
          float p = BIAS ? fast_exp2(fmaf(sT[r], sc, bias[r]) + nlse2) : fast_exp2(fmaf(sT[r], sc, nlse2));
          // (causal, a key past the end comes after every query)
          if (CAUSAL ? j > (q_ok ? i : -1) : j >= Sk || !q_ok) p = 0.f;
          sT[r] = p * (dp_masked(dpT[r], kept, kt * 16 + r) + ndv);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = BIAS ? fast_exp2(fmaf(sT[r], sc, bias[r]) + nlse2) : fast_exp2(fmaf(sT[r], sc, nlse2));
          sT[r] = p * (dp_masked(dpT[r], kept, kt * 16 + r) + ndv);
        }
      }
      // ---- bias gradient of this 32x32 sub-tile (wave-uniform branches)
      if constexpr (!BIAS) {
      } else if (j0s + 31 - i_w0 <= -far) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) t += sT[r];
        far_neg += t;
      } else if (!CAUSAL && j0s - i_w0 - 31 >= far) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) t += sT[r];
        far_pos += t;
      } else {
        float lo = 0.f, tot = 0.f;
        diag_accum(sT, 31 - i_lw, lo, tot);
        float* slot = ddgw + ((j0s - i_w0) / 32 + nb) * 32;
        slot[0] += lo;
        slot[32] += tot - lo;
      }
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        const bf16x8 dsf = pack8(sT, mm * 8);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          dqT[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              frag_cols_tr<DK>(Kt, kt * 32 + mm * 16, ct * 32, lane), dsf, dqT[ct], 0, 0, 0);
      }
    }
  }
  // (stored from the registers: staged through LDS like the other kernels' results it costs the third wave per SIMD
  // its registers, 576 -> 945 us at 32 x 1024 tokens, 32 heads)
  if (q_ok) {
    bf16* qrow = (bf16*)io.dq + ((size_t)b * S + i) * (size_t)io.lddq + h * DK;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)(dqT[ct][rq * 4 + e] * a.scale);
        *reinterpret_cast<bf16x4*>(qrow + ct * 32 + rq * 8 + g * 4) = o;
      }
  }
  if constexpr (!BIAS) return;
  // ---- flush: add the eight windows up (the upper lane half's diagonals sit 4 higher) and either issue one
  // global atomic per diagonal of this workgroup or, for a reproducible result, write the summed window to
  // this workgroup's row of ddiag_part (attn_ddiag_reduce_kernel adds the rows up in a fixed order)
  float* ddh = ddiag + (size_t)h * (2 * S - 1);
  float* part = nullptr;
  if (ddiag_part) part = ddiag_part + (((size_t)b * a.H + h) * ((S + BR - 1) / BR) + qt) * (size_t)attn_ddiag_part_stride(S);
  __syncthreads();
  for (int t = tid; t < W + 4; t += 256) {
    float v = 0.f;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) {
      if (t < W) v += ddg_all[(wv * 2) * W + t];
      if (t >= 4) v += ddg_all[(wv * 2 + 1) * W + t - 4];
    }
    // window entry t of wave wv: delta = t - 32 nb - 31 relative to that wave's first query, and
    // the waves' first queries are 32 apart -- but so are their windows' origins (m counts from the
    // wave's own queries), so the entry means the same diagonal for every wave
    const int idx = t - 32 * nb - 31 + (S - 1);
    if (part) part[t] = v;
    else if (v != 0.f && idx >= 0 && idx < 2 * S - 1) unsafeAtomicAdd(&ddh[idx], v);
  }
  far_neg = wave_sum(far_neg);
  far_pos = wave_sum(far_pos);
  if (part) {
    // per-wave sums, added by one lane in wave order
    float* fs = ddg_all;  // the windows have been read
    __syncthreads();
    if (lane == 0) { fs[wave * 2] = far_neg; fs[wave * 2 + 1] = far_pos; }
    __syncthreads();
    if (tid == 0) {
      part[W + 4] = (fs[0] + fs[2]) + (fs[4] + fs[6]);
      part[W + 5] = (fs[1] + fs[3]) + (fs[5] + fs[7]);
    }
  } else if (lane == 0) {
    if (far_neg != 0.f) unsafeAtomicAdd(&ddh[0], far_neg);
    if (far_pos != 0.f) unsafeAtomicAdd(&ddh[2 * S - 2], far_pos);
  }
}

// ddiag[h][..] += the window rows that the dq workgroups of head h wrote, always in the same order: a thread
// owns one window entry (or one of the two saturated-bucket sums behind the window), four threads share the
// rows (row r goes to thread group r % 4) and their sums are added in group order.  Where the window reaches an
// end diagonal, the saturated-bucket sum of that end lands on the same address: the window entry's thread adds
// both, so no two threads ever update one address.
__global__ __launch_bounds__(256) void attn_ddiag_reduce_kernel(const float* __restrict__ part,
                                                              float* __restrict__ ddiag, int B, int H, int S,
                                                              int nb) {
  __shared__ float red[2][4][64];
  const int nch = gridDim.x / H;
  const int h = blockIdx.x / nch, chunk = blockIdx.x % nch;
  const int nt = (S + 127) / 128, W = 32 * (2 * nb + 2), rows = B * nt;
  const size_t stride = (size_t)attn_ddiag_part_stride(S);
  const int tl = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int t = chunk * 64 + tl;                      // entry: [0, W+4) window, W+4 / W+5 the two sums
  const int last = 2 * S - 2;
  int idx = -1;
  if (t < W + 4) idx = t - 32 * nb - 31 + (S - 1);
  else if (t == W + 4) idx = 0;
  else if (t == W + 5) idx = last;
  const bool valid = idx >= 0 && idx <= last;
  // does a window entry own this end?  (entry t0 maps to diagonal 0, entry t1 to the last one)
  const int t0 = 32 * nb + 31 - (S - 1), t1 = t0 + last;
  const bool win0 = t0 >= 0 && t0 < W + 4, win1 = t1 >= 0 && t1 < W + 4;
  int extra = -1;                                      // second column this thread adds
  if (t < W + 4 && idx == 0) extra = W + 4;
  if (t < W + 4 && idx == last) extra = W + 5;
  const bool skip = (t == W + 4 && win0) || (t == W + 5 && win1);
  float s = 0.f, s2 = 0.f;
  if (valid && !skip) {
    // rows of head h: (b, q) -> ((b*H + h)*nt + q)
    for (int r = grp; r < rows; r += 4) {
      const size_t base = (((size_t)(r / nt) * H + h) * nt + r % nt) * stride;
      s += part[base + t];
      if (extra >= 0) s2 += part[base + extra];
    }
  }
  red[0][grp][tl] = s;
  red[1][grp][tl] = s2;
  __syncthreads();
  if (grp == 0 && valid && !skip) {
    const float tot = ((red[0][0][tl] + red[0][1][tl]) + (red[0][2][tl] + red[0][3][tl])) +
                      ((red[1][0][tl] + red[1][1][tl]) + (red[1][2][tl] + red[1][3][tl]));
    ddiag[(size_t)h * (2 * S - 1) + idx] += tot;
  }
}

// ------------------------------------------------------------------------------------------------
// dk and dv.  grid (Sk/128) * H * B; wave w owns keys j0 + 32w + lane%32; loops over query tiles.
// ------------------------------------------------------------------------------------------------
// What the two forms of the kernel share: a workgroup's operands, a ring of NST stages of query tiles, and the steps over a
// sub-tile of 32 queries x 32 keys.
template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN, int NST>
struct DkvTiles {
  static constexpr int BCK = 128, BQ = 64, KS = DK / 16, CT = DK / 32;
  static constexpr int TILE = BQ * DK * 2, STG = 2 * TILE;  // a stage holds a Q tile then a dO tile
  const AttnIO& io;
  const AttnDims& a;
  char* smem;
  // The score and dP accumulators start from -lse/scale and -dvec, so that the MFMA results are
  // already (s - lse/scale) and (dP - dvec): no per-element subtraction afterwards.
  float* lse_all;      // [stages][BQ]  -lse / scale
  float* dv_all;       // [stages][BQ]  -dvec
  uint32_t* keep_all;  // [stages][2 key tiles][2][BQ] keep decisions (DROP only)
  // Window, or [-BQ, S + BCK - 1), log2 units (BIAS only); the slice's BQ entries in front are only ever read for
  // queries past the end of a ragged last tile, whose probabilities are set to zero
  float* dg;
  const float* dgw;  // (WIN) the four diagonals of queries 8 rq + 4 g + 0..3 of a sub-tile, the last query's first
  BiasWin win;
  int tid, lane, g, wave, S, Sk, h, b;
  int j0, j_w0, j_loc;  // first key of the workgroup and of this wave, this lane's key in the workgroup
  int it_begin, it_tail, n_it;
  float sc;
  const bf16 *base, *dobase;
  size_t ld, ldo;
  TileDma<DK, BQ> tq, tdo, tq_tail, tdo_tail;  // _tail: the last tile of a query sequence that does not fill it
  uint32_t lds0, lds_lse, lds_dv, lds_keep;
  const float *ndvec, *nlse;
  const uint32_t* keep_w;
  int keep_n;  // this lane's key in a word
  bf16x8 kf[KS], vf[KS];
  f32x16 dkT[CT], dvT[CT];

  __device__ __forceinline__ DkvTiles(char* lds, const AttnIO& io_, const bf16* dout, const float* dvec, const AttnDims& a_)
      : io(io_), a(a_), smem(lds), win(a_.S, a_.far, CAUSAL) {
    lse_all = reinterpret_cast<float*>(smem + NST * STG);
    dv_all = lse_all + NST * BQ;
    keep_all = reinterpret_cast<uint32_t*>(dv_all + NST * BQ);
    dg = dv_all + NST * BQ + (DROP ? NST * 4 * BQ : 0) + (WIN ? 0 : BQ);
    tid = threadIdx.x; lane = tid & 63; g = lane >> 5;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    S = a.S; Sk = a.Sk;
    ld = (size_t)io.ldq; ldo = (size_t)(a.H * DK);
    int kt;
    decode_block((Sk + BCK - 1) / BCK, a.H, a.B, kt, h, b);
    j0 = kt * BCK;
    j_w0 = j0 + wave * 32;
    j_loc = wave * 32 + (lane & 31);
    base = (const bf16*)io.q + (size_t)b * S * ld + h * DK;
    dobase = dout + (size_t)b * S * ldo + h * DK;
    it_begin = CAUSAL ? (j0 / BQ) : 0;
    it_tail = S % BQ ? S / BQ : -1;
    n_it = (S + BQ - 1) / BQ;
    tq.init(wave, lane, ld);
    tdo.init(wave, lane, ldo);
    tq_tail.init(wave, lane, ld, S % BQ ? S % BQ : BQ);
    tdo_tail.init(wave, lane, ldo, S % BQ ? S % BQ : BQ);
    lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    // The -lse / scale and -dvec slices of a query tile (written by the dq kernel) travel by DMA as well, one
    // instruction each from waves 0 and 1.  Fetched with ordinary loads they put compiler-made vmcnt waits into
    // the loop, and since those count the tile DMA issued just before them, every iteration waited out the
    // whole DMA latency at its first matrix instruction.
    const size_t srow = ((size_t)b * a.H + h) * S;
    ndvec = dvec + srow;
    nlse = dvec + (size_t)a.B * a.H * S + srow;
    lds_lse = lds0 + NST * STG;
    lds_dv = lds_lse + NST * BQ * 4;
    // wave w fetches half w & 1 of key tile w >> 1 (past the last key: of the last tile, for keys that are not stored)
    lds_keep = lds_dv + NST * BQ * 4;
    const int keep_jt = min(j0 / 64 + (wave >> 1), (Sk + 63) / 64 - 1);
    keep_w = DROP ? keep_row(a, (size_t)b * a.H + h, keep_jt, wave & 1) : nullptr;
    keep_n = (wave & 1) * 16 + ((lane >> 3) & 3) * 4 + (lane & 3);
  }

  // what only the loop needs
  __device__ __forceinline__ void begin() {
    sc = a.scale * kLog2e;
    dgw = win.lane(dg, 28 + (lane & 31) - (g << 2));
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) { dkT[ct][r] = 0.f; dvT[ct][r] = 0.f; }
  }
  __device__ __forceinline__ void issue(int stage, int it) const {
    const int q_first = it * BQ;
    const uint32_t dst = lds0 + stage * STG;
    (it == it_tail ? tq_tail : tq).issue(dst, base + (size_t)q_first * ld, wave);
    (it == it_tail ? tdo_tail : tdo).issue(dst + TILE, dobase + (size_t)q_first * ldo, wave);
    const int qi = q_first + lane < S ? q_first + lane : S - 1;  // (rows past the end are masked)
    if (wave == 0) dma_64f(lds_lse + stage * BQ * 4, nlse, (uint32_t)qi * 4u);
    if (wave == 1) dma_64f(lds_dv + stage * BQ * 4, ndvec, (uint32_t)qi * 4u);
    if constexpr (DROP) dma_64f(lds_keep + (stage * 4 + wave) * BQ * 4, keep_w + q_first, (uint32_t)lane * 4u);
  }
  __device__ __forceinline__ void load_keys() {
    const int j = j0 + j_loc, j_ld = j < Sk ? j : Sk - 1;
    const bf16* krow = (const bf16*)io.k + ((size_t)b * Sk + j_ld) * (size_t)io.ldkv + h * DK;
    const bf16* vrow = (const bf16*)io.v + ((size_t)b * Sk + j_ld) * (size_t)io.ldkv + h * DK;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      kf[kk] = *reinterpret_cast<const bf16x8*>(krow + kk * 16 + g * 8);
      vf[kk] = *reinterpret_cast<const bf16x8*>(vrow + kk * 16 + g * 8);
    }
  }
  // The compiler waits for these loads where they are first used, and that is inside the loop: its
  // s_waitcnt vmcnt(n) there would run in every iteration and, since the counter also counts the tile DMA
  // issued at the top of the iteration, stall the first matrix instructions until the whole DMA has landed.
  // An empty use moves the wait in front of the loop.
  __device__ __forceinline__ void wait_keys() const {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" ::"v"(kf[kk]), "v"(vf[kk]));
  }
  __device__ __forceinline__ void fill_bias(const float* __restrict__ diag) const {
    if constexpr (WIN) {
      win.template fill<CAUSAL>(dg, diag + (size_t)h * (2 * S - 1), S, tid);
    } else if constexpr (BIAS) {
      // dg[t] = bias(delta) for delta = t + j0 - (S - 1), t in [0, S + BCK - 1)
      const float* dgh = diag + (size_t)h * (2 * S - 1);
      for (int t = tid; t < S + BCK - 1; t += 256) {
        int idx = t + j0;  // delta + S - 1
        idx = idx > 2 * S - 2 ? 2 * S - 2 : idx;
        dg[t] = dgh[idx] * kLog2e;
      }
      if (tid < BQ) dg[tid - BQ] = 0.f;
    }
  }
  // the score accumulators of queries past the end start from the infinity that makes exp2 zero
  __device__ __forceinline__ void seed_tail(int stage, int it) const {
    if (it == it_tail) {
      if (tid < BQ && it * BQ + tid >= S) lse_all[stage * BQ + tid] = sc > 0.f ? -INFINITY : INFINITY;
      __syncthreads();
    }
  }
  // s = S - lse / scale, dp = dP - dvec of sub-tile qb of the tile in `stage`
  __device__ __forceinline__ void scores(int stage, int qb, f32x16& s, f32x16& dp) const {
    const char* Qt = smem + stage * STG;
    const char* Dt = Qt + TILE;
    const float* lse_s = lse_all + stage * BQ;
    const float* dv_s = dv_all + stage * BQ;
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_s + qb * 32 + rq * 8 + g * 4);
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(dv_s + qb * 32 + rq * 8 + g * 4);
#pragma unroll
      // with dropout dP is rescaled before dvec is subtracted: it starts from zero
      for (int e = 0; e < 4; ++e) { s[rq * 4 + e] = l4[e]; dp[rq * 4 + e] = DROP ? 0.f : d4[e]; }
    }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DK>(Qt, qb * 32, kk, lane), kf[kk], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<DK>(Dt, qb * 32, kk, lane), vf[kk], dp, 0, 0, 0);
    }
  }
  // The scores of keys after their query: the infinity that makes exp2 zero, or with the window, whose bias is -infinity
  // there, zero.  q0: first query of the sub-tile.
  __device__ __forceinline__ void mask_later(int q0, f32x16& s) const {
    const float gone = WIN ? 0.f : sc > 0.f ? -INFINITY : INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (((r >> 2) << 3) + (r & 3) < j0 + j_loc - q0 - (g << 2)) s[r] = gone;
  }
  __device__ __forceinline__ void load_bias(int q0, float (&bias)[16]) const {
    if constexpr (WIN) {
      const float* bp = dgw + win.at(j_w0 - q0);
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const f32x4 b4 = *reinterpret_cast<const f32x4*>(bp - rq * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[rq * 4 + e] = b4[3 - e];
      }
    } else if constexpr (BIAS) {
      // dg index of (query i, key j): (j - i) - (j0 - (S-1)) = j_loc + (S - 1 - i).  Register r belongs to query
      // q0 + 4g + c_r with c_r = 8*(r/4) + r%4 <= 27, so bq[27 - c_r] with bq 27 below the first.  (a query past the
      // end of a ragged tile reads at most BQ - 1 entries below dg[0]: the padding)
      const float* bq = dg + (j_loc + S - 1 - q0 - (g << 2) - 27);
#pragma unroll
      for (int r = 0; r < 16; ++r) bias[r] = bq[27 - (((r >> 2) << 3) + (r & 3))];
    }
  }
  // P of element r of a sub-tile, and with its dropout decision the elements of P and dS that enter the products
  __device__ __forceinline__ float prob(float s, float bias) const {
    return BIAS ? fast_exp2(fmaf(s, sc, bias)) : fast_exp2(s * sc);
  }
  __device__ __forceinline__ void drop_elem(int stage, int qb, int r, float p, float dp, float& pd, float& ds) const {
    if constexpr (DROP) {
      const float* dv_s = dv_all + stage * BQ;
      const uint32_t* keep_s = keep_all + (stage * 4 + (wave & 2) + ((lane >> 2) & 1)) * BQ;
      const int il = qb * 32 + ((r >> 2) << 3) + (g << 2) + (r & 3);
      const int mask = keep_mask(keep_s[il], keep_n);
      pd = keep_if(mask, p);
      ds = p * (keep_if(mask, dp * a.drop.scale) + dv_s[il]);
    } else {
      pd = p;
      ds = p * dp;
    }
  }
  // the dV and dK products of queries 16 mm .. 16 mm + 15 of a sub-tile
  __device__ __forceinline__ void outer(int stage, int qb, int mm, const bf16x8& pf, const bf16x8& dsf) {
    const char* Qt = smem + stage * STG;
    const char* Dt = Qt + TILE;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      dvT[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_tr<DK>(Dt, qb * 32 + mm * 16, ct * 32, lane), pf, dvT[ct], 0, 0, 0);
      dkT[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_tr<DK>(Qt, qb * 32 + mm * 16, ct * 32, lane), dsf, dkT[ct], 0, 0, 0);
    }
  }
  __device__ __forceinline__ void store() const {
    __syncthreads();  // every wave is done with the tiles
    char* stage = smem + wave * 32 * (DK * 2 + 16);
    const size_t row0 = (size_t)b * Sk + j_w0, ldd = (size_t)io.lddkv;
    store_rows<DK>(stage, dkT, a.scale, (bf16*)io.dk + row0 * ldd + h * DK, ldd, Sk - j_w0, lane);
    store_rows<DK>(stage, dvT, DROP ? a.drop.scale : 1.f, (bf16*)io.dv + row0 * ldd + h * DK, ldd, Sk - j_w0, lane);
  }
};

// The first form takes a tile at a time from two stages: 64 channels without the causal mask, where two or three waves per
// SIMD cover for each other, or with dropout (causal 32 x 512, 12 heads: 68 us, the other form 72), or with a slice beside
// which three stages would be too much (dkv_takes_pipe).
template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool THREE, bool WIN>
__global__ __launch_bounds__(256, THREE ? 3 : 2)
void attn_bwd_dkv_mfma_kernel(AttnIO io, const bf16* __restrict__ dout, const float* __restrict__ diag,
                              const float* __restrict__ dvec, AttnDims a) {
  static_assert(DK == 64, "128 channels have the pipelined form");
  using Tiles = DkvTiles<DK, CAUSAL, BIAS, DROP, WIN, 2>;
  constexpr int BCK = Tiles::BCK, BQ = Tiles::BQ;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  Tiles t(smem, io, dout, dvec, a);
  t.load_keys();
  t.wait_keys();
  t.fill_bias(diag);
  t.begin();

  // How the queries past the end of a ragged last tile come to probability zero: by a masked copy of the element loop, or
  // from the score accumulators' seeds.  Without the copy (and its branch) an iteration is one block that the compiler
  // schedules whole; with dropout, with the slice, and bias-free with two waves, the copy is faster (slice: 32 x 256 tokens,
  // 12 heads 25.1 -> 23.9 us, 4 x 2048 124 -> 119, 4 x 333 13.2 -> 12.4; window: 128 x 512, 12 heads 267 with the copy, 266
  // without, 32 x 1024, 32 heads 594 and 587).
  constexpr bool TAIL_MASK = !CAUSAL && (BIAS ? DROP || !WIN : !DROP && !THREE);
  // P and dS of a sub-tile, in place of s and dp
  auto softmax = [&](auto tail, int stage, int qb, int q0, f32x16& s, f32x16& dp, const float (&bias)[16])
      __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float p = t.prob(s[r], bias[r]), pd, ds;
      if (decltype(tail)::value && q0 + ((r >> 2) << 3) + (t.g << 2) + (r & 3) >= t.S) p = 0.f;
      t.drop_elem(stage, qb, r, p, dp[r], pd, ds);
      s[r] = pd;
      dp[r] = ds;
    }
  };
  t.issue(0, t.it_begin);
  // diag: the tiles that the diagonal cuts have a loop of their own, so that the other loop has no branch (one loop with a branch
  // around the mask: causal 64 x 512, 6 heads 70 -> 71 us, 1 x 1024, 12 heads 27 -> 29)
  int it = t.it_begin;
#pragma unroll
  for (int diag = CAUSAL ? 1 : 0; diag >= 0; --diag) {
    for (const int end = diag ? min(t.it_begin + BCK / BQ, t.n_it) : t.n_it; it < end; ++it) {
      const int st = (it - t.it_begin) & 1, q0 = it * BQ;
      dma_wait_barrier();  // tile `it` and its lse / dvec slices landed; the other stage is free
      if constexpr (!TAIL_MASK) t.seed_tail(st, it);
      if (it + 1 < t.n_it) t.issue(st ^ 1, it + 1);
      // with the window, the score products of both sub-tiles first: 32 x 1024 tokens, 32 heads 609 -> 590 us
      constexpr bool BOTH = WIN && !DROP && !CAUSAL;
      f32x16 s[2], dp[2];
      float bias[2][16];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        if (diag && q0 + qb * 32 < t.j_w0) continue;  // masked whole for this wave
        if (qb == 0 || !BOTH) {
          t.load_bias(q0 + qb * 32, bias[qb]);
          t.scores(st, qb, s[qb], dp[qb]);
          if (diag) t.mask_later(q0 + qb * 32, s[qb]);
        }
        if (qb == 0 && BOTH) {
          t.load_bias(q0 + 32, bias[1]);
          t.scores(st, 1, s[1], dp[1]);
        }
        if (TAIL_MASK && q0 + qb * 32 + 32 > t.S) softmax(std::true_type{}, st, qb, q0 + qb * 32, s[qb], dp[qb], bias[qb]);
        else softmax(std::false_type{}, st, qb, q0 + qb * 32, s[qb], dp[qb], bias[qb]);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) t.outer(st, qb, mm, pack8(s[qb], mm * 8), pack8(dp[qb], mm * 8));
      }
    }
  }
  t.store();
}

// The pipelined form (128 channels, and 64 causal without dropout).  A unit is 32 queries x 32 keys; its dV / dK products follow the
// score products of the next unit and run beside that unit's softmax arithmetic, across the tiles' barriers too (a ring of
// three tile stages).  With 128 channels one wave has a SIMD to itself, and in program order matrix and vector unit took
// turns (28 % and 26 % busy): 16 x 2048 tokens causal, 16 heads 950 -> 843 us, 8 x 2048 not causal 740 -> 650; 64 channels
// causal, 8 x 2048, 12 heads 167 -> 148, 32 x 512 67 -> 62; with dropout, not causal, 8 x 2048, 16 heads of 128 827 -> 627.
// 64 channels without the mask: 1-4 % slower than the other form.
template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN>
__global__ __launch_bounds__(256, DK == 64 ? 2 : 1)
void attn_bwd_dkv_pipe_kernel(AttnIO io, const bf16* __restrict__ dout, const float* __restrict__ diag,
                              const float* __restrict__ dvec, AttnDims a) {
  using Tiles = DkvTiles<DK, CAUSAL, BIAS, DROP, WIN, 3>;
  constexpr int BQ = Tiles::BQ;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  Tiles t(smem, io, dout, dvec, a);
  t.issue(0, t.it_begin);
  t.load_keys();
  t.fill_bias(diag);
  t.wait_keys();
  t.begin();

  // Step n of the pipeline: the score products of unit n, then the dV / dK products of unit n - 1 beside the softmax
  // arithmetic of unit n.
  bf16x8 pf[2], dsf[2];  // P and dS of the unit whose products are still to come
  // unit qb of the tile in `stage`, whose first query is q0, behind unit pqb of `pst` (-1: none)
  auto step = [&](auto diag, int pst, int pqb, int stage, int qb, int q0) __attribute__((always_inline)) {
    f32x16 s, dp;
    float bias[16];
    bf16x8 pn[2], dn[2];
    t.load_bias(q0 + qb * 32, bias);
    t.scores(stage, qb, s, dp);
    if constexpr (decltype(diag)::value) t.mask_later(q0 + qb * 32, s);
    if (pqb >= 0) {
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) t.outer(pst, pqb, mm, pf[mm], dsf[mm]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pd, ds;
      t.drop_elem(stage, qb, r, t.prob(s[r], bias[r]), dp[r], pd, ds);
      pn[r >> 3][r & 7] = (bf16)pd;
      dn[r >> 3][r & 7] = (bf16)ds;
    }
#pragma unroll
    for (int mm = 0; mm < 2; ++mm) { pf[mm] = pn[mm]; dsf[mm] = dn[mm]; }
  };
  // tile `it` has landed in `stage`; every wave is done with tile it - 2
  auto enter = [&](int stage, int it) __attribute__((always_inline)) {
    dma_wait_barrier();
    t.seed_tail(stage, it);
    if (it + 1 < t.n_it) t.issue(stage == 2 ? 0 : stage + 1, it + 1);
  };
  // Causal, the diagonal cuts the w-th unit of wave w, which begins there (the units before it have no visible key): waves 2 and
  // 3 in the second tile, 1 and 3 with a tile's second unit.  The loop has no mask and no branch inside a step (with a select
  // in every unit, slice of diagonals: 2 x 8192 tokens, 8 heads of 128 channels 851 us, 600 like this; with a branch around
  // it, 16 x 2048, 16 heads 740 -> 825, like this 755).
  constexpr std::bool_constant<CAUSAL> cut{};
  constexpr std::false_type all{};
  int it = t.it_begin, st = 0, second = 0;
  enter(0, it);
  if constexpr (CAUSAL) {
    if (t.wave >= 2 && it + 1 < t.n_it) {
      enter(1, ++it);
      st = 1;
    }
    second = t.wave & 1;
    asm("" : "+s"(second));  // (known, it would become a copy of the loop)
  }
  step(cut, 0, -1, st, second, it * BQ);
  for (;; ++it) {
    const int q0 = it * BQ;
    if (!CAUSAL || !second) step(all, st, 0, st, 1, q0);
    second = 0;
    if (it + 1 == t.n_it) break;
    const int nst = st == 2 ? 0 : st + 1;
    enter(nst, it + 1);
    step(all, st, 1, nst, 0, q0 + BQ);
    st = nst;
  }
#pragma unroll
  for (int mm = 0; mm < 2; ++mm) t.outer(st, 1, mm, pf[mm], dsf[mm]);
  t.store();
}

// Whether dk/dv has a pipelined form.
constexpr bool dkv_pipe(int dk, bool causal, bool drop) { return dk == 128 || (causal && !drop); }
size_t dkv_lds_bytes(const AttnDims& a, bool window, int stages) {
  size_t floats = stages * ((size_t)64 * a.dk + 128 + (a.drop.on ? 256 : 0));  // Q and dO tiles, -lse, -dvec, keep words
  if (a.bias) floats += window ? BiasWin(a.S, a.far, a.causal != 0).floats() : 64 + a.S + 127;
  return floats * sizeof(float);
}
// It is taken where its third stage does not keep the second workgroup of 64 channels off the compute unit, as it does beside
// the slice of more than 7617 positions (causal, 12 heads, 4 x 7680: 1100 us, the other form 797; 4 x 7168: 685 and 696).
bool dkv_takes_pipe(const AttnDims& a, bool window) {
  return dkv_pipe(a.dk, a.causal != 0, a.drop.on != 0) && (a.dk == 128 || 2 * dkv_lds_bytes(a, window, 3) <= (size_t)160 * 1024);
}

template <typename K>
hipError_t set_lds(K kern, size_t bytes) {
  return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN>
hipError_t fwd_launch_as(const AttnIO& io, const float* diag, void* c, float* lse, const AttnDims& a, hipStream_t st) {
  auto kern = attn_fwd_mfma_kernel<DK, CAUSAL, BIAS, DROP, WIN>;
  const size_t lds = attn_lds_bytes(a, ATTN_FWD, WIN);
  hipError_t e = set_lds(kern, lds);
  if (e != hipSuccess) return e;
  kern<<<dim3(((a.S + 127) / 128) * a.H * a.B), 256, lds, st>>>(io, diag, (bf16*)c, lse, a);
  return hipGetLastError();
}

template <int DK, bool CAUSAL, bool BIAS, bool DROP = false>
hipError_t fwd_launch(const AttnIO& io, const float* diag, void* c, float* lse, const AttnDims& a, hipStream_t st) {
  if (BIAS && attn_bias_window(a, ATTN_FWD)) return fwd_launch_as<DK, CAUSAL, BIAS, DROP, BIAS>(io, diag, c, lse, a, st);
  return fwd_launch_as<DK, CAUSAL, BIAS, DROP, false>(io, diag, c, lse, a, st);
}

template <int DK, bool CAUSAL, bool BIAS, bool DROP, bool WIN>
hipError_t bwd_launch_as(const AttnIO& io, const void* c, const void* dc, const float* diag, const float* lse,
                      float* dvec, float* ddiag, float* ddiag_part, const AttnDims& a, int phase,
                      hipStream_t st) {
  hipError_t e = hipSuccess;
  if (phase == 1) {
    auto kern = attn_bwd_dq_mfma_kernel<DK, CAUSAL, BIAS, DROP, WIN>;
    const size_t lds = attn_lds_bytes(a, ATTN_BWD_DQ, WIN);
    if ((e = set_lds(kern, lds)) != hipSuccess) return e;
    kern<<<dim3(((a.S + 127) / 128) * a.H * a.B), 256, lds, st>>>(io, (const bf16*)c, (const bf16*)dc, diag, lse, dvec, ddiag,
                                                          BIAS ? ddiag_part : nullptr, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (BIAS && ddiag_part) {
      const int nb = attn_dq_window_blocks(a.S, a.far);
      attn_ddiag_reduce_kernel<<<a.H * ceil_div(32 * (2 * nb + 2) + 6, 64), 256, 0, st>>>(ddiag_part, ddiag, a.B, a.H,
                                                                                         a.S, nb);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  if (phase == 2) {
    const size_t lds = attn_lds_bytes(a, ATTN_BWD_DKV, WIN);
    const int wgs = ((a.Sk + 127) / 128) * a.H * a.B;
    if constexpr (dkv_pipe(DK, CAUSAL, DROP)) {
      if (DK == 128 || WIN || dkv_takes_pipe(a, WIN)) {
        auto kern = attn_bwd_dkv_pipe_kernel<DK, CAUSAL, BIAS, DROP, WIN>;
        if ((e = set_lds(kern, lds)) != hipSuccess) return e;
        kern<<<dim3(wgs), 256, lds, st>>>(io, (const bf16*)dc, diag, dvec, a);
        return hipGetLastError();
      }
    }
    if constexpr (DK == 64 && !(dkv_pipe(DK, CAUSAL, DROP) && WIN)) {
      // Bias-free with 64 channels: beyond two workgroups per compute unit the form that lets a third in, up to there the
      // one whose single workgroup is faster (1 x 1024 queries over 100 keys, 12 heads, 12 workgroups: 27 against 23 us;
      // 384 workgroups 39 and 38; 768 61 and 65; 128 x 114 over 512, 6144 workgroups: 103 and 106).
      constexpr bool CAN_THREE = !BIAS && !DROP;
      auto kern = CAN_THREE && wgs > 512 ? attn_bwd_dkv_mfma_kernel<DK, CAUSAL, BIAS, DROP, CAN_THREE, WIN>
                                         : attn_bwd_dkv_mfma_kernel<DK, CAUSAL, BIAS, DROP, false, WIN>;
      if ((e = set_lds(kern, lds)) != hipSuccess) return e;
      kern<<<dim3(wgs), 256, lds, st>>>(io, (const bf16*)dc, diag, dvec, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <int DK, bool CAUSAL, bool BIAS, bool DROP = false>
hipError_t bwd_launch(const AttnIO& io, const void* c, const void* dc, const float* diag, const float* lse,
                      float* dvec, float* ddiag, float* ddiag_part, const AttnDims& a, int phase, hipStream_t st) {
  if (BIAS && attn_bias_window(a, phase == 1 ? ATTN_BWD_DQ : ATTN_BWD_DKV))
    return bwd_launch_as<DK, CAUSAL, BIAS, DROP, BIAS>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
  return bwd_launch_as<DK, CAUSAL, BIAS, DROP, false>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
}

// 0: self-attention with bias, 1: the same with the causal mask, 2: cross-attention (no bias, no mask)
int attn_mode(const AttnDims& a) { return a.bias ? (a.causal ? 1 : 0) : 2; }

}  // namespace

size_t attn_lds_bytes(const AttnDims& a, AttnPass pass, bool window) {
  if (pass == ATTN_BWD_DKV) return dkv_lds_bytes(a, window, dkv_takes_pipe(a, window) ? 3 : 2);
  size_t floats = 2 * (size_t)64 * a.dk;  // two stages of a K and a V tile
  if (!a.bias) return floats * sizeof(float);
  floats += window ? BiasWin(a.S, a.far, a.causal != 0).floats() : a.S + 127;
  // the dq kernel keeps per-diagonal windows of about 2 * far entries for each half wavefront
  if (pass == ATTN_BWD_DQ) floats += 8 * 32 * (2 * (size_t)attn_dq_window_blocks(a.S, a.far) + 2);
  return floats * sizeof(float);
}

int attn_workgroups_per_unit(const AttnDims& a, AttnPass pass, bool window) {
  // (of four wavefronts: one on each SIMD.  What the registers allow: launch bounds, forward as built)
  int by_registers = 2;
  if (pass == ATTN_FWD && a.dk == 64) by_registers = a.causal && window ? 4 : 3;
  if (pass == ATTN_BWD_DQ && a.dk == 64) by_registers = !a.drop.on || (a.causal && window) ? 3 : 2;
  if (pass == ATTN_BWD_DKV && a.dk == 128) by_registers = 1;
  return std::min(by_registers, (int)((size_t)160 * 1024 / attn_lds_bytes(a, pass, window)));
}

// The window is used while its copies stay under 10 KB (two thirds of a K tile with 128 channels: distances up to 225,
// causal 449, or as many positions) and do not keep a workgroup off the compute unit.  The latter is a matter of dq, which has
// windows of diagonal sums beside it: not causal, 64 x 512 tokens, 16 heads of 128 channels, distance 130 (two workgroups
// with the slice, one with the window) 469 us with the window, 328 with the slice; 32 x 256, 12 heads of 64, distance 166
// (three and two) 34 and 28; causal, distance 216, 31 and 26.
bool attn_bias_window(const AttnDims& a, AttnPass pass) {
  return a.bias && BiasWin(a.S, a.far, a.causal != 0).floats() * sizeof(float) <= 10240 &&
         attn_workgroups_per_unit(a, pass, true) >= attn_workgroups_per_unit(a, pass, false);
}

bool attn_bwd_mfma_fits(const AttnDims& a) { return attn_lds_bytes(a, ATTN_BWD_DQ, false) <= (size_t)150 * 1024; }

bool attn_mfma_supported(const AttnDims& a) {
  // Any lengths from 32 up (tiles are rounded up and their tails masked); LDS holds the diagonal slice
  // (S + 127 floats).  Without the bias only the unmasked form exists; bias and mask need square scores.
  if (!(a.dk == 64 || a.dk == 128) || a.S < 32 || a.Sk < 32 || a.S > 8192 || a.Sk > 65536) return false;
  if (a.bias) return a.Sk == a.S;
  return !a.causal;
}

hipError_t launch_attn_fwd_mfma(const AttnIO& io, const float* diag, void* c, float* lse, const AttnDims& a,
                                hipStream_t st) {
  if (!attn_mfma_supported(a) || (a.drop.on && !a.keep)) return hipErrorInvalidValue;
  const int mode = attn_mode(a);
  if (a.drop.on) {
    if (a.dk == 64) {
      if (mode == 0) return fwd_launch<64, false, true, true>(io, diag, c, lse, a, st);
      if (mode == 1) return fwd_launch<64, true, true, true>(io, diag, c, lse, a, st);
      return fwd_launch<64, false, false, true>(io, diag, c, lse, a, st);
    }
    if (mode == 0) return fwd_launch<128, false, true, true>(io, diag, c, lse, a, st);
    if (mode == 1) return fwd_launch<128, true, true, true>(io, diag, c, lse, a, st);
    return fwd_launch<128, false, false, true>(io, diag, c, lse, a, st);
  }
  if (a.dk == 64) {
    if (mode == 0) return fwd_launch<64, false, true>(io, diag, c, lse, a, st);
    if (mode == 1) return fwd_launch<64, true, true>(io, diag, c, lse, a, st);
    return fwd_launch<64, false, false>(io, diag, c, lse, a, st);
  }
  if (mode == 0) return fwd_launch<128, false, true>(io, diag, c, lse, a, st);
  if (mode == 1) return fwd_launch<128, true, true>(io, diag, c, lse, a, st);
  return fwd_launch<128, false, false>(io, diag, c, lse, a, st);
}

size_t attn_keep_bytes(const AttnDims& a) {
  return a.drop.on ? (size_t)a.B * a.H * ((a.Sk + 63) / 64) * attn_keep_stride(a.S) * sizeof(uint32_t) : 0;
}

size_t attn_ddiag_part_bytes(const AttnDims& a) {
  return (size_t)a.B * a.H * ((a.S + 127) / 128) * (size_t)attn_ddiag_part_stride(a.S) * sizeof(float);
}

hipError_t launch_attn_bwd_mfma(const AttnIO& io, const void* c, const void* dc, const float* diag,
                                const float* lse, float* dvec, float* ddiag, const AttnDims& a, int phase,
                                hipStream_t st, float* ddiag_part) {
  // phase 1: dq, dvec = rowsum(dO * O) and the bias-gradient diagonals (added into ddiag); phase 2: dk, dv
  // (reads the dvec phase 1 wrote).
  // a.far: smallest distance that falls in the last (saturated) bucket; such offsets need no
  // per-diagonal resolution.  Never below 1, so offset 0 always takes the per-diagonal path.
  if (!attn_mfma_supported(a) || (a.drop.on && !a.keep)) return hipErrorInvalidValue;
  const int mode = attn_mode(a);
  if (a.drop.on) {
    if (a.dk == 64) {
      if (mode == 0) return bwd_launch<64, false, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
      if (mode == 1) return bwd_launch<64, true, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
      return bwd_launch<64, false, false, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
    }
    if (mode == 0) return bwd_launch<128, false, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
    if (mode == 1) return bwd_launch<128, true, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
    return bwd_launch<128, false, false, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
  }
  if (a.dk == 64) {
    if (mode == 0) return bwd_launch<64, false, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
    if (mode == 1) return bwd_launch<64, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
    return bwd_launch<64, false, false>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
  }
  if (mode == 0) return bwd_launch<128, false, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
  if (mode == 1) return bwd_launch<128, true, true>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
  return bwd_launch<128, false, false>(io, c, dc, diag, lse, dvec, ddiag, ddiag_part, a, phase, st);
}

}  // namespace t5mi
