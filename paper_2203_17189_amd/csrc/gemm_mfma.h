// Kernel and launch templates of the bf16 MFMA GEMM; gemm_mfma_*.hip instantiate them, one epilogue family each.
//
// bf16 MFMA GEMM for gfx950 (v_mfma_f32_32x32x16_bf16, float32 accumulation) with fused epilogues.
//
//   C[m,n] = sum_s sum_k A_s(m,k) B_s(n,k)
//
// Tiling: workgroup tile BM x BN, k-tiles of BK, WM x WN wavefronts, each wave owns
// (BM/WM) x (BN/WN) as 32x32 MFMA tiles; which tile a problem gets is decided in launch_layout.
//
// Data path: global -> LDS directly (global_load_lds_dwordx4: every lane fetches 16 bytes, a wave
// fills 1 KB of contiguous LDS), NS stages deep.  Global load latency on this part is on the order
// of a microsecond under load while one k-tile is ~0.4 us of MFMA work, so several k-tiles must be
// in flight; keeping them in LDS instead of registers leaves the register file to the accumulators.
// Because the DMA writes LDS linearly, the bank-conflict swizzle is applied on the global side: the
// lane that owns LDS slot (row, physical chunk) fetches the logical chunk that belongs there.
// Two operand layouts:
//   k-contiguous (A[m][k]):  LDS rows of BK k (64 or 128 B: 4 or 8 chunks), read with ds_read_b128;
//   (the weights of gemm_mfma_direct.hip: A k-contiguous, B n-contiguous, its columns from up to three matrices)
//   m-contiguous (A[k][m]):  LDS rows of BM m, 32-byte granules swizzled by k, read with the LDS
//                            transpose load ds_read_b64_tr_b16 (two per MFMA operand).
// The compiler does not see these DMA writes; ordering is explicit: s_waitcnt vmcnt(n) + s_barrier
// before a stage is read, and a stage is refilled only after a barrier that every wave reaches
// after its last read of that stage.
// Workgroup ids are remapped so that each XCD (ids are dealt round-robin to the 8 XCDs) works on a
// compact block of output tiles and shares operand tiles through its own L2.
#pragma once
#include "kernels.h"
#include <algorithm>
#include <atomic>

#include <type_traits>

namespace t5mi {

// Ends of a split reduction (gemm_mfma.hip): clears the outputs, or adds the slices in GemmEpi::aux0 up in order.
hipError_t launch_zero_split(const GemmEpi& e, int M, int N, hipStream_t st);
hipError_t launch_splitk_reduce(const GemmEpi& e, int M, int N, int slices, hipStream_t st);

namespace {

constexpr int KQ = 64;   // every segment's K must be a multiple of this (m-contiguous operands: any K)

typedef __attribute__((address_space(3))) short4v lds_short4;

// k-contiguous stage: row r (BK*2 bytes) holds logical 16-byte chunk c at physical chunk c ^ kc_swz(r).
template <int BK>
__device__ __forceinline__ int kc_swz(int row) {
  if constexpr (BK == 32) return ((row >> 1) & 3) ^ ((row >> 3) & 1);
  else return (row ^ (row >> 3)) & 7;
}

// m-contiguous stage of ROWS m: 32-byte granule g of row k lies at granule g ^ mc_swz(k).
template <int ROWS>
__device__ __forceinline__ int mc_swz(int krow) {
  return ((krow & 3) << 1) & (ROWS / 16 - 1);
}

// One MFMA operand (8 bf16 of k for row base + lane%32) for k-step kk of a stage.
template <int ROWS, bool KC, int BK>
__device__ __forceinline__ bf16x8 load_frag(const char* stage, int base, int kk, int lane) {
  if constexpr (KC) {
    const int row = base + (lane & 31);
    const int chunk = kk * 2 + (lane >> 5);
    return *reinterpret_cast<const bf16x8*>(stage + row * (BK * 2) + ((chunk ^ kc_swz<BK>(row)) << 4));
  } else {
    // 16-lane groups: lanes supply the address of 4 consecutive m at row k; the transpose load hands
    // lane i the 4 k-values of m = group_base + i.
    const int i16 = lane & 15;
    const int m_e = base + (((lane >> 4) & 1) << 4) + ((i16 & 3) << 2);
    const int krow = kk * 16 + ((lane >> 5) << 3) + (i16 >> 2);
    const int g = m_e >> 4;
    const int off0 = krow * (ROWS * 2) + ((g ^ mc_swz<ROWS>(krow)) << 5) + ((m_e & 15) << 1);
    const int off1 = off0 + 4 * (ROWS * 2);  // krow + 4 keeps (krow & 3)
    short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(stage + off0));
    short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(stage + off1));
    typedef __attribute__((ext_vector_type(8))) short short8v;
    short8v r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, r);
  }
}

// Position in a workgroup's sequence of k-tiles, in scalar registers: global base addresses of the next
// tile and the number of tiles left in the current run.  A k-slice is at most three runs of consecutive
// tiles (one per segment).  A wave issues one instruction every four cycles and a matrix instruction
// occupies its pipe for 32: seven other instructions fit between two of them for free, and every one
// beyond that is a bubble in the matrix pipe.  The cursor therefore advances without branches, in a few
// scalar and/or/add steps (a conditional expression on the fields compiles to a select of addresses,
// which puts the cursor into memory, or to branches), and the main loop calls the two halves of the
// update in two different gaps.  Past the end of the last run the cursor stays on the last tile: the
// pipeline requests NS - 1 tiles more than it uses, and those refetch valid data.
struct KCursor {
  uint64_t a, b;      // bases of the next tile
  int rem;            // tiles left in the current run, this one included
  uint64_t step_a, step_b;
  // runs after the current one (MULTI only): what to add to a / b at the switch instead of the step
  // (start of that run minus last tile of the one before), and the run lengths (0: no such run)
  uint64_t da1, db1, da2, db2;
  int rn1, rn2;
  // masks of the update in progress: all ones when the run has another tile / when the next run starts
  uint64_t m_stay, m_sw;
};
// first half: hands out the current tile and moves the bases on
template <bool MULTI>
__device__ __forceinline__ void cursor_bases(KCursor& c, const char*& abase, const char*& bbase) {
  abase = (const char*)c.a;
  bbase = (const char*)c.b;
  c.m_stay = (uint64_t)(int64_t)(c.rem > 1 ? -1 : 0);
  if constexpr (MULTI) {
    c.m_sw = (uint64_t)(int64_t)((c.rem <= 1 && c.rn1 > 0) ? -1 : 0);
    c.a += (c.step_a & c.m_stay) | (c.da1 & c.m_sw);
    c.b += (c.step_b & c.m_stay) | (c.db1 & c.m_sw);
  } else {
    c.a += c.step_a & c.m_stay;
    c.b += c.step_b & c.m_stay;
  }
}
// second half: the run counters
template <bool MULTI>
__device__ __forceinline__ void cursor_counts(KCursor& c) {
  const int i_stay = (int)c.m_stay;
  if constexpr (MULTI) {
    const int i_sw = (int)c.m_sw;
    c.rem = ((c.rem - 1) & i_stay) | (c.rn1 & i_sw) | (1 & ~(i_stay | i_sw));
    c.da1 = (c.da2 & c.m_sw) | (c.da1 & ~c.m_sw);
    c.db1 = (c.db2 & c.m_sw) | (c.db1 & ~c.m_sw);
    c.rn1 = (c.rn2 & i_sw) | (c.rn1 & ~i_sw);
    c.rn2 = c.rn2 & ~i_sw;
  } else {
    c.rem += i_stay;  // counts down to 1 and stays there
  }
}
template <bool MULTI>
__device__ __forceinline__ void cursor_next(KCursor& c, const char*& abase, const char*& bbase) {
  cursor_bases<MULTI>(c, abase, bbase);
  cursor_counts<MULTI>(c);
}

// EPI_T: the epilogue kind, plus EPI_DROP when the result passes a dropout site (a separate instantiation,
// so that the kernels without dropout keep their register budget).
constexpr int EPI_DROP = 8;
// k-tiles of 64 in three stages of A and two of B: the whole LDS for 256x256 tiles, half of it for 128x128
template <int BM, int BN, int NS, int BK>
constexpr bool ab_ring = BK == 64 && NS == 3 && (BM == 256 || (BM == 128 && BN == 128));
// ... plus EPI_GROUP for a grouped launch (several problems of one shape, operands from a pointer table).
constexpr int EPI_GROUP = 16;
template <int BM, int BN, int WM, int WN, bool A_KC, bool B_KC, int EPI_T, int NS, int MINW, int BK>
__global__ __launch_bounds__(WM * WN * 64, MINW) void gemm_mfma_kernel(GemmDesc g, GemmEpi e, int tiles_m,
                                                                int tiles_n, int split_k) {
  constexpr int EPI = EPI_T & (EPI_DROP - 1);
  constexpr bool DROP = (EPI_T & EPI_DROP) != 0;
  constexpr bool GROUP = (EPI_T & EPI_GROUP) != 0;
  constexpr int NW = WM * WN;
  constexpr bool AB32 = ab_ring<BM, BN, NS, BK>;  // three stages of A and two of B (see ab_loop)
  constexpr int TMW = BM / WM, TNW = BN / WN;
  constexpr int MI = TMW / 32, NI = TNW / 32;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int A_DMA = A_BYTES / 1024 / NW, B_DMA = B_BYTES / 1024 / NW;  // DMA instructions per wave
  constexpr int DMA_PER_TILE = A_DMA + B_DMA;
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "tile vs wave count");
  static_assert(AB32 || (NS - 1) * DMA_PER_TILE < 64, "vmcnt range");
  constexpr int KSTEPS = BK / 16;
  constexpr int RPB = 512 / BK;  // rows of a k-contiguous stage per 1 KB block
  constexpr int CPRK = BK / 8;   // 16-byte chunks per such row
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- XCD-aware mapping.  Workgroup ids are dealt round-robin to the 8 XCDs; give each XCD a
  // contiguous chunk of the (k-slice, tile) space so that whole k-slices, and compact blocks of
  // tiles inside them, share operand panels through one L2.
  const int nb = tiles_m * tiles_n;
  const int ngr = GROUP ? g.ngroups : 1;
  int L;
  {
    const int total = nb * split_k * ngr;
    const int bid = blockIdx.x;
    const int xcd = bid & 7, idx = bid >> 3;
    const int nb8 = (total + 7) >> 3, rem = total & 7;
    if (rem == 0 || xcd < rem) L = xcd * nb8 + idx; else L = rem * nb8 + (xcd - rem) * (nb8 - 1) + idx;
  }
  // grouped launch: the problem this workgroup belongs to, and its operands and outputs
  const void *seg_a = g.seg[0].A, *seg_b = g.seg[0].B;
  void *so0 = e.out0, *so1 = e.out1, *so2 = e.out2;
  if constexpr (GROUP) {
    {
      const int grp = L / (nb * split_k);
      L -= grp * nb * split_k;
      const void* const* t = g.groups + (size_t)grp * GEMM_GROUP_PTRS;
      seg_a = t[0]; seg_b = t[1];
      so0 = const_cast<void*>(t[2]); so1 = const_cast<void*>(t[3]); so2 = const_cast<void*>(t[4]);
    }
  }
  if constexpr (A_KC && !B_KC) {  // columns from several matrices: offsets count from the lowest
    for (int s = 1; s < g.nsrc; ++s) seg_b = (uint64_t)g.seg[s].B < (uint64_t)seg_b ? g.seg[s].B : seg_b;
  }
  const int ks = L / nb;  // split-k slice
  L -= ks * nb;
  constexpr int GM = 8;
  const int per_group = GM * tiles_n;
  const int group = L / per_group, in_g = L - group * per_group;
  const int first_m = group * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int tm = first_m + in_g % gsz, tn = in_g / gsz;
  const int m0 = tm * BM, n0 = tn * BN;

  // ---- k-tile range of this workgroup (flattened over segments; lda/ldb are equal across segments)
  int nk_total = 0;
  for (int s = 0; s < g.nseg; ++s) nk_total += g.seg[s].K / BK;
  const int per = (nk_total + split_k - 1) / split_k;
  const int kt_begin = ks * per;
  const int kt_end = (kt_begin + per) < nk_total ? (kt_begin + per) : nk_total;
  const int nk = kt_end - kt_begin;
  const int lda = g.seg[0].lda, ldb = g.seg[0].ldb;

  // ---- per-lane byte offsets of this wave's DMA slots (loop invariant)
  uint32_t a_off[A_DMA], b_off[B_DMA];
#pragma unroll
  for (int i = 0; i < A_DMA; ++i) {
    const int q = wave + i * NW;  // 1 KB block inside the A stage
    if constexpr (A_KC) {
      const int row = q * RPB + lane / CPRK;
      const int chunk = (lane % CPRK) ^ kc_swz<BK>(row);
      int gr = m0 + row;
      gr = gr < g.M ? gr : g.M - 1;
      a_off[i] = (uint32_t)gr * (uint32_t)lda * 2u + (uint32_t)chunk * 16u;
    } else {
      constexpr int CPR = BM / 8;  // 16-byte chunks per k-row
      const int slot = q * 64 + lane;
      const int krow = slot / CPR, pch = slot % CPR;
      const int gch = (((pch >> 1) ^ mc_swz<BM>(krow)) << 1) | (pch & 1);
      int mm = m0 + gch * 8;
      mm = mm < g.M ? mm : g.M - 8;
      a_off[i] = (uint32_t)krow * (uint32_t)lda * 2u + (uint32_t)mm * 2u;
    }
  }
#pragma unroll
  for (int i = 0; i < B_DMA; ++i) {
    const int q = wave + i * NW;
    if constexpr (B_KC) {
      const int row = q * RPB + lane / CPRK;
      const int chunk = (lane % CPRK) ^ kc_swz<BK>(row);
      int gr = n0 + row;
      gr = gr < g.N ? gr : g.N - 1;
      b_off[i] = (uint32_t)gr * (uint32_t)ldb * 2u + (uint32_t)chunk * 16u;
    } else {
      constexpr int CPR = BN / 8;
      const int slot = q * 64 + lane;
      const int krow = slot / CPR, pch = slot % CPR;
      const int gch = (((pch >> 1) ^ mc_swz<BN>(krow)) << 1) | (pch & 1);
      int nn = n0 + gch * 8;
      nn = nn < g.N ? nn : g.N - 8;
      b_off[i] = (uint32_t)krow * (uint32_t)ldb * 2u;
      if constexpr (A_KC) {  // weights as they are stored: the column's matrix, and its column there
        int src = 0;
        if constexpr (EPI == EPI_GEGLU_FWD) {  // packed columns: 32 of wi0, 32 of wi1, ...
          src = (nn >> 5) & 1;
          nn = ((nn >> 6) << 5) + (nn & 31);
        } else if (g.nsrc > 1) {
          src = nn / g.nsrc_cols;
          nn -= src * g.nsrc_cols;
        }
        b_off[i] += (uint32_t)((uint64_t)(src == 0 ? g.seg[0].B : src == 1 ? g.seg[1].B : g.seg[2].B) - (uint64_t)seg_b);
      }
      b_off[i] += (uint32_t)nn * 2u;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

  KCursor kc;
  kc.step_a = A_KC ? (uint64_t)BK * 2 : (uint64_t)BK * (uint64_t)lda * 2;
  kc.step_b = B_KC ? (uint64_t)BK * 2 : (uint64_t)BK * (uint64_t)ldb * 2;
  kc.da1 = kc.db1 = kc.da2 = kc.db2 = 0;
  kc.rn1 = kc.rn2 = 0;
  kc.m_stay = kc.m_sw = 0;
  if (g.nseg == 1) {
    kc.a = (uint64_t)seg_a + (uint64_t)kt_begin * kc.step_a;
    kc.b = (uint64_t)seg_b + (uint64_t)kt_begin * kc.step_b;
    kc.rem = nk;
  } else {  // several segments are never split along k
    const int n0 = g.seg[0].K / BK, n1 = g.seg[1].K / BK;
    kc.a = (uint64_t)g.seg[0].A; kc.b = (uint64_t)g.seg[0].B; kc.rem = n0;
    kc.da1 = (uint64_t)g.seg[1].A - (kc.a + (uint64_t)(n0 - 1) * kc.step_a);
    kc.db1 = (uint64_t)g.seg[1].B - (kc.b + (uint64_t)(n0 - 1) * kc.step_b);
    kc.rn1 = n1;
    if (g.nseg > 2) {
      kc.da2 = (uint64_t)g.seg[2].A - ((uint64_t)g.seg[1].A + (uint64_t)(n1 - 1) * kc.step_a);
      kc.db2 = (uint64_t)g.seg[2].B - ((uint64_t)g.seg[1].B + (uint64_t)(n1 - 1) * kc.step_b);
      kc.rn2 = g.seg[2].K / BK;
    }
  }
  // Issue DMA instructions [d0, d1) of a k-tile into stage `st`; a tile's DMA_PER_TILE instructions
  // per wave are numbered A slots first, then B slots.
  // The DMA instructions take their base address from scalar registers.  Addresses that came out of a group
  // table are the same in every lane but live in vector registers: broadcast them from the first lane.
  auto uniform = [](const char* q) __attribute__((always_inline)) {
    const uint64_t v = (uint64_t)q;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char*)(((uint64_t)hi << 32) | lo);
  };
  auto dma_part = [&](const char* abase, const char* bbase, int st, int d0, int d1) __attribute__((always_inline)) {
    // (also without a group table: where the compiler keeps a cursor value in vector registers across a
    // barrier this moves it back; on a value that is already scalar it folds away)
    abase = uniform(abase);
    bbase = uniform(bbase);
    const uint32_t sa = lds0 + st * STAGE, sb = sa + A_BYTES;
#pragma unroll
    for (int d = 0; d < DMA_PER_TILE; ++d) {
      if (d < d0 || d >= d1) continue;
      if (d < A_DMA) dma_1k(sa + (wave + d * NW) * 1024, abase, a_off[d < A_DMA ? d : 0]);
      else dma_1k(sb + (wave + (d - A_DMA) * NW) * 1024, bbase, b_off[d >= A_DMA ? d - A_DMA : 0]);
    }
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  bf16x8 fa[2][MI], fb[2][NI];
  auto load_frags = [&](int st, int kk, int slot) __attribute__((always_inline)) {
    const char* sa = smem + st * STAGE;
    const char* sb = sa + A_BYTES;
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[slot][i] = load_frag<BM, A_KC, BK>(sa, wm * TMW + i * 32, kk, lane);
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[slot][j] = load_frag<BN, B_KC, BK>(sb, wn * TNW + j * 32, kk, lane);
  };
  // One k-step in MI chunks.  Chunk i issues its share of `dcount` DMA instructions (numbers dbase..)
  // of a k-tile into stage dst, fetches its share of the next k-step's fragments (stage ld_st,
  // k-step ld_kk, into register set nxt) and runs the MFMAs of accumulator row i from register set
  // cur.  The DMA instructions are spread out because a wave that issues them back to back sits in
  // the memory pipeline's issue queue instead of feeding the matrix unit.  The fragment reads all go
  // into the first MI - 1 chunks, in the order the next k-step consumes them (its first chunk needs
  // A row 0 and every B column): the last chunk's MFMAs then cover their latency, so that neither the
  // next k-step's first MFMA nor the wait before a barrier finds a read still in flight.
  auto kstep = [&](int cur, int ld_st, int ld_kk, int nxt, const char* abase, const char* bbase, int dst,
                   int dbase, int dcount, auto&& gap) __attribute__((always_inline)) {
    const char* sa = smem + ld_st * STAGE;
    const char* sb = sa + A_BYTES;
    constexpr int NLD = MI + NI;              // fragment reads of one k-step
    constexpr int LCH = MI > 1 ? MI - 1 : 1;  // chunks that carry them
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (dcount > 0) dma_part(abase, bbase, dst, dbase + i * dcount / MI, dbase + (i + 1) * dcount / MI);
#pragma unroll
      for (int q = 0; q < NLD; ++q) {  // read q: A row 0, B columns 0 .. NI-1, A rows 1 .. MI-1
        if (q * LCH / NLD != i) continue;
        if (q == 0) fa[nxt][0] = load_frag<BM, A_KC, BK>(sa, wm * TMW, ld_kk, lane);
        else if (q <= NI) fb[nxt][q - 1] = load_frag<BN, B_KC, BK>(sb, wn * TNW + (q - 1) * 32, ld_kk, lane);
        else fa[nxt][q - NI] = load_frag<BM, A_KC, BK>(sa, wm * TMW + (q - NI) * 32, ld_kk, lane);
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
        if (j == 0) gap(i);  // scalar bookkeeping of the caller, in the shadow of the MFMA just issued
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto no_gap = [](int) __attribute__((always_inline)) {};
  constexpr int H0 = DMA_PER_TILE / 2;  // a tile's DMA is issued in two parts: [0, H0) and [H0, DMA_PER_TILE)

  // The k loop, compiled twice: for one run of tiles (one segment) and for several.
  auto k_loop = [&](auto multi_tag) __attribute__((always_inline)) {
    constexpr bool MULTI = decltype(multi_tag)::value;
    // Prologue: fill stages 0 .. NS-2 and the first part of stage NS-1, wait for tile 0.
    const char *ab, *bb;
#pragma unroll
    for (int s = 0; s + 1 < NS; ++s) {
      cursor_next<MULTI>(kc, ab, bb);
      dma_part(ab, bb, s, 0, DMA_PER_TILE);
    }
    cursor_next<MULTI>(kc, ab, bb);
    dma_part(ab, bb, NS - 1, 0, H0);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 2) * DMA_PER_TILE + H0) : "memory");
    load_frags(0, 0, 0);
    // One k-tile out of stage s.  k-step 0 also issues the second part of tile t+NS-1 (its stage was
    // released at the previous barrier) and, in two of its gaps, works out the addresses of tile t+NS:
    // whatever stands between the barrier and the next MFMA is a bubble in the matrix pipe.  k-steps
    // 1 .. KSTEPS-2 issue nothing.  At the barrier tile t+1 has landed (this wave's part) and all of
    // this wave's reads of stage s are done; after it that holds for every wave, so the last k-step
    // refills stage s with the first part of tile t+NS.
    auto ktile = [&](int s) __attribute__((always_inline)) {
      const char *an = ab, *bn = bb;
      kstep(0, s, 1, 1, ab, bb, (s + NS - 1) % NS, H0, DMA_PER_TILE - H0, [&](int i) __attribute__((always_inline)) {
        if (i == 0) cursor_bases<MULTI>(kc, an, bn);
        if (i == 1) cursor_counts<MULTI>(kc);
      });
#pragma unroll
      for (int kk = 1; kk + 1 < KSTEPS; ++kk) kstep(kk & 1, s, kk + 1, (kk + 1) & 1, ab, bb, 0, 0, 0, no_gap);
      ab = an; bb = bn;  // tile t + NS
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * DMA_PER_TILE) : "memory");
      kstep((KSTEPS - 1) & 1, (s + 1) % NS, 0, 0, ab, bb, s, 0, H0, no_gap);
    };
    // whole rounds of the stage ring run without a test per tile; the last, partial round tests
    int t = 0;
    for (; t + NS <= nk; t += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) ktile(s);
    }
#pragma unroll
    for (int s = 0; s + 1 < NS; ++s)
      if (t + s < nk) ktile(s);
    // drain DMA that was issued past the end before LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  // The same loop for k-tiles of 64 with three A stages and two B stages (5 x 32 KB, the whole LDS).  Two stages of both
  // force a tile's 16 DMA instructions per wavefront into the first half of the tile before (the second half is their
  // latency), two per group of MFMAs, which is as fast as the address path takes them (a DMA instruction of 1 KB keeps
  // it busy for 16 cycles, four wavefronts' two for the 128 cycles of a group): the wavefronts queue there and the
  // matrix pipe waits.  With a third A stage the period between two barriers has 16 groups of MFMAs and one DMA
  // instruction in each: B of tile t+1 in the first half (needed at the end of the period), A of tile t+2 in the second.
  auto ab_loop = [&](auto multi_tag) __attribute__((always_inline)) {
    constexpr bool MULTI = decltype(multi_tag)::value;
    KCursor ka = kc, kb = kc;
    const char *an, *bn, *skip;
    auto dma_a = [&](const char* base, int st, int d0, int d1) __attribute__((always_inline)) {
      base = uniform(base);
#pragma unroll
      for (int d = 0; d < A_DMA; ++d)
        if (d >= d0 && d < d1) dma_1k(lds0 + st * A_BYTES + (wave + d * NW) * 1024, base, a_off[d]);
    };
    auto dma_b = [&](const char* base, int st, int d0, int d1) __attribute__((always_inline)) {
      base = uniform(base);
#pragma unroll
      for (int d = 0; d < B_DMA; ++d)
        if (d >= d0 && d < d1) dma_1k(lds0 + 3 * A_BYTES + st * B_BYTES + (wave + d * NW) * 1024, base, b_off[d]);
    };
    // one k-step: see kstep above; dma(i) issues chunk i's DMA instruction
    auto step = [&](int cur, int sa, int sb, int kk, auto&& dma, auto&& gap) __attribute__((always_inline)) {
      const char* pa = smem + sa * A_BYTES;
      const char* pb = smem + 3 * A_BYTES + sb * B_BYTES;
      const int nxt = cur ^ 1;
      constexpr int NLD = MI + NI, LCH = MI - 1;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        dma(i);
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
          if (q * LCH / NLD != i) continue;
          if (q == 0) fa[nxt][0] = load_frag<BM, A_KC, BK>(pa, wm * TMW, kk, lane);
          else if (q <= NI) fb[nxt][q - 1] = load_frag<BN, B_KC, BK>(pb, wn * TNW + (q - 1) * 32, kk, lane);
          else fa[nxt][q - NI] = load_frag<BM, A_KC, BK>(pa, wm * TMW + (q - NI) * 32, kk, lane);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
          if (j == 0) gap(i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    cursor_next<MULTI>(ka, an, skip); dma_a(an, 0, 0, A_DMA);
    cursor_next<MULTI>(kb, skip, bn); dma_b(bn, 0, 0, B_DMA);
    cursor_next<MULTI>(ka, an, skip); dma_a(an, 1, 0, A_DMA);
    cursor_next<MULTI>(kb, skip, bn); dma_b(bn, 1, 0, B_DMA / 2);
    cursor_next<MULTI>(ka, an, skip);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(A_DMA + B_DMA / 2) : "memory");
    {
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[0][i] = load_frag<BM, A_KC, BK>(smem, wm * TMW + i * 32, 0, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[0][j] = load_frag<BN, B_KC, BK>(smem + 3 * A_BYTES, wn * TNW + j * 32, 0, lane);
    }
    // tile t in A stage sa and B stage sb; an: A of tile t+2, bn: B of tile t+1
    auto ktile = [&](int sa, int sb) __attribute__((always_inline)) {
      constexpr int QA = A_DMA / 2 / MI;  // A's DMA instructions per group of MFMAs
      constexpr int G1 = MI > 2 ? 1 : 0;  // the gaps that move the cursors
      constexpr int HB = B_DMA / 2;       // B's: half in each of two k-steps, over the groups (256x192 tiles: 0 1 1 1)
      static_assert(QA * 2 * MI == A_DMA && HB * 2 == B_DMA, "shares of the groups");
      const char *a2 = an, *b2 = bn;
      step(0, sa, sb, 1, [&](int i) __attribute__((always_inline)) { dma_b(bn, sb ^ 1, HB + i * HB / MI, HB + (i + 1) * HB / MI); },
           [&](int i) __attribute__((always_inline)) { if (i == G1) cursor_bases<MULTI>(kb, skip, b2); if (i == G1 + 1) cursor_counts<MULTI>(kb); });
      step(1, sa, sb, 2, [&](int i) __attribute__((always_inline)) { dma_a(an, (sa + 2) % 3, i * QA, (i + 1) * QA); }, no_gap);
      step(0, sa, sb, 3, [&](int i) __attribute__((always_inline)) { dma_a(an, (sa + 2) % 3, A_DMA / 2 + i * QA, A_DMA / 2 + (i + 1) * QA); },
           [&](int i) __attribute__((always_inline)) { if (i == G1) cursor_bases<MULTI>(ka, a2, skip); if (i == G1 + 1) cursor_counts<MULTI>(ka); });
      an = a2; bn = b2;
      // tile t+1 has landed but for nothing (only A of tile t+2, requested last, may be in flight), and this
      // wavefront's reads of tile t are done
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(A_DMA) : "memory");
      step(1, (sa + 1) % 3, sb ^ 1, 0, [&](int i) __attribute__((always_inline)) { dma_b(bn, sb, i * HB / MI, (i + 1) * HB / MI); }, no_gap);
    };
    int t = 0;
    for (; t + 6 <= nk; t += 6) {
      ktile(0, 0); ktile(1, 1); ktile(2, 0); ktile(0, 1); ktile(1, 0); ktile(2, 1);
    }
    if (t < nk) ktile(0, 0);
    if (t + 1 < nk) ktile(1, 1);
    if (t + 2 < nk) ktile(2, 0);
    if (t + 3 < nk) ktile(0, 1);
    if (t + 4 < nk) ktile(1, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  if (nk > 0) {
    if constexpr (AB32) {
      if (g.nseg == 1) ab_loop(std::false_type{});
      else ab_loop(std::true_type{});
    } else {
      if (g.nseg == 1) k_loop(std::false_type{});
      else k_loop(std::true_type{});
    }
  }
  // Rows of a reduction whose length is not a multiple of BK (weight gradients over a ragged number of tokens):
  // one more k-tile, fetched through registers with zeros past the end, by the last k-slice.  Its cost is one
  // exposed load latency per workgroup (3 us), where the whole product used to go to the general-shape kernel
  // (d 768, 8991 tokens: 2270 us per weight gradient against 60 here).
  if constexpr (!A_KC) {
    const int ktail = g.seg[0].K - nk_total * BK;
    if (ktail > 0 && ks == split_k - 1) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the stages are free
      const char* pa = (const char*)seg_a + (size_t)nk_total * BK * lda * 2;
      const char* pb = (const char*)seg_b + (size_t)nk_total * BK * ldb * 2;
#pragma unroll
      for (int i = 0; i < A_DMA; ++i) {
        const int blk = wave + i * NW, krow = (blk * 64 + lane) / (BM / 8);
        u32x4 v = {0, 0, 0, 0};
        if (krow < ktail) v = *reinterpret_cast<const u32x4*>(pa + a_off[i]);
        *reinterpret_cast<u32x4*>(smem + blk * 1024 + lane * 16) = v;
      }
#pragma unroll
      for (int i = 0; i < B_DMA; ++i) {
        const int blk = wave + i * NW, krow = (blk * 64 + lane) / (BN / 8);
        u32x4 v = {0, 0, 0, 0};
        if (krow < ktail) v = *reinterpret_cast<const u32x4*>(pb + b_off[i]);
        *reinterpret_cast<u32x4*>(smem + A_BYTES + blk * 1024 + lane * 16) = v;
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        load_frags(0, kk, 0);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[0][j], acc[i][j], 0, 0, 0);
      }
    }
  }

  // Output placement of the epilogue, in locals: the reproducible split reduction redirects it.  There this
  // k-slice stores its partial sums, as a plain M x N float32 matrix of its own, instead of adding them into the
  // output; splitk_reduce_kernel adds the slices up afterwards.
  int ep_ld0 = e.ld0, ep_split_n = e.split_n, ep_acc = e.accumulate, ep_sk = split_k;
  if constexpr (EPI == EPI_SPLIT_F32 && !GROUP) {
    if (e.aux0 != nullptr && split_k > 1) {
      so0 = (float*)const_cast<void*>(e.aux0) + (size_t)ks * (size_t)g.M * (size_t)g.N;
      ep_ld0 = g.N;
      ep_split_n = 1 << 30;
      ep_acc = 0;
      ep_sk = 1;
    }
  }
  // ---- epilogue.  acc[i][j][r]: row = (r/4)*8 + (lane/32)*4 + r%4, col = lane%32 of the 32x32 tile.
  // Interior wave tiles (the common case) are transposed through LDS, 64 rows at a time, so that
  // each lane ends up with 4 consecutive columns of one row: auxiliary loads and the stores are
  // then 8- or 16-byte vector accesses covering whole rows of the wave tile.  Edge tiles take the
  // predicated per-element path further down.
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every wave is done with the k-loop stages
  {
    constexpr int EP_LD = TNW + 8;  // floats per staged row
    const int mw = m0 + wm * TMW, nw = n0 + wn * TNW;
    bool interior = (mw + TMW <= g.M) && (nw + TNW <= g.N) && (ep_ld0 % 8 == 0) && (e.ld_aux % 8 == 0);
    if constexpr (EPI == EPI_SPLIT_F32)
      interior = interior && (nw / ep_split_n == (nw + TNW - 1) / ep_split_n) && (ep_split_n % 4 == 0);
    if constexpr (EPI == EPI_SPLIT_F32) {
      // split-k partial sums go out as float atomics straight from the accumulator registers
      // (32 consecutive floats per half-wave and row)
      if (interior && ep_sk > 1) {
        const int cl = lane & 31, rl = (lane >> 5) << 2;
        const int which = nw / ep_split_n;
        float* dst0 = (float*)(which == 0 ? so0 : which == 1 ? so1 : so2) + (nw - which * ep_split_n) + cl;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float* rowp = dst0 + (size_t)(mw + i * 32 + ((r >> 2) << 3) + rl + (r & 3)) * ep_ld0;
#pragma unroll
            for (int j = 0; j < NI; ++j) unsafeAtomicAdd(rowp + j * 32, acc[i][j][r]);
          }
        return;
      }
    }
#define T5MI_EPI_EDGE 0
    if (interior) {
      float* stg = reinterpret_cast<float*>(smem) + wave * (64 * EP_LD);
      const int cl = lane & 31, rl = (lane >> 5) << 2;
      // 64 rows of the wave tile into the staging block (a macro, so that the textually included copies of the
      // row-wise epilogue below can use it as well)
#define T5MI_STAGE_HALF(half)                                                                              \
  do {                                                                                                     \
    _Pragma("unroll") for (int ii = 0; ii < 2; ++ii)                                                       \
      _Pragma("unroll") for (int j = 0; j < NI; ++j)                                                       \
        _Pragma("unroll") for (int r = 0; r < 16; ++r)                                                     \
          stg[(ii * 32 + ((r >> 2) << 3) + rl + (r & 3)) * EP_LD + j * 32 + cl] = acc[(half) * 2 + ii][j][r]; \
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                                     \
    __builtin_amdgcn_wave_barrier();                                                                       \
  } while (0)
      if constexpr (EPI == EPI_GEGLU_FWD) {
        // The activation is chosen once per tile, outside the element loops: tested per element, the choice
        // becomes a branch around every evaluation and the epilogue falls apart into hundreds of short blocks.
        auto passes = [&](auto erf_tag) __attribute__((always_inline)) {
        constexpr bool ERF = decltype(erf_tag)::value;
#pragma unroll
        for (int half = 0; half < MI / 2; ++half) {
          T5MI_STAGE_HALF(half);
          const int mh = mw + half * 64;
          // staged columns: [u 32 | w 32] pairs; lane takes 4 consecutive f of one row
          constexpr int LPR = TNW / 8;  // lanes per row
          const int fl = (lane % LPR) * 4;
          const int pc = (fl >> 5) * 64 + (fl & 31);  // staged column of u; w is 32 further
          const int f = (nw >> 1) + fl;
#pragma unroll
          for (int it = 0; it < 64 / (64 / LPR); ++it) {
            const int rloc = it * (64 / LPR) + lane / LPR;
            const f32x4 uu = *reinterpret_cast<const f32x4*>(stg + rloc * EP_LD + pc);
            const f32x4 ww = *reinterpret_cast<const f32x4*>(stg + rloc * EP_LD + pc + 32);
            bf16x4 gpb, glb, ab;
            f32x4 mk = {1.f, 1.f, 1.f, 1.f};
            if constexpr (DROP) {
              const uint32_t k1 = drop_row_key(e.drop, (uint32_t)(mh + rloc));
#pragma unroll
              for (int q = 0; q < 4; ++q) mk[q] = drop_mult(e.drop, k1, (uint32_t)(f + q));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float gl, dgl;
              if constexpr (ERF) gelu_erf_both(uu[q], gl, dgl); else gelu_tanh_both(uu[q], gl, dgl);
              gpb[q] = (bf16)(ww[q] * dgl * mk[q]);
              glb[q] = (bf16)(gl * mk[q]);
              ab[q] = (bf16)(gl * ww[q] * mk[q]);
            }
            const size_t o = (size_t)(mh + rloc) * ep_ld0 + f;
            st_stream(reinterpret_cast<bf16x4*>((bf16*)e.out0 + o), gpb);
            st_stream(reinterpret_cast<bf16x4*>((bf16*)e.out1 + o), glb);
            st_stream(reinterpret_cast<bf16x4*>((bf16*)e.out2 + o), ab);
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_wave_barrier();
        }
        };
        if (e.act == ACT_GELU_ERF) passes(std::true_type{}); else passes(std::false_type{});
      } else {
        // Run-time properties of the epilogue (operand and output types, the rarely used ReLU forms, accumulation)
        // are turned into compile-time ones here, once per tile: tested where they are used, inside the unrolled
        // element loops, each becomes a branch per instruction and the epilogue falls apart into short blocks that
        // the scheduler cannot overlap (gated-GELU forward +13 %, output projection with the float32 residual +5 %).
        // The rare combinations share one copy that reads them at run time, so that the number of copies stays small.
        if constexpr (EPI == EPI_GEGLU_BWD) {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 1
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
        } else if constexpr (EPI == EPI_SPLIT_F32) {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 0
#define T5MI_EPI_SP 2
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
        } else if constexpr (EPI == EPI_RESID) {
          const bool af = e.aux_type != IN_BF16;
          const bool ob = e.out_type == IN_BF16;
          if (e.aux_mask != 0) {
#define T5MI_EPI_AF 2
#define T5MI_EPI_OB 2
#define T5MI_EPI_SP 1
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
          } else if (af) {
            if (ob) {
#define T5MI_EPI_AF 1
#define T5MI_EPI_OB 1
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
            } else {
#define T5MI_EPI_AF 1
#define T5MI_EPI_OB 0
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
            }
          } else {
            if (ob) {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 1
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
            } else {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 0
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
            }
          }
        } else {
          // plain store
          if (e.act == ACT_RELU) {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 2
#define T5MI_EPI_SP 1
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
          } else if (e.out_type == IN_BF16) {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 1
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
          } else {
#define T5MI_EPI_AF 0
#define T5MI_EPI_OB 0
#define T5MI_EPI_SP 0
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
          }
        }
      }
      return;
    }
#undef T5MI_EPI_EDGE
    // A last tile of rows that is not full takes the row-wise path too, its missing rows left out.  Element by element,
    // with the residual read one value at a time, it took longer than the rest of the launch: 18668 x 512 x 1024 with
    // residual, 146 tiles of 256x256, 106 -> 45 us (18432 rows: 36); 31713 x 2048 x 5120 614 -> 545.
    // A wave whose tile lies wholly outside ends here (no barrier follows) instead of stepping over its elements one by
    // one: 9344 x 1024 x 1024 52 -> 41 us.  Plain stores and gated-GELU backward keep the walk: with a return at the
    // top of the epilogue for every kind, 25600 x 3072 x 1024 went from 155 to 190 us.
    if constexpr (EPI == EPI_RESID)
      if (mw >= g.M || nw >= g.N) return;
    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID || EPI == EPI_GEGLU_BWD) {
      if (mw < g.M && nw + TNW <= g.N && ep_ld0 % 8 == 0 && e.ld_aux % 8 == 0) {
        float* stg = reinterpret_cast<float*>(smem) + wave * (64 * EP_LD);
        const int cl = lane & 31, rl = (lane >> 5) << 2;
#define T5MI_EPI_EDGE 1
#define T5MI_EPI_AF 2
#define T5MI_EPI_OB 2
#define T5MI_EPI_SP 2
#include "gemm_epilogue_rows.inc"
#undef T5MI_EPI_EDGE
#undef T5MI_EPI_AF
#undef T5MI_EPI_OB
#undef T5MI_EPI_SP
        return;
      }
    }
  }
  // ---- edge tiles: per-element bounds checks
  const int col_l = lane & 31, row_l = (lane >> 5) << 2;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + wm * TMW + i * 32 + ((r >> 2) << 3) + row_l + (r & 3);
      if (m >= g.M) continue;
      if constexpr (EPI == EPI_GEGLU_FWD) {
#pragma unroll
        for (int j = 0; j < NI; j += 2) {
          const int n = n0 + wn * TNW + j * 32;  // packed column of the u tile; w tile follows
          if (n >= g.N) continue;
          const int f = (n >> 6) * 32 + col_l;
          const float uu = acc[i][j][r], ww = acc[i][j + 1][r];
          float gl, dgl;
          gelu_both(e.act, uu, gl, dgl);
          const size_t o = (size_t)m * ep_ld0 + f;
          const float mk = DROP ? drop_mult(e.drop, drop_row_key(e.drop, (uint32_t)m), (uint32_t)f) : 1.f;
          ((bf16*)e.out0)[o] = (bf16)(ww * dgl * mk);
          ((bf16*)e.out1)[o] = (bf16)(gl * mk);
          ((bf16*)e.out2)[o] = (bf16)(gl * ww * mk);
        }
      } else {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int n = n0 + wn * TNW + j * 32 + col_l;
          if (n >= g.N) continue;
          float v = acc[i][j][r];
          const size_t o = (size_t)m * ep_ld0 + n;
          float mk = 1.f;
          if constexpr (EPI == EPI_STORE || EPI == EPI_RESID)
            if constexpr (DROP) mk = drop_mult(e.drop, drop_row_key(e.drop, (uint32_t)m), (uint32_t)n);
          if constexpr (EPI == EPI_STORE) {
            if (e.act == ACT_RELU) v = fmaxf(v, 0.f);
            v *= mk;
            if (e.out_type == IN_BF16) ((bf16*)e.out0)[o] = (bf16)v; else ((float*)e.out0)[o] = v;
          } else if constexpr (EPI == EPI_RESID) {
            const size_t oa = (size_t)m * (e.ld_aux ? e.ld_aux : ep_ld0) + n;
            const float a = e.aux_type == IN_BF16 ? (float)((const bf16*)e.aux0)[oa] : ((const float*)e.aux0)[oa];
            const float r = e.aux_mask ? (a > 0.f ? v * (DROP ? e.drop.scale : 1.f) : 0.f) : fmaf(v, mk, a);
            if (e.out_type == IN_BF16) ((bf16*)e.out0)[o] = (bf16)r; else ((float*)e.out0)[o] = r;
          } else if constexpr (EPI == EPI_GEGLU_BWD) {
            const size_t oa = (size_t)m * (e.ld_aux ? e.ld_aux : ep_ld0) + n;
            const float gp = (float)((const bf16*)e.aux0)[oa], gl = (float)((const bf16*)e.aux1)[oa];
            ((bf16*)e.out0)[o] = (bf16)(v * gp);
            ((bf16*)e.out1)[o] = (bf16)(v * gl);
          } else {  // EPI_SPLIT_F32
            const int which = n / ep_split_n, nn = n - which * ep_split_n;
            float* dst = (float*)(which == 0 ? so0 : which == 1 ? so1 : so2) + (size_t)m * ep_ld0 + nn;
            if (ep_sk > 1) unsafeAtomicAdd(dst, v);
            else *dst = ep_acc ? *dst + v : v;
          }
        }
      }
    }
  }
}

// Tile size and k split of a weight-gradient GEMM (EPI_SPLIT_F32): the cheapest of both tiles with up to 32 slices.  In
// microseconds: a workgroup's k-tile of 64 takes 0.58 with 128x128 tiles and a compute unit to itself (measured 0.54 to 0.62; 1.75 times
// that with two on every unit, 1.65 with two slices' tiles on up to 224 of them) and 1.45 with 256x256; the float atomics of all slices run
// at 340 G/s whatever the split; without slices the tiles leave by plain stores.  Model / measured with operands from
// memory: 768 x 4096 over 8960 tokens 256x256 in five slices 92 / 94, 128x128 unsliced 84 / 80; over 512 tokens 256x256 25 / 21, 128x128
// 8 / 11; 768 x 2304 over 20480, 128x128 in four (432 workgroups) 100 / 90, 256x256 in nine 104 / 103; 2048 x 768 over 28672, 128x128 in five
// 112 / 102, 256x256 in ten 116 / 116; over 65536, 256x256 in ten 200 / 200; 512 x 1024 over 32768, 128x128 in eight 52 / 50, in sixteen
// 60 / 58; 768 x 768 over 8960 in seven 27 / 27.  256x256 tiles that leave a quarter of the units idle take 1.2 a k-tile in short
// runs, but not under the power limit of long ones: charged so, a layer of d 1024 over 32768 tokens went from 3.1 to 3.2 ms.
// From four rounds of 256x256 tiles on a quarter of the atomics hides behind the products of the rounds that follow.  2048 x 10240 over
// 16384: in three slices, four rounds, 612, in two 600, 128x128 731, which a full charge would take.  With the quarter off
// at two and three rounds already, 1024 x 5632 over 13440 would go to five slices (two rounds, 197; two slices in one round 161), 5120 x
// 2048 over 8960 to three (two rounds, 224; unsliced 167), 2048 x 6144 over 19200 to four (three rounds, 453; unsliced 390).
// Grouped launches run many rounds: the atomics hide behind the products of the rounds that follow, but for 17 us each, and
// 128x128 tiles take 0.62 a k-tile (12 x 768 x 4096 over 16384: 1260 us with those, 1080 with 256x256).
void wgrad_plan(const GemmDesc& g, const GemmEpi& e, int ngr, bool& big, int& split_k) {
  int nk = 0;
  for (int s = 0; s < g.nseg; ++s) nk += g.seg[s].K / KQ;
  const int64_t t256 = (int64_t)ceil_div(g.M, 256) * ceil_div(g.N, 256) * ngr;
  const int64_t t128 = (int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 128) * ngr;
  double best = -1.0;
  big = false;
  split_k = 1;
  for (int sp = 1; sp <= 32; ++sp) {
    if (sp > 1 && nk / sp < 8) break;
    const int64_t w256 = t256 * sp, w128 = t128 * sp, rem = w128 % 512;
    const double r256 = (double)((w256 + 255) / 256);
    const double k256 = 1.45 * r256 * nk / sp, atomics = sp > 1 ? (ngr <= 1 && r256 >= 4.0 ? 0.145 : 0.193) * (double)w256 : 8.0;
    const double c256 = k256 + 5.0 + (ngr > 1 ? std::max(17.4 * (r256 - 1.0), atomics - k256 * (r256 - 1.0) / r256) : atomics);
    const double rounds = (double)(w128 / 512) * 1.75 + (rem > 256 ? (ngr <= 1 && sp > 1 && rem <= 480 ? 1.65 : 1.75) : rem > 0 ? 1.0 : 0.0);
    const double c128 = (ngr > 1 && w128 > 512 ? 0.62 : 0.58) * rounds * nk / sp + (sp > 1 ? 0.048 * (double)w128 : 0.0) + 3.0;
    if (best < 0.0 || c128 < best) { best = c128; big = false; split_k = sp; }
    if (c256 < best) { best = c256; big = true; split_k = sp; }
  }
  (void)e;
}
// whether the reproducible two-pass reduction applies to this problem
bool split_partials_ok(const GemmDesc& g, const GemmEpi& e) {
  return e.aux0 != nullptr && g.ngroups <= 1 && g.N % 4 == 0 && e.split_n % 4 == 0 && e.ld0 % 4 == 0;
}

template <int BM, int BN, int WM, int WN, bool A_KC, bool B_KC, int EPI, int NS = 4, int MINW = 1, int BK = 32>
hipError_t launch_cfg(const GemmDesc& g, const GemmEpi& e, int split_k, hipStream_t st) {
  auto kern = gemm_mfma_kernel<BM, BN, WM, WN, A_KC, B_KC, EPI, NS, MINW, BK>;
  constexpr int lds_loop = (ab_ring<BM, BN, NS, BK> ? 3 * BM + 2 * BN : NS * (BM + BN)) * BK * 2;
  constexpr int lds_epi = WM * WN * 64 * (BN / WN + 8) * 4;
  constexpr int lds = lds_loop > lds_epi ? lds_loop : lds_epi;
  // once per instantiation; setting it twice is harmless, so a relaxed flag is enough
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load(std::memory_order_relaxed)) {
    hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (err != hipSuccess) return err;
    attr_set.store(true, std::memory_order_relaxed);
  }
  const int tiles_m = ceil_div(g.M, BM), tiles_n = ceil_div(g.N, BN);
  const int ngr = (EPI & EPI_GROUP) ? g.ngroups : 1;
  kern<<<tiles_m * tiles_n * split_k * ngr, WM * WN * 64, lds, st>>>(g, e, tiles_m, tiles_n, split_k);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, int EPI_T>
hipError_t launch_layout(const GemmDesc& g, const GemmEpi& e, hipStream_t st) {
  constexpr int EPI = EPI_T & (EPI_DROP - 1);
  // a grouped launch (weight gradients of several layers) counts the tiles of all its problems
  const int ngr = (EPI_T & EPI_GROUP) ? g.ngroups : 1;
  const int64_t t256 = (int64_t)ceil_div(g.M, 256) * ceil_div(g.N, 256) * ngr;
  const int64_t t128 = (int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 128) * ngr;
  if constexpr (EPI == EPI_SPLIT_F32) {
    // Partial sums of the k-slices meet in float32 atomics on a zeroed output, or, when the caller provides
    // room for them, in a second pass that adds them up in a fixed order.
    bool big;
    int split_k;
    wgrad_plan(g, e, ngr, big, split_k);
    if (ngr > 1 && !e.accumulate) return hipErrorInvalidValue;  // grouped outputs are cleared by the caller
    const bool two_pass = split_k > 1 && split_partials_ok(g, e);  // through the partial-sum buffer in GemmEpi::aux0
    if (split_k > 1 && !e.accumulate && !two_pass) {
      hipError_t err = launch_zero_split(e, g.M, g.N, st);
      if (err != hipSuccess) return err;
    }
    GemmEpi ee = e;
    if (!two_pass) ee.aux0 = nullptr;
    const hipError_t err = big ? launch_cfg<256, 256, 2, 2, A_KC, B_KC, EPI_T, 3, 1, 64>(g, ee, split_k, st)
                               : launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI_T, 4, 1>(g, ee, split_k, st);
    if (err != hipSuccess || !two_pass) return err;
    return launch_splitk_reduce(ee, g.M, g.N, split_k, st);
  }
  if constexpr (EPI != EPI_SPLIT_F32) {
    // k-contiguous operands, k-tiles of 64 (a DMA instruction then covers eight whole 128-byte rows instead of sixteen
    // half rows; the L1 processes a line per request whatever part of it is used).  In the order tried:
    //  * 256x256, one workgroup per compute unit, three A and two B stages: the fewest operand bytes per flop, so the
    //    fastest where its last round over the 256 compute units is full (32768 x 6144 x 2048: 646 us against 770); also
    //    for the residual epilogue with dropout (32768 x 2048 x 5120 557 us against 675 with 128x128 and 736 with 256x128;
    //    65536 x 768 x 2048 209, 231, 242);
    //  * 128x128, two workgroups per compute unit: a round of 512 tiles costs w of a 256x256 round, which
    //    is four times the work for w = 0.62 (plain store and gated-GELU forward; 0.53 at K < 640, 0.40 for a plain store
    //    whose last 256 columns are not all there: 12800 x 1152 x 512 40 us with 256x256, 25 with this, 25600 rows 59 and
    //    43), with the residual epilogue, whose extra traffic the second workgroup hides, 0.49 (K <= 768), 0.56, from K = 1024 on
    //    0.52, above that 0.555 and from 2049 on 0.61.  A last round of up to 256 tiles costs 0.65 of a full one; as much as a
    //    full one above K = 3072, and from 1024 on where there is only one before it.  (us with 256x256 and with this.  N = 2048, plain
    //    store of 2096 tiles: K 1536 124 and 114, 2048 155 and 144, 3072 210 and 201, 4096 275 and 262, but 2128 of N = 1024 272 and 284;
    //    of 2560: K 1536 130 and 131, 2048 161 and 164, 4096 284 and 296; of 640: 39 and 41, 47 and 51, 80 and 90.  Gated, K 2048, 2304
    //    tiles 172 and 162, 2560 175 and 176.  Residual, 4352 tiles: K 1024 203 and 176, 2048 312 and 299, 4096 527 and 549; 2560 tiles:
    //    123 and 112, 186 and 185, 313 and 329; 3584, K 2560 299 and 315; 520 of N = 1024, K 2048 55 and 60.)  The cheaper sum of rounds is taken
    //    (14592 x 768 x 2304, 171 against 684 tiles: 59 us against 68; 8991 x 768 x 4096, 108 against 426: 92 against 64).
    //    The gated-GELU backward, two tensors in and two out, always takes it (32768 x 5120 x 2048: 1149 us with 256x256,
    //    850 with 256x128, 761 with this in two stages, 730 with three stages of A and two of B, which fill the half of the
    //    LDS that a workgroup has: a tile's requests spread over the whole period between two barriers).  The others have
    //    those stages from K = 1024 on (8991 x 768 x 4096 64.7 -> 59.5 us, 8991 x 768 x 2304 41.6 -> 38.6, 2048 x 10240 x 2048
    //    gated 108 -> 101) and two up to there, where the longer ramp costs as much as it gives (8991 x 2304 x 768 42 -> 41 and
    //    46 in two runs, 32768 x 1152 x 512 54 -> 51 and 57).  A plain store whose round leaves many units with one workgroup
    //    keeps two stages: from K = 1025 up to 384 tiles, from 3072 up to 480 (us with two stages and with the ring, 264 tiles of
    //    5592 x 768: k 1280 20.6 and 22.1, 3072 36.9 and 39.0; 368 of 2904 x 2048: 1536 23.4 and 23.9, 3072 40.6 and 42.1; 464 of
    //    3672 x 2048: 2048 33.8 and 33.3, 3072 46.6 and 46.9; 1024 up to 464 tiles 2-5 % less with the ring; several rounds,
    //    16896 x 1024 x 2048: 83 and 80).  With residual the ring is faster there too (6000 x 768 x 2048, 282 tiles: 35 and 30);
    //  * 256x192, the same loop with three quarters of the columns, where that fills rounds that 256x256 leaves part empty
    //    (widths of 768: 16384 x 768 is 192 tiles of 256x256 and 256 of these).  A round costs 0.88 of a 256x256 one, not
    //    0.75: more units share the power and the L2.  k 4096 98 -> 92 us, 2048 62 -> 57, 768 30 -> 26; 16384 x 2304 x 768,
    //    three rounds of each: 73 -> 69; 8991 x 2304 x 768, two rounds against 2.5 of 128x128: 42 with those, 50 with this.
    //    Above K = 1024 it is compared with 0.62 for every round of 128x128 that is begun, residual or not: two rounds of this against
    //    three, the last one full or not, us: N = 768, residual, 22016 rows, K 2048 85 and 89, 4096 145 and 162; 32768 rows, 104 and
    //    116, 175 and 206; plain store, 24576 rows, K 1536 65 and 65, 2304 85 and 90, 4096 133 and 144 (K 1024 53 and 49);
    //  * 256x128, two workgroups, k-tiles of 32 in three stages: gated-GELU forward up to K = 704, residual up to K = 512
    //    (32768 x 512 x 384: 31 us against 32 and 34);
    //  * up to 256 tiles of 128x128 (one per compute unit): latency counts, so more stages (four of 64, 128 KB) and,
    //    while they fit one round, smaller tiles, 128x64 and 64x64 (1332 x 768 x 2048 with residual: 37 us -> 21;
    //    1332 x 768 x 768: 25 -> 18).  What bounds them is the path from L2 to LDS, 65 GB/s a compute unit with rows of 128 bytes:
    //    four stages of 32 (rows of 64 bytes) took 39.9 us for 3648 x 768 x 4096, these 31.9; k 2304 30.4 and 25.3, 2048 29.5 and
    //    25.3; three stages of 64 43.  The longer ramp of 64 pays from K = 1025 on, with 192 tiles or more from 768 on, for plain
    //    stores always from 768 on, in the gated-GELU backward always (us with 32 and with 64, launched again and again: 160 tiles of
    //    2520 x 1024: k 512 7.8 and 8.9, 1280 15.7 and 13.4; 228 of 4824 x 768: 512 8.7 and 9.5, 768 11.2 and 11.1, 1024 13.3 and 12.8.
    //    Between the other launches of a layer's backward, which leave neither the code nor the operands near: plain store of 138, 156
    //    and 174 tiles, N = K = 768 12.8, 12.9, 13.2 and 11.9, 12.0, 12.4, of 136, 160 and 176, N = K = 1024 15.1, 15.0, 15.5 and 13.6,
    //    13.4, 14.1; with residual 160 tiles of N = K = 1024 17.2 and 18.0).
    //    Beside launches on another stream, whose workgroups find no room on a unit with 128 KB taken, only from 5120 on (backward
    //    with the weight gradients overlapped, us with 32 and with 64 throughout: d 768, k 768, 2304 and 4096, 4096 tokens 253 and
    //    261, 5000 tokens 297 and 309; d 2048, k 2048, 6144 and 10240, 2000 tokens 590 and 536; d 1024, k 1024, 3072 and 5632, 3500
    //    tokens 339 and 332, like this 310 where 64 throughout takes 317);
    int64_t K = 0;
    for (int s = 0; s < g.nseg; ++s) K += g.seg[s].K;
    const double last = K > 3072 || (K >= 1024 && t128 <= 1024) ? 1.0 : 0.65;
    const double w_resid = K <= 768 ? 0.49 : K < 1024 ? 0.56 : K == 1024 ? 0.52 : K <= 2048 ? 0.555 : 0.61;
    const double w = EPI == EPI_RESID ? w_resid : K < 640 ? (EPI == EPI_STORE && g.N % 256 != 0 ? 0.40 : 0.53) : 0.62;
    const double c256 = (double)((t256 + 255) / 256);
    const int64_t rem = t128 % 512;
    const double c128 = w * ((double)(t128 / 512) + (rem > 256 ? 1.0 : rem > 0 ? last : 0.0));
    const double c128_192 = K > 1024 ? 0.62 * (double)((t128 + 511) / 512) : c128;  // (against 256x192)
    if (t128 <= 256) {
      if constexpr (EPI != EPI_GEGLU_FWD) {  // (which needs 64 columns in a wavefront)
        if ((int64_t)ceil_div(g.M, 64) * ceil_div(g.N, 64) <= 256)
          return launch_cfg<64, 64, 1, 2, A_KC, B_KC, EPI_T, 4, 1, 64>(g, e, 1, st);
        if ((int64_t)ceil_div(g.M, 128) * ceil_div(g.N, 64) <= 256)
          return launch_cfg<128, 64, 2, 2, A_KC, B_KC, EPI_T, 3, 1, 64>(g, e, 1, st);
      }
      if (!(g.beside && K < 5120) && (EPI == EPI_GEGLU_BWD || K > 1024 || (K >= 768 && (EPI == EPI_STORE || t128 >= 192))))
        return launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI_T, 4, 1, 64>(g, e, 1, st);
      return launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI_T, 4, 1>(g, e, 1, st);
    }
    if constexpr (EPI_T == EPI_STORE || EPI_T == EPI_RESID) {  // (the dropout copies are not built: 14592 x 768 x 2048 with residual 65 us, 59 like this)
      if (g.N % 192 == 0) {
        const double c192 = 0.88 * (double)(((int64_t)ceil_div(g.M, 256) * (g.N / 192) + 255) / 256);
        if (c192 < c256 && c192 < c128_192) return launch_cfg<256, 192, 2, 2, A_KC, B_KC, EPI_T, 3, 1, 64>(g, e, 1, st);
      }
    }
    if constexpr (EPI == EPI_GEGLU_FWD || EPI == EPI_RESID)
      if (t256 >= 192 && K <= (EPI == EPI_RESID ? 512 : 704))
        return launch_cfg<256, 128, 2, 2, A_KC, B_KC, EPI_T, 3, 2>(g, e, 1, st);
    if constexpr (EPI != EPI_GEGLU_BWD)
      if (c256 <= c128) return launch_cfg<256, 256, 2, 2, A_KC, B_KC, EPI_T, 3, 1, 64>(g, e, 1, st);
    const bool part = EPI == EPI_STORE && K > 1024 && (t128 <= 384 || (K >= 3072 && t128 <= 480));
    if (EPI == EPI_GEGLU_BWD || (K >= 1024 && !part)) return launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI_T, 3, 1, 64>(g, e, 1, st);
    if constexpr (EPI != EPI_GEGLU_BWD) return launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI_T, 2, 1, 64>(g, e, 1, st);
  }
}

}  // namespace
}  // namespace t5mi
