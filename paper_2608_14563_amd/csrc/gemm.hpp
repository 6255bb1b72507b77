// fp32 MFMA tile core for the three contractions of the FPO hot path on
// gfx950 (the logits Y W_U^T, the projection P W_U and the per-layer outer
// product g~^T a) when the operands are fp32: one workgroup of 4 waves (2 x 2)
// computes a 64 x 64 tile of C = A B with v_mfma_f32_16x16x4_f32 (exact
// fp32 products, fp32 accumulation), A stored K-contiguous ([M][K]
// row-major) and B either K-contiguous ([N][K], "Bt") or N-contiguous
// ([K][N]); 32-deep K tiles, register-staged double buffering. bf16 operands
// run on the LDS-DMA core of gemm2.hpp; TileBF16 here only carries their tile
// constants.
//
// Bound by the matrix pipe (64 flop per cycle and SIMD, 157 TFLOP/s), which
// waits for nothing else when four workgroups share a CU: a 64 x 64 tile takes
// 32 KB of LDS and under 128 registers a lane. 128 x 128 tiles (one or two
// workgroups a CU) were 4 to 25% slower at every size measured with the same
// loop, and left most of the chip idle at small ones. Eight layers' outer
// products of 2048 x 2048 x 6144 reach 135 TFLOP/s (127 with the 128 x 128 tiles
// and operands read right before use), T = 600, d = 1032, V = 20000 logits and
// projection 88 (73), T = 128, d = 256, V = 4096 13 (6).
//
// Lane layout. Within one 32-wide K step every lane l owns the eight K
// indices 8*(l>>4) + s, s = 0..7, for both operands (the K order inside the
// sum is a summation order only). Output columns are interleaved: the lane
// owns columns FN*(l&15) + i, i = 0..FN-1, of its wave's tile, so that its
// FN accumulator blocks hold FN consecutive output columns (8-byte epilogue
// stores) and an N-contiguous B tile is read with one 8-byte LDS load per K
// row.
//
// Accumulator acc[f][i][r] holds C[row, col] with
//   row = m0 + wm*WTM + 16*f + 4*(l>>4) + r,  col = n0 + wn*WTN + FN*(l&15) + i.
//
// K-contiguous LDS tiles are stored in 16-byte chunks, 8 chunks per row, with
// chunk index XOR-swizzled by (row ^ (row >> 3)) & 7 so that the lanes of a
// fragment read (consecutive rows, or rows 8 apart) hit distinct banks.
#pragma once

#include "common.hpp"

namespace fpo {

// SB: width of a logits statistics block (the columns of one wave).
struct TileBF16 {  // gemm2.hpp
  using T = uint16_t;
  static constexpr int BM = 256, BN = 256, BK = 64, FM = 8, FN = 8, EPC = 8, SB = 128;
};
struct TileBF16S {  // gemm2s.hpp
  using T = uint16_t;
  static constexpr int BM = 128, BN = 128, BK = 64, FM = 4, FN = 4, EPC = 8, SB = 128;
};
struct TileF32 {
  using T = float;
  static constexpr int BM = 64, BN = 64, BK = 32, FM = 2, FN = 2, EPC = 4, SB = 32;
};

template <class E>
struct Tile {
  using T = typename E::T;
  static constexpr int BM = E::BM, BN = E::BN, BK = E::BK, FM = E::FM, FN = E::FN, EPC = E::EPC, SB = E::SB;
  static constexpr int NT = 256;                 // threads per workgroup
  static constexpr int WTM = 16 * FM, WTN = 16 * FN;
  static constexpr int CPR = BK / EPC;           // chunks per K-contiguous row (8)
  static constexpr int KSTEPS = BK / 32;
  static constexpr int KC = 8 / EPC;             // chunks per lane per K step
  static constexpr int A_CHUNKS = BM * CPR;
  static constexpr int B_CHUNKS = BN * CPR;      // == BK * BN / EPC
  static constexpr int BN_CPR = BN / EPC;        // chunks per N-contiguous row
  static constexpr int A_PT = A_CHUNKS / NT;
  static constexpr int BT_PT = B_CHUNKS / NT;
  static constexpr int BNC_PT = (BK * BN_CPR) / NT;
  static_assert(CPR == 8, "swizzle assumes 8 chunks per row");
};

template <class E>
struct GemmSmem {
  u32x4 a[2][Tile<E>::A_CHUNKS];
  u32x4 b[2][Tile<E>::B_CHUNKS];
};

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

// ---------------------------------------------------------------- loaders
// A [M][lda] K-contiguous; B N-contiguous [K][ldb] (BNC) or K-contiguous
// [N][ldb]. load() takes the K tiles one after the other. Rows (columns) past
// M (N) take the last one's data: they only reach outputs that no epilogue
// stores or reduces, so a whole K tile is loaded without any check. In the last,
// partial K tile whatever lies past K reads as zero.
template <class E, bool BNC>
struct TileLoader {
  using TT = Tile<E>;
  using T = typename E::T;
  static constexpr int NA = TT::A_PT, NB = BNC ? TT::BNC_PT : TT::BT_PT;
  u32x4 ra[NA], rb[NB];
  const T* pa[NA];
  const T* pb[NB];
  int64_t stepb;
  int ka, kb[BNC ? NB : 1];  // K index of the lane's chunks (BNC: of its rows) in K tile 0

  __device__ __forceinline__ void setup(const T* __restrict__ A, int64_t lda, int M, int m0,
                                        const T* __restrict__ B, int64_t ldb, int N, int n0, int kt0) {
    const int t = threadIdx.x, c = t & 7;
    const int64_t k0 = (int64_t)kt0 * TT::BK;
    ka = c * TT::EPC;
#pragma unroll
    for (int j = 0; j < NA; ++j) pa[j] = A + (int64_t)min(m0 + (t >> 3) + 32 * j, M - 1) * lda + k0 + ka;
    if constexpr (BNC) {
      const int cc = t % TT::BN_CPR, r = t / TT::BN_CPR;
      stepb = TT::BK * ldb;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        kb[j] = r + TT::NT / TT::BN_CPR * j;
        pb[j] = B + (k0 + kb[j]) * ldb + min(n0 + cc * TT::EPC, N - TT::EPC);
      }
    } else {
      stepb = TT::BK;
      kb[0] = ka;
#pragma unroll
      for (int j = 0; j < NB; ++j) pb[j] = B + (int64_t)min(n0 + (t >> 3) + 32 * j, N - 1) * ldb + k0 + ka;
    }
  }
  // The loads themselves are unconditional (a branch around them would make the
  // compiler wait for them where it ends): in the partial K tile chunks past K
  // read the tile's first ones, and store() writes zeros for them.
  __device__ __forceinline__ void load(int kt, int K) {
    const int k_rem = K - kt * TT::BK;
    if (k_rem < TT::BK) {
#pragma unroll
      for (int j = 0; j < NA; ++j) pa[j] -= ka < k_rem ? 0 : ka;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int k = kb[BNC ? j : 0];
        pb[j] -= k < k_rem ? 0 : (BNC ? k * (stepb / TT::BK) : k);
      }
    }
#pragma unroll
    for (int j = 0; j < NA; ++j) ra[j] = *reinterpret_cast<const u32x4*>(pa[j]);
#pragma unroll
    for (int j = 0; j < NB; ++j) rb[j] = *reinterpret_cast<const u32x4*>(pb[j]);
#pragma unroll
    for (int j = 0; j < NA; ++j) pa[j] += TT::BK;
#pragma unroll
    for (int j = 0; j < NB; ++j) pb[j] += stepb;
  }
  __device__ __forceinline__ void store(u32x4* sa, u32x4* sb, int kt, int K) {
    const int t = threadIdx.x;
    const int k_rem = K - kt * TT::BK;
    if (k_rem < TT::BK) {
#pragma unroll
      for (int j = 0; j < NA; ++j)
        if (ka >= k_rem) ra[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (kb[BNC ? j : 0] >= k_rem) rb[j] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int row = (t >> 3) + 32 * j, c = t & 7;
      sa[row * 8 + (c ^ swz(row))] = ra[j];
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (BNC) {
        sb[t + TT::NT * j] = rb[j];
      } else {
        const int row = (t >> 3) + 32 * j, c = t & 7;
        sb[row * 8 + (c ^ swz(row))] = rb[j];
      }
    }
  }
};

// ---------------------------------------------------------------- compute
// A wave's operands of one 32-deep K tile, in registers: av[f][s], bv[s][i] for
// the lane's eight K indices s.
template <class E>
struct Frags {
  f32x4 a[E::FM][2];                                // A fragment f, K indices 4q..4q+3
  float __attribute__((ext_vector_type(E::FN))) b[8];  // N-contiguous B: columns of K index s
  f32x4 bt[E::FN][2];                               // K-contiguous B: column i, K indices 4q..4q+3
};

// The LDS reads of a tile are cut into 8 parts, one issued ahead of the MFMAs
// of each K index of the tile before it.
template <class E, bool BNC>
__device__ __forceinline__ void read_part(Frags<E>& fr, const u32x4* __restrict__ sa,
                                          const u32x4* __restrict__ sb, int wm, int wn, int part) {
  using TT = Tile<E>;
  constexpr int FM = E::FM, FN = E::FN;
  using fvec = float __attribute__((ext_vector_type(FN)));
  const int l = threadIdx.x & 63;
  const int lr = l & 15, lg = l >> 4;
  // parts 0 .. FM-1: A fragment `part`, both halves (FM <= 4)
  if (part < FM) {
    const int row = wm * TT::WTM + 16 * part + lr;
#pragma unroll
    for (int q = 0; q < 2; ++q) fr.a[part][q] = __builtin_bit_cast(f32x4, sa[row * 8 + ((2 * lg + q) ^ swz(row))]);
  }
  if constexpr (BNC) {  // every part: K index `part`
    fr.b[part] = reinterpret_cast<const fvec*>(sb)[(8 * lg + part) * (TT::BN / FN) + wn * (TT::WTN / FN) + lr];
  } else if (part >= 4 && part < 4 + FN) {  // parts 4 ..: column part - 4
    const int i = part - 4;
    const int row = wn * TT::WTN + FN * lr + i;
#pragma unroll
    for (int q = 0; q < 2; ++q) fr.bt[i][q] = __builtin_bit_cast(f32x4, sb[row * 8 + ((2 * lg + q) ^ swz(row))]);
  }
}

// The MFMAs of K index s.
template <class E, bool BNC>
__device__ __forceinline__ void mma_part(const Frags<E>& fr, f32x4 (&acc)[E::FM][E::FN], int s) {
#pragma unroll
  for (int f = 0; f < E::FM; ++f)
#pragma unroll
    for (int i = 0; i < E::FN; ++i) {
      const float bv = BNC ? fr.b[s][i] : fr.bt[i][s >> 2][s & 3];
      acc[f][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr.a[f][s >> 2][s & 3], bv, acc[f][i], 0, 0, 0);
    }
}

// Main loop over K tiles [kt0, kt1). While tile kt's products run from
// registers, tile kt + 1 is read from LDS into a second register set, tile kt + 2
// goes from its staging registers to the LDS stage that tile kt left, and the
// loads of tile kt + 3 are issued; everything sits between MFMAs, and one
// barrier closes the tile. (With each operand read right before its MFMAs and
// the loads waited for at the end of the tile, the waves that share a SIMD came
// to meet in the same gaps and the matrix pipe was 60% busy.) Ends with a
// barrier, so the caller may reuse LDS.
template <class E, bool BNC>
__device__ __forceinline__ void gemm_mainloop(GemmSmem<E>& sm, f32x4 (&acc)[E::FM][E::FN],
                                              const typename E::T* __restrict__ A, int64_t lda,
                                              int M, const typename E::T* __restrict__ B,
                                              int64_t ldb, int N, int K, int m0, int n0, int kt0,
                                              int kt1) {
  static_assert(E::EPC == 4, "this core computes fp32 tiles only");
  const int w = threadIdx.x >> 6;
  const int wm = w >> 1, wn = w & 1;
  TileLoader<E, BNC> ld;
  if (kt0 >= kt1) return;
  ld.setup(A, lda, M, m0, B, ldb, N, n0, kt0);
  Frags<E> f0, f1;
  ld.load(kt0, K);
  ld.store(sm.a[0], sm.b[0], kt0, K);
  if (kt0 + 1 < kt1) {
    ld.load(kt0 + 1, K);
    ld.store(sm.a[1], sm.b[1], kt0 + 1, K);
  }
  __syncthreads();
  if (kt0 + 2 < kt1) ld.load(kt0 + 2, K);
#pragma unroll
  for (int p = 0; p < 8; ++p) read_part<E, BNC>(f0, sm.a[0], sm.b[0], wm, wn, p);
  __syncthreads();
  // tile kt: operands in cur, its LDS stage st free, tile kt + 1 in stage st ^ 1
  auto tile = [&](Frags<E>& cur, Frags<E>& nxt, int kt, int st) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      read_part<E, BNC>(nxt, sm.a[st ^ 1], sm.b[st ^ 1], wm, wn, s);  // past the last tile: unused
      if (s == 5 && kt + 2 < kt1) ld.store(sm.a[st], sm.b[st], kt + 2, K);
      if (s == 6 && kt + 3 < kt1) ld.load(kt + 3, K);
      __builtin_amdgcn_sched_barrier(0);
      mma_part<E, BNC>(cur, acc, s);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the LDS writes and reads of this tile; the global loads stay in flight
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  int kt = kt0;
  for (; kt + 1 < kt1; kt += 2) {
    tile(f0, f1, kt, 0);
    tile(f1, f0, kt + 1, 1);
  }
  if (kt < kt1) tile(f0, f1, kt, 0);
}

template <class E>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[E::FM][E::FN]) {
#pragma unroll
  for (int f = 0; f < E::FM; ++f)
#pragma unroll
    for (int i = 0; i < E::FN; ++i) acc[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Workgroup -> tile mapping. Consecutive workgroup ids are dispatched
// round-robin over the 8 XCDs, each with its own L2. xcd_remap gives every
// XCD a contiguous range of logical tile ids; grouped_tile walks a range in
// groups of `gm` tile rows, so the workgroups resident on one XCD at a time
// cover a few tile rows x a few tile columns and share A rows and B columns
// in that XCD's L2 while they stream through K together.
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_remap(int bid, int nblk) {
  const int xcd = bid % kXcds, slot = bid / kXcds;
  const int per = nblk / kXcds, rem = nblk % kXcds;
  return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

__device__ __forceinline__ void grouped_tile(int id, int ntm, int ntn, int gm, int& tm, int& tn) {
  const int width = gm * ntn;
  const int first = (id / width) * gm;
  const int rows = (ntm - first) < gm ? (ntm - first) : gm;
  const int r = id % width;
  tm = first + r % rows;
  tn = r / rows;
}

// The id that grouped_tile maps to (tm, tn).
__device__ __forceinline__ int grouped_id(int tm, int tn, int ntm, int ntn, int gm) {
  const int first = tm / gm * gm, rows = (ntm - first) < gm ? (ntm - first) : gm;
  return first * ntn + tn * rows + (tm - first);
}

// A uniform value that the compiler may have computed in vector registers (an
// integer division), in a scalar one: the copies' scalar offsets derive from it.
// The empty asm hides that the value is uniform, or the builtin would be folded
// away; the lane read itself is the builtin, so that the compiler sees it and
// places the wait states it needs around it.
__device__ __forceinline__ int to_scalar(int v) {
  asm("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane(v);
}

// Tile of a workgroup: ids [0, nbig) are tiles of the 256 x 256 grid (tm, tn),
// in a launch of their own; the grid's other tiles are taken as four 128 x 128
// quarters each by a second launch, in whose units (tm, tn) then are (a quarter
// may lie outside a ragged matrix). With nbig == 0 the quarters are those of the
// qm x qn grid of 128 x 128 tiles, none outside: empty ones leave at once, but
// the shader engines of an XCD are dealt workgroups in turn, so that with every
// second quarter empty (at most 128 rows) half of the CUs had two of the others to
// run one after the other. Projection, T = 64, d = 4096, V = 32000, 8 splits 68 -> 50 us;
// logits, T = 64, d = 4096, V = 131072 281 -> 193; errh, T = 111, d = 656, d_ff = 16496 78 -> 45.
// Four rows at a time: a range of few tiles shares most panels when it is nearly
// square (full MLP with SGD, T = 92, 408 x 1440 x 3, sixteen rows 153 to 155, four 146 to 149 us).
template <bool QUARTERS>
__device__ __forceinline__ void split_tile(int id, int nbig, int ntm, int ntn, int qm, int qn, int& tm, int& tn) {
  if constexpr (QUARTERS) {
    if (nbig == 0) {
      grouped_tile(id, qm, qn, 4, tm, tn);
    } else {
      grouped_tile(nbig + (id >> 2), ntm, ntn, 8, tm, tn);
      tm = 2 * tm + (id & 1);
      tn = 2 * tn + ((id >> 1) & 1);
    }
  } else {
    grouped_tile(id, ntm, ntn, 8, tm, tn);
  }
}

// Output coordinates of accumulator element [f][i][r] (relative to the tile).
template <class E>
struct AccMap {
  static constexpr int R = 4;     // accumulator elements per (f, i): rows 4 consecutive
  static constexpr int LPR = 16;  // lanes sharing one output row
  int row0, col0;  // tile-relative row of (f=0, r=0), col of i=0
  __device__ __forceinline__ AccMap() {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    row0 = (w >> 1) * Tile<E>::WTM + 4 * (l >> 4);
    col0 = (w & 1) * Tile<E>::WTN + E::FN * (l & 15);
  }
  __device__ __forceinline__ int row(int f, int r) const { return row0 + 16 * f + r; }
  __device__ __forceinline__ int col(int i) const { return col0 + i; }
};

}  // namespace fpo
