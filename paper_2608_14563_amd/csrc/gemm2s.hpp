// bf16 MFMA core for 128 x 128 tiles, for launches whose 256 x 256 tiles
// (gemm2.hpp) would leave most CUs without one. Same operands (A K-contiguous,
// B N-contiguous or K-contiguous), the same 64-deep K stages, LDS-DMA copies and
// chunk swizzle, and v_mfma_f32_32x32x16_bf16; 4 waves.
//
// Such a launch has about one workgroup per CU, so what bounds it is the latency
// of its K loop: a K tile is 512 MFMA cycles a wave, a copy from L2 or HBM takes
// several times that. Hence a ring of four 32 KB stages (three tiles of copies in
// flight) and a second register set: while tile j's products run, tile j + 1 is
// read from LDS and tile j + 4 is copied into the stage that tile j left; one
// barrier a tile.
//
// One wave a SIMD also means that every instruction between two MFMAs (32 cycles)
// counts, hence:
//  * offsets run with the K position (one add a copy), so that the buffer range
//    check covers it: rows past M or N keep an out-of-range offset, K rows of B past
//    K lie past its end, and both read as zero. Chunks past K of a K-contiguous row
//    read whatever follows; the last K tile's registers are cleared there instead
//    of selecting an offset for every copy of every tile.
//  * an N-contiguous B is read with the transposing LDS read (ds_read_b64_tr_b16):
//    in each group of 16 lanes, lane j addresses 4 columns of K row j >> 2 and gets
//    column j of the four rows. No packing; with 4-byte reads, v_perm and a select
//    per copy a K tile took 95 vector instructions a wave and 1490 cycles for 512 of
//    MFMAs, now 63 and 1230.
//
// Layouts: K-contiguous tiles as in gemm2.hpp. An N-contiguous B tile is
// [64 K rows][16 chunks], chunk c of K row k at c ^ 2 (k & 7), so that the four rows
// of a transposing read lie in different banks. The lane owns column 32 i + (l & 31)
// of its wave's 64 in B operand i.
// Accumulator acc[f][i] element r: row 32f + 8*(r>>2) + 4*(l>>5) + (r&3).
#pragma once

#include "gemm2.hpp"

namespace fpo {

struct G2S {
  static constexpr int BM = 128, BN = 128, BK = 64, NST = 4;
  static constexpr int A_CHUNKS = BM * 8, B_CHUNKS = BN * 8;
  static constexpr int STAGE_CHUNKS = A_CHUNKS + B_CHUNKS;  // 32 KB
  static constexpr int COPIES = 8;                          // DMA instructions per wave per stage
};

struct G2SSmem {
  u32x4 s[G2S::NST * G2S::STAGE_CHUNKS];
};

// Wave grid and 32 x 32 blocks per wave: N-contiguous B: 2 x 2 waves of 2 x 2
// blocks. K-contiguous B (the logits): 1 x 4 waves of 4 x 1 blocks, so that a wave
// holds 128 rows (a statistics block) of each of its 32 columns.
template <bool BNC>
struct G2SWave {
  static constexpr int WN = BNC ? 2 : 4, FM = BNC ? 2 : 4, FN = BNC ? 2 : 1;
  static constexpr int WTM = 32 * FM, WTN = 32 * FN;
};

// Output coordinates of acc[f][i] element r relative to the tile.
template <bool BNC>
struct AccMap2S {
  using W = G2SWave<BNC>;
  static constexpr int VEC = 1;
  int row0, colb, lc;
  __device__ __forceinline__ AccMap2S() {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    lc = l & 31;
    row0 = (w / W::WN) * W::WTM + 4 * (l >> 5);
    colb = (w % W::WN) * W::WTN;
  }
  __device__ __forceinline__ int row(int f, int r) const { return row0 + 32 * f + 8 * (r >> 2) + (r & 3); }
  __device__ __forceinline__ int col(int i) const { return colb + 32 * i + lc; }
};

template <bool BNC>
struct Pipe2S {
  using W = G2SWave<BNC>;
  u32x4 ra, rb;
  uint32_t lds;               // LDS byte address of stage 0
  int w, l;
  uint32_t offA[4], offB[4];  // byte offsets of the wave's next copies, or out of range
  uint32_t stepB;             // a K tile further in B
  uint32_t rdA[4], rdB[4];    // LDS offsets in a stage: A by K step; B by K step, or (BNC) by 2 i + half

  __device__ __forceinline__ void setup(const u32x4* smem, const Operand& A, const Operand& B, int M_rem,
                                        int N_rem, int kt0) {
    w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    l = threadIdx.x & 63;
    ra = make_rsrc(A);
    rb = make_rsrc(B);
    lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
    const uint32_t ldA2 = (uint32_t)(A.ld * 2), ldB2 = (uint32_t)(B.ld * 2), k0 = (uint32_t)kt0 * G2S::BK;
    stepB = BNC ? G2S::BK * ldB2 : G2S::BK * 2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 8 * (4 * w + q) + (l >> 3), c = (l & 7) ^ swz8(row);
      offA[q] = row < M_rem ? (uint32_t)row * ldA2 + 16 * c + 2 * k0 : kOOB;
      if constexpr (BNC) {
        const int krow = 4 * (4 * w + q) + (l >> 4), col = 8 * ((l & 15) ^ (2 * (krow & 7)));
        offB[q] = col < N_rem ? (k0 + krow) * ldB2 + 2 * col : kOOB;
      } else {
        offB[q] = row < N_rem ? (uint32_t)row * ldB2 + 16 * c + 2 * k0 : kOOB;
      }
    }
    const int lc = l & 31, wn = w % W::WN, wm = w / W::WN;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int row = wm * W::WTM + lc;
      rdA[h] = (row * 8 + ((2 * h + (l >> 5)) ^ swz8(row))) * 16;
      if constexpr (BNC) {  // h = 2 i + half: K rows 8 (l >> 5) + 4 half + (j >> 2) of a K step, j = l & 15
        const int i = h >> 1, half = h & 1, j = l & 15, krow = 8 * (l >> 5) + 4 * half + (j >> 2);
        const int c = 8 * wn + 4 * i + 2 * ((l >> 4) & 1) + ((j & 3) >> 1);
        rdB[h] = G2S::A_CHUNKS * 16 + krow * 256 + (c ^ (2 * (krow & 7))) * 16 + 8 * (j & 1);
      } else {
        const int rb_ = wn * W::WTN + lc;
        rdB[h] = (G2S::A_CHUNKS + rb_ * 8 + ((2 * h + (l >> 5)) ^ swz8(rb_))) * 16;
      }
    }
  }
  // copy j (0..3: A, 4..7: B) of the next K tile into ring stage st
  __device__ __forceinline__ void issue(int st, int j) {
    const int q = j & 3, inst = 4 * w + q;
    const uint32_t dst = lds + (uint32_t)st * (G2S::STAGE_CHUNKS * 16) + 1024u * inst;
    if (j < 4) {
      dma16(ra, dst, offA[q]);
      offA[q] += G2S::BK * 2;
    } else {
      dma16(rb, dst + G2S::A_CHUNKS * 16, offB[q]);
      offB[q] += stepB;
    }
  }
};

// A wave's operands of one K tile, [K step][block].
template <bool BNC>
struct Frags2S {
  using W = G2SWave<BNC>;
  u32x4 a[4][W::FM];
  u32x4 b[4][W::FN];
};

__device__ __forceinline__ u32x4 lds_read16(uint32_t addr) {
  return *(__attribute__((address_space(3))) const u32x4*)(uintptr_t)addr;
}
__device__ __forceinline__ u32x2 lds_read_tr(uint32_t addr) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(
      u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr));
}

// Part (0..3) of the LDS reads of K step h from the stage at LDS address st.
template <bool BNC>
__device__ __forceinline__ void read_step(Frags2S<BNC>& fr, const Pipe2S<BNC>& p, uint32_t st, int h, int part) {
  using W = G2SWave<BNC>;
  if constexpr (BNC) {  // parts 0, 1: A blocks; each part one transposing read (i, half)
    if (part < W::FM) fr.a[h][part] = lds_read16(st + p.rdA[h] + part * 4096);
    const u32x2 v = lds_read_tr(st + p.rdB[part] + h * 4096);
    u32x4& b = fr.b[h][part >> 1];
    if (part & 1) {
      b.z = v.x;
      b.w = v.y;
    } else {
      b.x = v.x;
      b.y = v.y;
    }
  } else {  // the A blocks, with the first the B block
    fr.a[h][part] = lds_read16(st + p.rdA[h] + part * 4096);
    if (part == 0) fr.b[h][0] = lds_read16(st + p.rdB[h]);
  }
}

// C tile accumulated over K tiles [kt0, kt1); acc starts at zero. Ends with a
// barrier and no copy in flight, so the caller may reuse LDS.
template <bool BNC>
__device__ __forceinline__ void gemm2s_mainloop(G2SSmem& sm, f32x16 (&acc)[G2SWave<BNC>::FM][G2SWave<BNC>::FN],
                                                const Operand& A, const Operand& B, int M_rem, int N_rem, int K,
                                                int kt0, int kt1) {
  using W = G2SWave<BNC>;
  constexpr uint32_t kStage = G2S::STAGE_CHUNKS * 16;
  const int n = kt1 - kt0;
  if (n <= 0) return;
  Pipe2S<BNC> p;
  p.setup(sm.s, A, B, M_rem, N_rem, kt0);
#pragma unroll
  for (int t = 0; t < G2S::NST; ++t)
#pragma unroll
    for (int q = 0; q < G2S::COPIES; ++q) p.issue(t, q);
  Frags2S<BNC> f0, f1;
  wait_vmcnt<3 * G2S::COPIES>();
  stage_barrier();
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q) read_step<BNC>(f0, p, p.lds, h, q);
  auto tile = [&](Frags2S<BNC>& cur, Frags2S<BNC>& nxt, int j) {
    const int k_rem = K - (kt0 + j) * G2S::BK;
    // this wave's reads of tile j are complete and its copies of tile j + 1 have
    // landed (those of the two tiles after it stay in flight); past the barrier
    // that holds for every wave
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    wait_vmcnt<2 * G2S::COPIES>();
    stage_barrier();
    if (k_rem < G2S::BK) {  // the partial last tile
#pragma unroll
      for (int h = 0; h < 4; ++h)
        if (16 * h + 8 * (p.l >> 5) >= k_rem) {
#pragma unroll
          for (int f = 0; f < W::FM; ++f) cur.a[h][f] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int i = 0; i < W::FN; ++i) cur.b[h][i] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    const uint32_t sn = p.lds + (uint32_t)((j + 1) % G2S::NST) * kStage;
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int m = 0; m < 4; ++m) {  // the step's four MFMAs, a part of the reads and copies ahead of each
        read_step<BNC>(nxt, p, sn, h, m);
        if (m & 1) p.issue(j % G2S::NST, 2 * h + (m >> 1));
        __builtin_amdgcn_sched_barrier(0);
        const int f = m / W::FN, i = m % W::FN;
        acc[f][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cur.a[h][f]),
                                                            __builtin_bit_cast(bf16x8, cur.b[h][i]), acc[f][i], 0, 0,
                                                            0);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  int j = 0;
  for (; j + 1 < n; j += 2) {
    tile(f0, f1, j);
    tile(f1, f0, j + 1);
  }
  if (j < n) tile(f0, f1, j);
  wait_vmcnt<0>();
  __syncthreads();
}

template <bool BNC>
__device__ __forceinline__ void zero_acc2s(f32x16 (&acc)[G2SWave<BNC>::FM][G2SWave<BNC>::FN]) {
#pragma unroll
  for (int f = 0; f < G2SWave<BNC>::FM; ++f)
#pragma unroll
    for (int i = 0; i < G2SWave<BNC>::FN; ++i) acc[f][i] = f32x16{};
}

}  // namespace fpo
