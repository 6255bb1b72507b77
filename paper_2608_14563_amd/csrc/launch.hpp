// Host-side launch descriptors shared between the C-ABI layer and the kernel
// translation units. Every pointer is a device pointer; the ABI layer has
// validated sizes and carved the workspace before filling these.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace fpo {

constexpr int kMaxMats = 64;

// Vocabulary chunk c of a plan: the first nwide chunks are cw + cq wide, the
// others cw, and the last one runs to V. Sets its first entry and width.
inline void chunk_span(int64_t V, int nchunk, int64_t cw, int64_t cq, int nwide, int c, int64_t* v0,
                       int64_t* w) {
  *v0 = (int64_t)c * cw + (int64_t)std::min(c, nwide) * cq;
  *w = c == nchunk - 1 ? V - *v0 : cw + (c < nwide ? cq : 0);
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int64_t kCus = 256;  // compute units: one 256 x 256 or 128 x 128 bf16 tile each

// How a bf16 launch of `mats` M x N products over K is cut: its 256 x 256 tiles
// [0, nbig) as such, the others as 128 x 128 quarters (split_tile), by the least
// estimated time. A wave of 256 tiles takes 1.6 us per 64-deep K tile when it is
// full, towards 1.0 when few CUs compete for memory, and 14 us around the K loop;
// a wave of quarters 0.55 us and 7.5 us (measured over K = 256 .. 4096 with 64 to
// 256 tiles and 256 to 768 quarters: 64 tiles over K = 256 / 1024 / 4096 take 18 / 30
// / 79 us, as 256 quarters 11 / 16 / 40 us; 192 tiles 20 / 37 / 117 us, 24 / 46 / 141
// us as quarters). So the last wave goes over when it is a quarter full or less, a
// launch of at most 64 tiles altogether, and a ragged one whose big tiles are
// mostly padding.
// The quarters' copies run up to four K tiles past the end in 32-bit offsets: rows
// longer than 2^21 entries (ld: of the N-contiguous B operand) keep the big tiles.
struct TileSplit {
  int64_t nbig;
  double us;
};
inline TileSplit big_tiles(int64_t M, int64_t N, int64_t K, int64_t mats, int64_t ld = 0) {
  const int64_t n = ceil_div(M, 256) * ceil_div(N, 256) * mats, rem = n % kCus, whole = n - rem;
  const double kt = (double)ceil_div(K, 64);
  auto big = [&](int64_t tiles) { return tiles ? (1.0 + 0.6 * (double)tiles / kCus) * kt + 14.0 : 0.0; };
  auto quarters = [&](int64_t q) { return (double)ceil_div(q, kCus) * (0.55 * kt + 7.5); };
  const double waves = (double)(n / kCus) * big(kCus);
  TileSplit best{n, waves + big(rem)};
  if (ld > ((int64_t)1 << 21)) return best;
  // quarters move more data for the same work: only where they are clearly faster
  const double part = quarters(4 * rem) + 2.0;  // one more launch
  if (whole && part < 0.85 * big(rem)) best = TileSplit{whole, waves + part};
  const double all = quarters(ceil_div(M, 128) * ceil_div(N, 128) * mats);
  if (all < 0.85 * best.us) best = TileSplit{0, all};
  return best;
}

// Workgroups of the quarters launch of `mats` M x N products (split_tile).
inline int quarter_grid(int64_t M, int64_t N, int64_t mats, int64_t nbig) {
  if (nbig == 0) return (int)(ceil_div(M, 128) * ceil_div(N, 128) * mats);
  return (int)(4 * (ceil_div(M, 256) * ceil_div(N, 256) * mats - nbig));
}

// The fused bf16 pseudogradient + update with the gradient clip (fpo_pseudograd):
// how its launches are laid out, from estimates in us (big_tiles; a layer of a batched
// call takes gemm + upd within 5%).
struct FusedCase {
  bool full;              // W1, W2 and W3, or W3 only
  int64_t T, d, d_ff, L;
  bool grad_bf16;         // staged in bf16
  bool adam, state;       // state: the optimizer keeps any
  bool ref;               // against reference gradients too
};
struct FusedPlan {
  bool overlap;           // each matrix's update beside the GEMM launches that follow it;
                          // else all layers' outer products in one launch, all updates in the next
  bool w3_first;          // overlapped full MLP: the W3 launches before the W1/W2 ones
  bool two_per_cu;        // overlapped: two smaller update workgroups a CU instead of one
};
inline FusedPlan plan_fused(const FusedCase& c) {
  FusedPlan p{};
  const double L = (double)c.L;
  const int64_t Tp = ceil_div(c.T, 64) * 64;
  const double kt = (double)ceil_div(c.T, 64);
  const TileSplit w3 = big_tiles(c.d, c.d_ff, c.T, c.L, c.d_ff);
  // a layer's GEMMs, launched for all layers at once (W3) and on their own (gemm1; gemmw
  // with its partly filled waves taken as full ones)
  double gemm = w3.us / L, gemm1 = big_tiles(c.d, c.d_ff, c.T, 1, c.d_ff).us;
  double gemmw = w3.nbig ? ceil_div(ceil_div(c.d, 256) * ceil_div(c.d_ff, 256), kCus) * (1.6 * kt + 14.0)
                         : ceil_div(ceil_div(c.d, 128) * ceil_div(c.d_ff, 128), kCus) * (0.55 * kt + 7.5);
  if (c.full) {
    const double w12 = big_tiles(Tp, c.d_ff, c.d, 1, c.d_ff).us + big_tiles(c.d_ff, c.d, c.T, 2, c.d).us;
    gemm += w12;
    gemm1 += w12;
    gemmw += w12;
  }
  // one matrix's update at 5.8 TB/s: gradient, W read and written, its bf16 copy, state
  // read and written
  const int grad_bytes = c.grad_bf16 ? 2 : 4, bytes = grad_bytes + 10 + (c.adam ? 16 : c.state ? 8 : 0);
  const double numel = (double)c.d * (double)c.d_ff, upd = numel * bytes / 5.8e6;
  // Overlapped or batched. Of L layers' updates (three a layer with the full MLP) all
  // but the last run beside a GEMM, which hides about half of the shorter of the two:
  // less with staged gradients, which have the GEMM write and the update read half the
  // bytes, least for the short update without state. Against that stand
  //  * the pace of one or two workgroups a CU when the update outlasts its GEMM,
  //  * a launch, a hand-over and an event a layer,
  //  * partly filled waves: a batched launch packs all layers' tiles, and beside an
  //    update a partly filled wave takes as long as a full one,
  //  * gradients that fit the 256 MB Infinity Cache: a batched update finds them there
  //    (past it only a layer's update right behind its outer products does).
  // The factors are fitted to 2861 timed (size, optimizer, gradient type) points, T 128
  // to 8192, d 600 to 8192, 1 to 16 layers: the path taken is 0.15% from the best one
  // on average, more than 3% at 1.5% of them. Overlapped / batched, us (T, d x d_ff x
  // L): fp32 gradients: SGD 1024, 4096 x 12288 x 6 1519 / 1805; 700, 3072 x 23040 x 16 5758 /
  // 6504; 1024, 1536 x 8960 x 16 1227 / 1360; 1792, 1840 x 9088 x 3 (288 tiles: 1.1 waves)
  // 447 / 391; 1536, 2048 x 5504 x 4 (172 MB) 336 / 308; AdamW 2048, 2048 x 5504 x 8 785 / 864;
  // 6020, 1472 x 6584 x 5 (156 tiles) 1010 / 813; staged: SGD 512, 4096 x 11008 x 8 1596 /
  // 1734; 1024, x 8 1732 / 1999; AdamW 512, x 8 2374 / 2272; 1536, x 8 2698 / 2831; without
  // state 512, 3744 x 9048 x 5 618 / 594. Full MLP, SGD: 256, 2048 x 5504 x 6 1253 / 1394; 824,
  // 1248 x 5432 x 3 530 / 610; 2048, 1024 x 4096 x 6 1182 / 1028.
  const double per = c.full ? 3.0 : 1.0, beside = per * L - 1.0, m = gemmw / per;
  // (against references the update goes one workgroup a CU, as AdamW's does)
  const double hide = c.full ? 0.60 : !c.grad_bf16 ? 0.47 : c.adam || c.ref ? 0.41 : c.state ? 0.49 : 0.31;
  const double pace = c.full ? 0.06 : 0.14, layer = c.full ? 9.0 : 13.0, waves = c.full ? 0.83 : 0.39;
  const double grads = per * L * numel * grad_bytes, mib = (double)(1 << 20);
  const double cached = (c.full ? 2.5 : 0.56) * std::max(0.0, std::min(1.0, (256.0 - grads / mib) / 200.0));
  const double gain = beside * (hide * std::min(m, upd) - pace * std::max(0.0, upd - m)) -
                      L * (layer + waves * (gemmw - gemm)) - cached * grads / 5.8e6;
  p.overlap = beside > 0.0 && gain > 0.0;
  // Overlapped full MLP, which launches come last. W3 last leaves one update without
  // a GEMM to run beside, W1/W2 last leaves two; but W3 first releases the first
  // update after a quarter of a layer's GEMM time, and where the updates are the
  // longer chain that is what counts (and the two that are left have the whole
  // machine, where beside the short W3 launches they would go at the pace of one
  // workgroup per CU). W3 first / last, us (T, d x d_ff x L, 3 upd / gemm1): AdamW 1024,
  // 2048 x 5504 x 1 (1.08) 333 / 381; 1024, 4096 x 11008 x 2 (1.55) 2029 / 2166;
  // SGD 256, 4096 x 11008 x 1 (2.29) 701 / 781; 2048, 2048 x 5504 x 1 (0.54) 386 / 413;
  // 2048, 4096 x 11008 x 2 (0.66) 2280 / 2270; 3000, 4096 x 11008 x 2 (0.49) 3216 / 3095;
  // AdamW 3000, 3072 x 23040 x 1 (0.70) 3013 / 2863; 4096, 3072 x 23040 x 2 (0.53) 5954 /
  // 5874. Over 344 sizes the order taken is at most 3% slower than the other one.
  p.w3_first = 3 * upd >= 0.75 * (gemm1 - 70.0);
  // Overlapped W3-only SGD: two workgroups of one block each a CU stream faster beside
  // the GEMM, one with two blocks in flight is gentler to it. The GEMM's time goes with
  // T, the update's does not: with few tokens the updates are the longer chain. fp32
  // gradients (twice the bytes written beside them) cross over earlier, and past 2^27
  // entries a matrix, with state, are always better with one. Two / one, us (T, d x
  // d_ff x L): staged, momentum 1024, 4096 x 11008 x 8 1732 / 2035; 2048, x 8 2177 / 2340;
  // 2944, x 8 2677 / 2670; 4096, 3072 x 23040 x 6 3950 / 3929; fp32 700, 4096 x 12288 x 6 1509 /
  // 1568; 1024, x 16 3917 / 4331; 1536, 4096 x 11008 x 8 2128 / 2158; 1800, 3072 x 23040 x 16 7379 /
  // 6956; 1024, 8192 x 28672 x 6 7756 / 7536, without state 5624 / 5946. Three per CU
  // took 2396 where two took 2122. AdamW's workgroup is too large for two
  // (116 registers beside 328 to 348 of 512), and against references (a GEMM
  // workgroup of 336 to 356) two of 76 fit at best by a few registers: 2048, 4096 x
  // 11008 x 6 staged 2147 / 2020, 700, 4096 x 12288 x 6 fp32 1844 / 1798. The full MLP has four
  // GEMMs to three updates: 2048, 4096 x 11008 x 4 4433 / 4391.
  p.two_per_cu = !c.full && !c.adam && !c.ref &&
                 c.T < (c.grad_bf16 ? 3072 : !c.state || c.d * c.d_ff < ((int64_t)1 << 27) ? 1200 : 0);
  return p;
}

struct OeLaunch {
  bool bf16;
  int64_t T, d, V, Vc;  // Vc: widest chunk, rounded up to 256
  int64_t ldp;          // row pitch of the staged p~ (elements, >= Vc)
  int nchunk, nwide;    // chunk layout (chunk_span)
  int64_t cw, cq;
  int nsplit;
  float eps, min_rms;
  const void* h_final;
  const void* gamma;
  const void* W_U;
  const int32_t* targets;
  float* g_tilde;
  void* g_tilde_lp;
  float* g_pre;
  float* lse;
  float* loss;
  int32_t* argmax;
  int32_t* bad_targets;
  // workspace
  void* y;
  void* P;
  float* blk_m;
  float* blk_s;
  int32_t* blk_i;
  float* fout;   // [T] exp(Ref - M_new) of the current chunk
  float* alpha;  // [T] exp(M_old - M_new)
  float* ref;    // [T] staging reference of the current chunk
  float* zt;     // [T] target logit <y_t, W_U[y_t]> (from the stored y)
  float* runM;
  float* runS;
  int32_t* runA;
  float* G;
  void* stream;
};
hipError_t launch_output_error(const OeLaunch& a);

struct PgLaunch {
  bool bf16;
  bool full_mlp;
  int64_t T, d, d_ff, Tp;
  int L;
  int tile;                         // edge of the GEMM tiles: 256 (bf16; see big_tiles) or 64 (fp32)
  float scale;
  const void* g_lp;                 // [T, d]
  const void* a[kMaxMats];          // [T, d_ff]
  const void* W3i[kMaxMats];        // [d, d_ff]
  const void* q[kMaxMats];
  const void* u[kMaxMats];
  const void* x_in[kMaxMats];       // [T, d]
  float* dW3[kMaxMats];
  uint16_t* dW3_bf16[kMaxMats];     // staged bf16 pseudogradient (instead of dW3), or null
  float* dW1[kMaxMats];
  float* dW2[kMaxMats];
  const float* ref[kMaxMats];
  // norm chain: per layer, g_l = VJP_pre(VJP_post(g~ fp32; mlp_out_l, gamma_l); pre_in_l, gamma_pre_l),
  // either factor optional
  bool pffn;
  const float* g_f32;               // [T, d]
  const void* mlp_out[kMaxMats];    // [T, d]
  const void* gamma_pffn[kMaxMats]; // [d]
  float pffn_eps, pffn_min_rms;
  bool pre;
  const void* pre_in[kMaxMats];     // [T, d] cached pre-MLP norm input
  const void* gamma_pre[kMaxMats];  // [d]
  float pre_eps, pre_min_rms;
  double* sumsq;                    // [n_mats] or null
  double* ref_dot;
  double* ref_sumsq;
  float* ref_cos;
  // workspace
  void* gT;                         // [d, Tp] transposed signal
  void* g_row;                      // [T, d] per-layer signal (post-FFN composition, full-MLP)
  float* chain_stats;               // [L, T, 4] per-token norm-chain statistics
  void* dq_T;                       // [d_ff, Tp] full-MLP gate error (transposed)
  void* du_T;                       // [d_ff, Tp] full-MLP up error (transposed)
  double* part;                     // per-tile partials
  bool defer_norms;                 // W3 only, no ref: sumsq is left to launch_update (its tile_part)
  void* stream;
};
hipError_t launch_pseudograd(const PgLaunch& a);
int64_t pseudograd_tiles(int tile, int64_t M, int64_t N);

// Tile partials (three doubles each) of a list of matrices: tile ids run over
// (matrix, tile) in dispatch order; tile g < nbig has slot g, the quarters of a
// later one four slots each.
__host__ __device__ inline int64_t part_slot(int64_t g, int64_t nbig) { return g < nbig ? g : 4 * g - 3 * nbig; }
// The split of launch_pseudograd's W3 outer products (all layers as one list).
int64_t pseudograd_w3_nbig(const PgLaunch& a);

constexpr int kOptAdamW = 1;  // fpo_opt_kind FPO_OPT_ADAMW

struct UpdLaunch {
  int kind;
  double lr, momentum, beta1, beta2, adam_eps, weight_decay, clip_frac;
  int64_t step;
  int n;
  int64_t numel[kMaxMats];
  const void* grad[kMaxMats];       // float32, or bf16 when grad_bf16
  bool grad_bf16;
  float* W[kMaxMats];
  void* W_lp[kMaxMats];
  bool lp_bf16;
  float* s1[kMaxMats];
  float* s2[kMaxMats];
  const double* grad_sumsq;
  double* W_sumsq;
  float* clip_scale;
  double* part;
  // when set, ||dW||^2 comes from these tile partials (one-pass update only): every
  // update block sums its matrix's, the matrix's first one stores it in sumsq_out
  const double* tile_part;
  int64_t ntiles, nbig;
  double* sumsq_out;
  // clip-the-update mode: the clip bounds ||W' - W|| instead of ||dW|| (two
  // passes; dsq: [n] ||delta||^2 scratch)
  bool clip_update;
  double* dsq;
  void* stream;
};
// blocks = false: only the per-matrix reductions (||W'||^2, clip factors) of
// blocks already applied (by the fused pseudogradient launch).
hipError_t launch_update(const UpdLaunch& a, bool blocks = true);
// The update blocks of matrix m of `a` on `stream` (partials at part + blk_base);
// grid > 0: that many workgroups (two_per_cu: twice as many smaller ones, SGD)
// visit the blocks grid-stride.
hipError_t launch_update_blocks(const UpdLaunch& a, int m, int64_t blk_base, void* stream, int grid = 0,
                                bool two_per_cu = false);
// Caller-owned side stream and events of the overlapped path.
struct OverlapLaunch {
  void* side;
  void* ready;
  void* done;
};
// bf16 pseudogradients with the optimizer step overlapped (u: the update of the same
// matrices, grad = the dW outputs, grad_sumsq = a.sumsq), laid out as in `plan`;
// ov: the caller's side stream and events, or null for the library's own.
hipError_t launch_pseudograd_update(const PgLaunch& a, const UpdLaunch& u, const FusedPlan& plan,
                                    const OverlapLaunch* ov);
int64_t update_blocks(int64_t numel);

struct CosLaunch {
  int n;
  int64_t numel[kMaxMats];
  const float* A[kMaxMats];
  const void* B[kMaxMats];
  bool b_bf16;
  double* dot;
  double* sa;
  double* sb;
  float* cos;
  double* part;
  void* stream;
};
hipError_t launch_cosine(const CosLaunch& a);
int64_t cosine_blocks(int64_t numel);

}  // namespace fpo
