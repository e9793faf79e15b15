// Launcher of the product-rule kernel (gemm_linear.h): choice of the tile and of a k-split.
#include "gemm_linear.h"

#include <algorithm>

namespace hf {

// us per 64-deep slab of a block with all CUs busy and operands partly from beyond the L2, with four, five and six operand
// tiles (0: no such kernel).  Measured at 4096 x 768 and 4096 x 3072 of k = 768 and 3072, 512 x 4096 and 512 x 11008 of k = 4096
// and 11008, 4096 x 2048 of k = 2048 and 8192.
struct LinCfg { int bm, bn; double slab_us[3]; };
static const LinCfg kLin[LIN_CFGS] = {{64, 64, {0.5, 0.68, 0.9}},  {64, 128, {0.68, 1.2, 1.5}}, {128, 64, {0.68, 0, 0}}, {128, 96, {1.02, 0, 0}},
                                      {128, 128, {1.17, 1.7, 0}}, {128, 192, {1.62, 2.3, 0}},  {128, 256, {2.4, 0, 0}}};

template <bool TB>
static hipError_t launch_linear_nt4(int cfg, const LinP& p, int nb, int ks, hipStream_t st) {
  switch (cfg) {
    case LIN_64x64: return launch_linear_one<64, 64, 32, 32, 16, 64, 4, 4, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_64x128: return launch_linear_one<64, 128, 32, 32, 16, 64, 3, 3, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_128x64: return launch_linear_one<128, 64, 32, 32, 16, 64, 3, 3, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_128x96: return launch_linear_one<128, 96, 32, 48, 16, 64, 3, 2, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_128x128: return launch_linear_one<128, 128, 64, 32, 16, 64, 3, 2, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_128x192: return launch_linear_one<128, 192, 64, 48, 16, 64, 2, 2, 2, false, TB, 4>(p, nb, ks, st);
    case LIN_128x256: return launch_linear_one<128, 256, 64, 64, 32, 32, 3, 3, 1, false, TB, 4>(p, nb, ks, st);
    default: return hipErrorNotSupported;
  }
}

// A^T B: only the batched products of stored attention come here (one head wide).
static hipError_t launch_linear_tn(int cfg, const LinP& p, int nb, int ks, hipStream_t st) {
  switch (cfg) {
    case LIN_64x64: return launch_linear_one<64, 64, 32, 32, 16, 64, 4, 4, 2, true, false, 4>(p, nb, ks, st);
    case LIN_64x128: return launch_linear_one<64, 128, 32, 32, 16, 64, 3, 3, 2, true, false, 4>(p, nb, ks, st);
    default: return hipErrorNotSupported;
  }
}

// Tile (index of the table) and parts of k for a product with its tangent; -1: two products in one launch are the better choice.
int linear_plan(const Gemm& g, int* parts) {
  const int nb = g.nb1 * g.nb2;
  const int64_t mn = (int64_t)g.M * g.N;
  const int nt = 4 + (g.A[1] != nullptr) + (g.A[2] != nullptr);  // operand tiles
  // Tile and k-split: the shortest estimate, rounds of one block per CU times a block's length (blocks of a round that leaves
  // CUs idle run up to 15 % faster).  A block's length is its slabs, 3 us of start and its results (with addends) at 20 bytes a
  // ns, a CU's share of the memory rate; the parts of a cut k are then added by another launch, 6 us and 4.5 TB/s.  (The 6 us decide
  // for 92 of 690 shapes of 256 to 4096 tokens and widths 256 to 4096: with 3 us those take 5.5 % longer, with 9 us 1.8 %.)  Measured /
  // estimated (us): 512 x 4096 x 11008 64 x 128 whole 164 / 126, 128 x 128 in two parts 140 / 127, 128 x 256 in four 142 / 144;
  // 4096 x 2048 x 2048 128 x 256 98 / 106, 128 x 128 105 / 107; 4096 x 3072 x 768 128 x 192 54 / 55, 128 x 128 60 / 61;
  // 4096 x 768 x 3072 128 x 96 62 / 62; 2048 x 768 x 3072 64 x 128 35 / 40, 128 x 96 in two parts 44 / 47;
  // 999 x 768 x 3072 64 x 64 24 / 29, 128 x 64 34 / 43.
  int cfg = -1;
  int& ks = *parts;
  ks = 1;
  double best = 1e300;
  for (int c = 0; c < LIN_CFGS; ++c) {
    if (kLin[c].slab_us[nt - 4] == 0.) continue;
    if (g.transA && c > LIN_64x128) continue;
    if (g.force_cfg >= 0 && c != g.force_cfg) continue;
    const LinCfg& lc = kLin[c];
    const int64_t tiles = ((int64_t)g.M + lc.bm - 1) / lc.bm * (((int64_t)g.N + lc.bn - 1) / lc.bn) * nb;
    const double slabs = (g.K + 63) / 64 * (g.klimit ? 0.5 : 1.) * lc.slab_us[nt - 4];
    const double out_us = (double)lc.bm * lc.bn * ((g.out_bf16 ? 4 : 8) + (g.Cadd ? 4 : 0) + (g.Cadd_t ? 4 : 0)) / 20e3;
    const int max_ks = g.ws && nb == 1 && !g.klimit && !g.skip_upper && ((uintptr_t)g.ws % 16) == 0 ? std::min(8, g.K / 512) : 1;
    for (int k = 1; k == 1 || (k <= max_ks && 2 * k * mn <= g.ws_elems); ++k) {
      if (g.force_ks > 0 && k != std::min(g.force_ks, max_ks)) continue;
      const double full = (double)(tiles * k / 256), part = (double)(tiles * k % 256) / 256;
      const double blocks = full + (part > 0. ? 0.85 + 0.15 * part : 0.);
      const double us = k == 1 ? blocks * (slabs + 3. + out_us)
                               : blocks * (slabs / k + 3. + lc.bm * lc.bn * 8 / 20e3) + 6. + (double)mn * (8 * k + 8) / 4.5e6;
      if (us < best) { best = us; cfg = c; ks = k; }
    }
  }
  // Many rounds: 256 x 256 tiles of the two products in one launch load as little per product and spend their epilogues on
  // fewer, larger tiles.  Measured (us, this kernel / those): 4096 x 50257 x 768 1117 / 1080, 4096 x 8192 x 2048 346 / 341,
  // 4096 x 6144 x 2048 254 / 273, 4096 x 2048 x 8192 346 / 381, 4096 x 2048 x 2048 100 / 118.  With A_lo both products have two
  // terms, so that rounds come out even, from the first full one on: one round (256 blocks) 2048 x 4096 x 768 60 / 53, x 1024 64 / 65,
  // x 4096 232 / 217, x 11008 615 / 573, 4096 x 2048 x 2048 120 / 117, 512 x 16384 x 1024 68 / 65; two rounds (from 448 blocks) 512 x 28672
  // x 768 124 / 100, x 4096 483 / 410, 1024 x 14336 x 2048 242 / 206, 4096 x 3584 x 512 80 / 73, 512 x 32000 x 4096 491 / 432; three
  // (688) 2048 x 11008 x 4096 604 / 591; unevenly filled rounds lose (512 x 25600 x 4096 425 / 514, 2048 x 6144 x 2048 172 / 243).
  const int64_t pair_blocks = 2 * gemm_tiles256(g.M, g.N);
  if (g.force_cfg < 0 && nb == 1 && !g.klimit && !g.skip_upper && !g.transA && ks == 1 && g.K >= 512 && pair_blocks >= (nt > 4 ? 256 : 1024) &&
      pair_blocks * 100 >= (pair_blocks + 255) / 256 * 256 * 85)
    return -1;
  return cfg;
}

// g.Ct != nullptr, operands on the fast path.  hipErrorNotSupported: the description does not fit, or two single-output
// products are the better choice; the caller then issues those.
hipError_t launch_gemm_linear(const Gemm& g, hipStream_t st) {
  if (!g.At || !g.Bt || g.epi != EPI_NONE || (g.transA && g.transB)) return hipErrorNotSupported;
  LinP p = {};
  p.A = g.A[0]; p.B = g.B[0]; p.At = g.At; p.Bt = g.Bt;
  for (int i = 1; i < 3; ++i) {  // optional low-order terms must be (A_lo, B) and (A, B_lo)
    if (!g.A[i]) continue;
    if (g.B[i] == g.B[0] && g.A[i] != g.A[0] && !p.Alo) p.Alo = g.A[i];
    else if (g.A[i] == g.A[0] && g.B[i] != g.B[0] && !p.Blo) p.Blo = g.B[i];
    else return hipErrorNotSupported;
  }
  if (p.Blo && !p.Alo) return hipErrorNotSupported;
  const int nt = p.Blo ? 6 : p.Alo ? 5 : 4;
  if (g.transA && nt != 4) return hipErrorNotSupported;
  int ks;
  const int cfg = linear_plan(g, &ks);
  if (cfg < 0) return hipErrorNotSupported;
  const int nb = g.nb1 * g.nb2;
  const int64_t mn = (int64_t)g.M * g.N;
  p.C = g.C; p.Ct = g.Ct; p.Clo = g.C_lo; p.Cadd = g.Cadd; p.Cadd_t = g.Cadd_t; p.bias = g.bias; p.bias_t = g.bias_t;
  p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.nb2 = g.nb2; p.divB = g.divB > 0 ? g.divB : 1;
  p.sA1 = g.sA1; p.sA2 = g.sA2; p.sB1 = g.sB1; p.sB2 = g.sB2; p.sC1 = g.sC1; p.sC2 = g.sC2;
  p.alpha = g.alpha; p.out_bf16 = g.out_bf16; p.klimit = g.klimit; p.skip_upper = g.skip_upper;
  {
    const int64_t q = g.out_bf16 ? 8 : 4;
    auto al = [&](const void* x) { return x == nullptr || ((uintptr_t)x % 16) == 0; };
    p.vec = al(g.C) && al(g.Ct) && al(g.C_lo) && al(g.Cadd) && al(g.Cadd_t) && g.ldc % q == 0 && g.sC1 % q == 0 && g.sC2 % q == 0;
  }
  if (ks > 1) {
    p.C = g.ws; p.Ct = g.ws + ks * mn; p.Clo = nullptr; p.Cadd = nullptr; p.Cadd_t = nullptr; p.bias = nullptr; p.bias_t = nullptr;
    p.out_bf16 = 0; p.ldc = g.N; p.sCk = mn; p.vec = g.N % 4 == 0 ? 1 : 0;
  }
  hipError_t e;
  if (nt > 4) e = launch_linear_lo(cfg, nt, g.transB, p, nb, ks, st);
  else if (g.transA) e = launch_linear_tn(cfg, p, nb, ks, st);
  else if (g.transB) e = launch_linear_nt4<true>(cfg, p, nb, ks, st);
  else e = launch_linear_nt4<false>(cfg, p, nb, ks, st);
  if (e != hipSuccess || ks == 1) return e;
  SplitKOut o0, o1;
  o0.part = g.ws; o0.bias_bf16 = (const bf16*)g.bias; o0.Cadd = g.Cadd; o0.C = g.C; o0.C_lo = g.C_lo;
  o1.part = g.ws + ks * mn; o1.bias_f32 = g.bias_t; o1.Cadd = g.Cadd_t; o1.C = g.Ct;
  return launch_splitk_reduce(o0, o1, ks, g.M, g.N, g.ldc, g.out_bf16, st);
}

}  // namespace hf
