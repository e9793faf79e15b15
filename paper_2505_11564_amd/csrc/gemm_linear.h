// Product rule of a linear map on the matrix cores: a primal product and its tangent in one launch,
//
//   C   = alpha (A B + A_lo B + A B_lo) + bias   + Cadd
//   C_t = alpha (A_t B + A B_t)         + bias_t + Cadd_t
//
// (Y = X W next to Y_t = X_t W + X W_t; dX = dY W^T next to dX_t = dY_t W^T + dY W_t^T; the attention products.)  The tiles of
// A and B are loaded once for both results: four operand tiles feed three products.  A_lo, B_lo: optional low-order halves
// of the bf16 primal operands.
//
// What bounds it: operand slabs on their way into LDS.  A block of 128 x 128 with four waves (one a SIMD) turned a 64-deep
// slab over in 1.7 us, of which its matrix instructions take 0.75: with one wave a SIMD every wait for a barrier, for LDS or
// for a slab that comes from beyond the L2 stops the matrix cores.  Hence
//   * eight waves a block, two a SIMD, so that one wave's matrix instructions run while the other waits;
//   * as many slabs in LDS as fit: half of what a block loads comes from beyond the L2 and takes 1 to 2 us, so the activations
//     (A side) are loaded further ahead than the weights, which neighbouring blocks share, where LDS does not hold another
//     slab of both (128 x 96 and 128 x 128: three slabs of A, two of B; 4096 x 768 x 3072 73 -> 64 us, A B^T 69 -> 57);
//   * slabs of 64 (whole 128-byte lines of a k-contiguous row; 32-deep slabs fetch each line in two requests) except where LDS
//     does not hold two of them;
//   * tiles from 64 x 64 to 128 x 256, chosen by the launcher so that the blocks fill the CUs in whole rounds: the wide ones
//     load least per product (128 x 192: 80 KB for 3 x 128 x 192 x 64), the small ones fill the chip where M N is small;
//   * 16 x 16 x 32 matrix instructions where a wave's tile is no multiple of 32 wide: 96 and 192 divide the model widths that
//     128 leaves with a nearly empty last round (4096 x 768: 256 tiles of 128 x 96 instead of 192 of 128 x 128);
//   * the addend of small tiles is loaded during the last slab's products.
// us, cold operands (four waves, 128 x 128 and two or four slabs / this kernel): 4096 x 2304 x 768 58 / 50, 4096 x 768 x 768
// 29 / 24, 4096 x 3072 x 768 70 / 54, 4096 x 768 x 3072 78 / 62, A B^T 77 / 56; 999 x 768 x 768 25 / 11, 999 x 768 x 3072 38 / 24;
// 512 x 11008 x 4096 179 / 121; 4096 x 2048 x 2048 119 / 98.  Of the 62 us of 4096 x 768 x 3072 the matrix instructions alone
// take 27, results and addends 9; reading every slab from the L2 instead of beyond it would still save about 8.
#pragma once
#include "gemm_mfma_common.h"

namespace hf {

struct LinP {
  const void *A, *At, *Alo, *B, *Bt, *Blo;
  void *C, *Ct, *Clo;
  const float *Cadd, *Cadd_t;
  const void* bias;  // bf16
  const float* bias_t;
  int M, N, K;
  int64_t lda, ldb, ldc;
  int nb2, divB;
  int64_t sA1, sA2, sB1, sB2, sC1, sC2;
  int64_t sCk;  // k-split (gridDim.z > 1): elements between the partial results of consecutive parts
  float alpha;
  int out_bf16;
  int klimit, skip_upper;
  int vec;  // C, Ct, Clo, Cadd, Cadd_t rows allow 16-byte accesses
};

// LDS layout of an operand tile of R rows and KT deep; a line is a row (k-contiguous operand) or one k (row-contiguous).
template <int R, bool KC, int KT>
struct LinTile {
  static constexpr int CPL = KC ? KT / 8 : R / 8;
  static constexpr int LINES = KC ? R : KT;
  static __device__ __forceinline__ int swz(int line, int c) {
    if (KC) return c ^ ((line / (128 / KT)) & (KT / 8 - 1));
    const int b = (R * 2) % 256 == 0 ? (line & 3) << 2 : (R * 2) % 256 == 128 ? ((line >> 1) & 1) << 2 : 0;
    return c ^ b ^ (((line >> 3) & 1) << 1);
  }
  static_assert(KC || (R / 8) % 4 == 0, "the rotation stays inside a line");
  static_assert(KC || (R * 2) % 256 != 0 || (R / 8) % 16 == 0, "");
};
template <int R, bool KC, int KT, int MT>
__device__ __forceinline__ uint32_t lin_frag_addr(int rbase, int kk, int lane) {
  using L = LinTile<R, KC, KT>;
  constexpr int KS = MT == 32 ? 16 : 32;
  if (KC) {
    const int r = rbase + (lane & (MT - 1)), c = kk * (KS / 8) + lane / MT;
    return (uint32_t)((r * KT + (L::swz(r, c) << 3)) * 2);
  } else {
    const int i = lane & 15, g = lane >> 4;
    const int kq = (MT == 32 ? (g >> 1) : g) * 8 + (i >> 2);
    const int c = rbase + (MT == 32 ? (g & 1) * 16 : 0) + (i & 3) * 4;
    return (uint32_t)((kq * R + (L::swz(kq, c >> 3) << 3) + (c & 7)) * 2);
  }
}
template <int R, bool KC, int KT, int NTHR>
__device__ __forceinline__ void lin_slab_guarded(const bf16* __restrict__ src, int64_t ld, int r0, int k0, int rmax, int kend,
                                             HF_LDS bf16* lds, int t) {
  using L = LinTile<R, KC, KT>;
  constexpr int TOTAL = R * KT / 8, N = (TOTAL + NTHR - 1) / NTHR;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int P = t + i * NTHR;
    if (TOTAL % NTHR != 0 && P >= TOTAL) break;
    const int line = P / L::CPL, c = (P % L::CPL) * 8;
    uint4 v;
    if (KC) {
      const int64_t gr = min(r0 + line, rmax - 1);
      v = *(const uint4*)(src + gr * ld + (k0 + c < kend ? k0 + c : k0));
    } else {
      const int64_t gk = min(k0 + line, kend - 1);
      v = *(const uint4*)(src + gk * ld + min(r0 + c, ((rmax - 1) >> 3) << 3));
    }
    const int valid = KC ? kend - k0 - c : (k0 + line < kend ? 8 : 0);
    unsigned* w = (unsigned*)&v;
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = valid >= 2 * q + 2 ? w[q] : valid == 2 * q + 1 ? w[q] & 0xffffu : 0u;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    *(HF_LDS u32x4*)(lds + line * (L::CPL * 8) + L::swz(line, c >> 3) * 8) = (u32x4){w[0], w[1], w[2], w[3]};
  }
}
constexpr int lin_min(int a, int b) { return a < b ? a : b; }

template <int MT> struct Acc;
template <> struct Acc<32> { typedef f32x16 T; static constexpr int NR = 16; };
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <> struct Acc<16> { typedef f32x4 T; static constexpr int NR = 4; };
template <int MT>
__device__ __forceinline__ typename Acc<MT>::T mfma(bf16x8 a, bf16x8 b, typename Acc<MT>::T c) {
  if constexpr (MT == 32) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// WM, WN: a wave's part of the tile; MT: edge of its matrix instructions; KT: slab depth; NSA, NSB: slabs of A- and B-side
// operands that LDS holds; FL: the loads of an iteration follow its first 1/FL of matrix instructions.
template <int BM, int BN, int WM, int WN, int MT, int KT, int NSA, int NSB, int FL, bool TA, bool TB, int NT>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, (BM / WM) * (BN / WN) / 4) void linear_kernel(LinP p) {
  constexpr int NW = (BM / WM) * (BN / WN), NTHR = NW * 64;
  constexpr bool AKC = !TA, BKC = TB;
  constexpr int KS = MT == 32 ? 16 : 32, NKK = KT / KS, TM = WM / MT, TN = WN / MT, NR = Acc<MT>::NR;
  constexpr bool hasAlo = NT >= 5, hasBlo = NT >= 6;
  constexpr int NA = hasAlo ? 3 : 2, NB = hasBlo ? 3 : 2;
  constexpr int A_EL = BM * KT, B_EL = BN * KT;
  constexpr int STA = NA * A_EL * 2, STB = NB * B_EL * 2, B0 = NSA * STA;  // bytes of a slab's A and B side; where the B sides start
  static_assert(STA % (NW * 1024) == 0 && STB % (NW * 1024) == 0, "whole load instructions per wave");
  static_assert(NSA >= NSB && NSB >= 2, "pipeline");
  constexpr int NLA = STA / (NW * 1024), NLB = STB / (NW * 1024), NLOAD = NLA + NLB;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  HF_LDS char* const smem_c = (HF_LDS char*)(HF_LDS void*)smem_raw;
  typedef typename Acc<MT>::T acc_t;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int tile = blockIdx.x, z = blockIdx.y;
  {
    const int nt = gridDim.x;
    if ((p.klimit || p.skip_upper) && (gridDim.y & 7) == 0) {
      // batched causal products: XCD c takes whole batch entries (heads) c, c + 8, ..., so that every XCD gets the same mix
      // of long and short tile rows and a head's operands are fetched by one L2 only
      const int L = blockIdx.y * nt + blockIdx.x, r = L >> 3;
      z = (r / nt) * 8 + (L & 7);
      tile = r % nt;
    } else if (nt >= 16) {  // each XCD takes a run of neighbouring tiles, which share operand rows in its L2
      const int per = nt / 8, rem = nt % 8;
      const int x = tile % 8, q = tile / 8;
      tile = x * per + min(x, rem) + q;
    }
  }
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tm, tn;
  {
    constexpr int GROUP_M = 8;
    const int band = GROUP_M * tiles_n;
    const int g = tile / band, first = g * GROUP_M;
    const int gsz = min(GROUP_M, tiles_m - first);
    const int in_band = tile - g * band;
    tm = first + in_band % gsz;
    tn = in_band / gsz;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  if (p.skip_upper && n0 > m0 + BM - 1) return;
  const int z1 = z / p.nb2, z2 = z % p.nb2;
  const int ksp = blockIdx.z, nks = gridDim.z;
  const int64_t offA = z1 * p.sA1 + z2 * p.sA2, offB = z1 * p.sB1 + (z2 / p.divB) * p.sB2,
                offC = z1 * p.sC1 + z2 * p.sC2 + ksp * p.sCk;
  int kbeg = 0, kend = p.K;
  if (p.klimit == 1) kend = min(p.K, m0 + BM);
  if (p.klimit == 2) kbeg = (m0 / 64) * 64;
  const int wm0 = (wave / (BN / WN)) * WM, wn0 = (wave % (BN / WN)) * WN;
  acc_t accp[TM][TN], acct[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < NR; ++r) { accp[i][j][r] = 0.f; acct[i][j][r] = 0.f; }

  const int nfull_all = (kend - kbeg) / KT;
  const int ktail = (ksp == nks - 1) ? (kend - kbeg) - nfull_all * KT : 0;
  const int it0 = (int)((int64_t)nfull_all * ksp / nks), nfull = (int)((int64_t)nfull_all * (ksp + 1) / nks) - it0;

  // this lane's source of each of its wave's load instructions; one step per slab
  const int64_t stepA = (AKC ? (int64_t)KT : (int64_t)KT * p.lda) * 2, stepB = (BKC ? (int64_t)KT : (int64_t)KT * p.ldb) * 2;
  const char *baseA[NLA], *baseB[NLB];  // wave-uniform
  uint32_t voffA[NLA], voffB[NLB];
#pragma unroll
  for (int j = 0; j < NLA; ++j) {
    using L = LinTile<BM, AKC, KT>;
    const int b = (wave * NLA + j) * 1024, ti = b / (A_EL * 2), P = (b - ti * A_EL * 2) / 16 + lane, line = P / L::CPL, c = L::swz(line, P % L::CPL) * 8;
    baseA[j] = (const char*)(ti == 0 ? p.A : ti == 1 ? p.At : p.Alo) + (offA + (AKC ? (int64_t)m0 * p.lda + kbeg : (int64_t)kbeg * p.lda + m0)) * 2 + it0 * stepA;
    voffA[j] = (uint32_t)((AKC ? (int64_t)(min(m0 + line, p.M - 1) - m0) * p.lda + c : (int64_t)line * p.lda + min(m0 + c, ((p.M - 1) >> 3) << 3) - m0) * 2);
  }
#pragma unroll
  for (int j = 0; j < NLB; ++j) {
    using L = LinTile<BN, BKC, KT>;
    const int b = (wave * NLB + j) * 1024, ti = b / (B_EL * 2), P = (b - ti * B_EL * 2) / 16 + lane, line = P / L::CPL, c = L::swz(line, P % L::CPL) * 8;
    baseB[j] = (const char*)(ti == 0 ? p.B : ti == 1 ? p.Bt : p.Blo) + (offB + (BKC ? (int64_t)n0 * p.ldb + kbeg : (int64_t)kbeg * p.ldb + n0)) * 2 + it0 * stepB;
    voffB[j] = (uint32_t)((BKC ? (int64_t)(min(n0 + line, p.N - 1) - n0) * p.ldb + c : (int64_t)line * p.ldb + min(n0 + c, ((p.N - 1) >> 3) << 3) - n0) * 2);
  }
  // load l of the next slab of the B side (l < NLB) and of the A side, into that side's stages sB and sA
  HF_LDS char* const waveA = smem_c + wave * (NLA * 1024);
  HF_LDS char* const waveB = smem_c + B0 + wave * (NLB * 1024);
  auto issue_one = [&](int sA, int sB, auto l_c) {
    constexpr int l = decltype(l_c)::value;
    if constexpr (l < NLB) {
      __builtin_amdgcn_global_load_lds((const void*)(baseB[l] + voffB[l]), (HF_LDS void*)(waveB + sB * STB + l * 1024), 16, 0, 0);
      baseB[l] += stepB;
    } else {
      constexpr int a = l - NLB;
      __builtin_amdgcn_global_load_lds((const void*)(baseA[a] + voffA[a]), (HF_LDS void*)(waveA + sA * STA + a * 1024), 16, 0, 0);
      baseA[a] += stepA;
    }
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem_c;
  // k-contiguous tiles: rows MT apart lie a constant apart (the rotation repeats every 16 rows) and the k-steps differ in
  // one bit field of the address; row-contiguous ones: k-steps lie a constant apart, row blocks need an address each
  constexpr int NAA = AKC ? 1 : TM, NAB = BKC ? 1 : TN;
  uint32_t adA[NAA], adB[NAB];
#pragma unroll
  for (int i = 0; i < NAA; ++i) adA[i] = lds0 + lin_frag_addr<BM, AKC, KT, MT>(wm0 + i * MT, 0, lane);
#pragma unroll
  for (int j = 0; j < NAB; ++j) adB[j] = lds0 + B0 + lin_frag_addr<BN, BKC, KT, MT>(wn0 + j * MT, 0, lane);

  static_assert(NKK % 2 == 0, "two register sets alternate by k-step");
  constexpr int NFR = NA * TM + NB * TN, MQ = TM * TN * (NT - 1);
  static_assert(NLOAD <= NKK * MQ, "at most one load per matrix instruction");
  Frag<AKC> fa[2][NA][TM];
  Frag<BKC> fb[2][NB][TN];
  // fragment f of a k-step: A, B, A_t, B_t, A_lo, B_lo
  auto request_one = [&](auto sa_c, auto sb_c, auto kk_c, auto f_c, uint32_t dynA, uint32_t dynB) {
    constexpr int kk = decltype(kk_c)::value, f = decltype(f_c)::value, c = kk & 1;
    constexpr int pairf = TM + TN, pr = f / pairf < 2 ? f / pairf : 2, w = f - pr * pairf;
    constexpr bool isA = w < TM;
    if constexpr (isA) {
      constexpr int off = decltype(sa_c)::value * STA + pr * A_EL * 2 + (AKC ? w * MT * KT * 2 : kk * KS * BM * 2);
      fa[c][pr][w].template read<off, 4 * BM * 2>((adA[AKC ? 0 : w] ^ (AKC ? kk * KS * 2 : 0)) + dynA);
    } else {
      constexpr int j = w - TM, off = decltype(sb_c)::value * STB + pr * B_EL * 2 + (BKC ? j * MT * KT * 2 : kk * KS * BN * 2);
      fb[c][pr][j].template read<off, 4 * BN * 2>((adB[BKC ? 0 : j] ^ (BKC ? kk * KS * 2 : 0)) + dynB);
    }
  };
  auto landed = [&](auto kk_c) {
    constexpr int c = decltype(kk_c)::value & 1;
    __builtin_amdgcn_sched_barrier(0);
    lds_wait_all();
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[c][a][i].tie();
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[c][b][j].tie();
  };
  // The matrix instructions of k-step kk, in phase PH (0 .. NKK - 1) of a pipeline iteration.  Everything else the wave has to
  // issue is dealt out between them: with REQ the fragment reads of k-step rk of stages (sa, sb), with ISSUE = 2 the loads of
  // the next slabs of both sides into stages (lA, lB), with ISSUE = 1 of the B side only.
  auto mfmas = [&](auto kk_c, auto ph_c, auto issue_c, int lA, int lB, auto req_c, auto sa_c, auto sb_c, auto rk_c, uint32_t dynA, uint32_t dynB) {
    constexpr int c = decltype(kk_c)::value & 1, PH = decltype(ph_c)::value, ISSUE = decltype(issue_c)::value;
    constexpr bool REQ = decltype(req_c)::value;
    static_for<MQ>([&](auto q_c) {
      constexpr int q = decltype(q_c)::value, ty = q / (TM * TN), i = (q % (TM * TN)) / TN, j = q % TN;
      constexpr int ai = ty == 1 ? 1 : ty == 3 ? 2 : 0, bi = ty == 2 ? 1 : ty == 4 ? 2 : 0;
      if constexpr (ty == 1 || ty == 2) acct[i][j] = mfma<MT>(fa[c][ai][i].get(), fb[c][bi][j].get(), acct[i][j]);
      else accp[i][j] = mfma<MT>(fa[c][ai][i].get(), fb[c][bi][j].get(), accp[i][j]);
      if constexpr (REQ) {
        static_for<NFR>([&](auto f_c) {
          constexpr int f = decltype(f_c)::value;
          if constexpr ((f * MQ) / (2 * NFR) == q) request_one(sa_c, sb_c, rk_c, f_c, dynA, dynB);
        });
      }
      constexpr int gq = PH * MQ + q;
      constexpr int l0 = lin_min(gq * NLOAD * FL / (NKK * MQ), NLOAD), l1 = lin_min((gq + 1) * NLOAD * FL / (NKK * MQ), NLOAD);
      static_assert(l1 - l0 <= 1, "at most one load per matrix instruction");
      if constexpr (l1 > l0 && (ISSUE == 2 || (ISSUE == 1 && l0 < NLB))) issue_one(lA, lB, std::integral_constant<int, l0>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using IL = std::integral_constant<int, NKK - 1>;
  auto ksteps = [&](auto sa_c, auto sb_c, auto issue_c, int lA, int lB, uint32_t dynA, uint32_t dynB) {
    static_for<NKK - 1>([&](auto k_c) {
      using K1 = std::integral_constant<int, decltype(k_c)::value + 1>;
      landed(k_c);
      mfmas(k_c, K1{}, issue_c, lA, lB, std::true_type{}, sa_c, sb_c, K1{}, dynA, dynB);
    });
    landed(IL{});
  };
  // One pipeline iteration, entered after the barrier that publishes the slab in stages (sa, sb): last k-step of the slab
  // before it, whose fragments are in registers (so that its stages are free), then this slab's k-steps but the last.
  auto iteration = [&](auto sa_c, auto sb_c, auto issue_c, int lA, int lB, uint32_t dynA, uint32_t dynB) {
    mfmas(IL{}, I0{}, issue_c, lA, lB, std::true_type{}, sa_c, sb_c, I0{}, dynA, dynB);
    ksteps(sa_c, sb_c, issue_c, lA, lB, dynA, dynB);
  };
  auto last_kstep = [&]() { mfmas(IL{}, I0{}, I0{}, 0, 0, std::false_type{}, I0{}, I0{}, I0{}, 0u, 0u); };
  auto first_slab = [&]() {
    static_for<NFR>([&](auto f_c) { request_one(I0{}, I0{}, I0{}, f_c, 0u, 0u); });
    ksteps(I0{}, I0{}, I0{}, 0, 0, 0u, 0u);
  };

  // epilogue geometry: passes of 32 rows, 8 consecutive columns per lane
  constexpr int CPRW = WN / 8, EPP = 32 * CPRW / 64, NPASS = (WM / 32) * EPP;
  static_assert((32 * CPRW) % 64 == 0 && WM % 32 == 0, "whole epilogue passes");
  constexpr bool PREF = NPASS <= 4 && BM * BN <= 128 * 96;
  float4 pre[PREF ? NPASS : 1][4];
  const bool pref = PREF && p.Cadd && p.Cadd_t && p.vec;
  auto prefetch_add = [&]() {
    if constexpr (PREF) {
      if (pref) {
#pragma unroll
        for (int e = 0; e < NPASS; ++e) {
          const int ch = (e % EPP) * 64 + lane, gm = m0 + wm0 + (e / EPP) * 32 + ch / CPRW, gn = n0 + wn0 + ch % CPRW * 8;
          if (gm < p.M && gn + 8 <= p.N) {
            const int64_t ci = offC + (int64_t)gm * p.ldc + gn;
            pre[e][0] = *(const float4*)(p.Cadd + ci); pre[e][1] = *(const float4*)(p.Cadd + ci + 4);
            pre[e][2] = *(const float4*)(p.Cadd_t + ci); pre[e][3] = *(const float4*)(p.Cadd_t + ci + 4);
          }
        }
      }
    }
  };

  // Loads leave slab by slab, the B side of a slab before its A side.  Iteration j multiplies slab j's last and slab j + 1's
  // other k-steps and loads slab j + NSB of the B side and j + NSA of the A side; at its start everything up to slab j + 1 has
  // to have landed, which leaves what was issued after that in flight (vmcnt counts in order).
#pragma unroll
  for (int s = 0; s < NSA; ++s) {
    if (s < NSB && s < nfull) static_for<NLB>([&](auto l_c) { issue_one(s, s, l_c); });
    if (s < nfull) static_for<NLA>([&](auto l_c) { issue_one(s, s, std::integral_constant<int, NLB + decltype(l_c)::value>{}); });
  }
  if (nfull > 0) {
    constexpr int STEADY = NSA == NSB ? (NSB - 2) * NLOAD : (NSB - 1) * NLA + (NSB - 2) * NLB;
    constexpr int UNROLL = NSA == NSB ? NSA : NSA * NSB;  // stages as compile-time constants
    static_assert(STEADY + NLOAD < 64, "vmcnt");
    if (nfull >= NSA) HF_WAIT_VMCNT((NSA - 1) * NLA + (NSB - 1) * NLB);
    else HF_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    first_slab();
    const int n_issue = max(0, nfull - NSA);
    for (int j0 = 0; j0 < n_issue; j0 += UNROLL) {
      static_for<UNROLL>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        if (j0 + s < n_issue) {
          HF_WAIT_VMCNT(STEADY);
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
          iteration(std::integral_constant<int, (s + 1) % NSA>{}, std::integral_constant<int, (s + 1) % NSB>{}, I2{}, s % NSA, s % NSB, 0u, 0u);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    }
    // the last slabs: B side only, then no more loads (stages as run-time offsets)
    auto rest = [&](int j, auto issue_c) {
      iteration(I0{}, I0{}, issue_c, 0, j % NSB, (uint32_t)(((j + 1) % NSA) * STA), (uint32_t)(((j + 1) % NSB) * STB));
    };
    int j = n_issue;
    if constexpr (NSA > NSB) {
      for (; j + NSB < nfull; ++j) {
        if (j == nfull - NSA) HF_WAIT_VMCNT(STEADY);
        else HF_WAIT_VMCNT(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        rest(j, I1{});
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (; j + 1 < nfull; ++j) {
      if (NSB > 3 && NSA == NSB && j + 3 < nfull) HF_WAIT_VMCNT(2 * NLOAD);
      else if (NSB > 2 && NSA == NSB && j + 2 < nfull) HF_WAIT_VMCNT(NLOAD);
      else HF_WAIT_VMCNT(0);
      __builtin_amdgcn_s_barrier();
      if (j + 2 >= nfull && ktail == 0) prefetch_add();
      __builtin_amdgcn_sched_barrier(0);
      rest(j, I0{});
      __builtin_amdgcn_sched_barrier(0);
    }
    last_kstep();
  }
  if (ktail > 0 || nfull < 2) {
    prefetch_add();
    if (ktail > 0) {
      const int k0 = kbeg + nfull_all * KT;
      __syncthreads();
      HF_LDS bf16* const sm = (HF_LDS bf16*)smem_c;
      static_for<NA>([&](auto a) {
        constexpr int ai = decltype(a)::value;
        lin_slab_guarded<BM, AKC, KT, NTHR>((const bf16*)(ai == 0 ? p.A : ai == 1 ? p.At : p.Alo) + offA, p.lda, m0, k0, p.M, kend, sm + ai * A_EL, t);
      });
      static_for<NB>([&](auto b) {
        constexpr int bi = decltype(b)::value;
        lin_slab_guarded<BN, BKC, KT, NTHR>((const bf16*)(bi == 0 ? p.B : bi == 1 ? p.Bt : p.Blo) + offB, p.ldb, n0, k0, p.N, kend, sm + B0 / 2 + bi * B_EL, t);
      });
      __syncthreads();
      first_slab();
      last_kstep();
    }
  }

  // ---- epilogue
  constexpr int LDW = WN + 4;
  HF_LDS float* const stg = (HF_LDS float*)smem_c + wave * (32 * LDW);
  __syncthreads();  // every wave is done reading operand tiles
  auto write_out = [&](auto tangent_c) {
    constexpr bool TG = decltype(tangent_c)::value;
    const float* const add = TG ? p.Cadd_t : p.Cadd;
    void* const X = TG ? p.Ct : p.C;
    void* const Xlo = TG ? nullptr : p.Clo;
    float bs[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int gn = n0 + wn0 + j * MT + (lane & (MT - 1));
      bs[j] = 0.f;
      if (gn < p.N) {
        if (TG && p.bias_t) bs[j] = p.bias_t[gn];
        if (!TG && p.bias) bs[j] = (float)((const bf16*)p.bias)[gn];
      }
    }
#pragma unroll
    for (int h = 0; h < WM / 32; ++h) {
#pragma unroll
      for (int ii = 0; ii < 32 / MT; ++ii)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            const int i = h * (32 / MT) + ii;
            const int row = MT == 32 ? (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3) : ii * 16 + (lane >> 4) * 4 + r;
            stg[row * LDW + j * MT + (lane & (MT - 1))] = p.alpha * (TG ? acct[i][j][r] : accp[i][j][r]) + bs[j];
          }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int ps = 0; ps < EPP; ++ps) {
        const int ch = ps * 64 + lane, row = ch / CPRW, cc = ch % CPRW * 8;
        const int gm = m0 + wm0 + h * 32 + row, gn = n0 + wn0 + cc;
        typedef float f32x4_t __attribute__((ext_vector_type(4)));
        const f32x4_t a0 = *(const HF_LDS f32x4_t*)(stg + row * LDW + cc), a1 = *(const HF_LDS f32x4_t*)(stg + row * LDW + cc + 4);
        float v[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
        if (gm >= p.M || gn >= p.N) continue;
        const int64_t ci = offC + (int64_t)gm * p.ldc + gn;
        if (p.vec && gn + 8 <= p.N) {
          if (add) {
            float4 c0, c1;
            if (PREF && pref) { c0 = pre[PREF ? h * EPP + ps : 0][TG ? 2 : 0]; c1 = pre[PREF ? h * EPP + ps : 0][TG ? 3 : 1]; }
            else { c0 = *(const float4*)(add + ci); c1 = *(const float4*)(add + ci + 4); }
            v[0] += c0.x; v[1] += c0.y; v[2] += c0.z; v[3] += c0.w; v[4] += c1.x; v[5] += c1.y; v[6] += c1.z; v[7] += c1.w;
          }
          if (p.out_bf16) {
            bf16 hi[8], lo[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) { hi[q] = (bf16)v[q]; lo[q] = (bf16)(v[q] - (float)hi[q]); }
            *(uint4*)((bf16*)X + ci) = *(const uint4*)hi;
            if (Xlo) *(uint4*)((bf16*)Xlo + ci) = *(const uint4*)lo;
          } else {
            *(float4*)((float*)X + ci) = make_float4(v[0], v[1], v[2], v[3]);
            *(float4*)((float*)X + ci + 4) = make_float4(v[4], v[5], v[6], v[7]);
          }
        } else {
          for (int q = 0; q < 8; ++q) {
            if (gn + q >= p.N) break;
            float x = v[q];
            if (add) x += add[ci + q];
            if (p.out_bf16) {
              const bf16 hi = (bf16)x;
              ((bf16*)X)[ci + q] = hi;
              if (Xlo) ((bf16*)Xlo)[ci + q] = (bf16)(x - (float)hi);
            } else {
              ((float*)X)[ci + q] = x;
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  write_out(std::false_type{});
  write_out(std::true_type{});
}

template <int BM, int BN, int WM, int WN, int MT, int KT, int NSA, int NSB, int FL, bool TA, bool TB, int NT>
static hipError_t launch_linear_one(const LinP& p, int nb, int ks, hipStream_t st) {
  static OncePerDevice once;
  auto kern = linear_kernel<BM, BN, WM, WN, MT, KT, NSA, NSB, FL, TA, TB, NT>;
  constexpr int NW = (BM / WM) * (BN / WN);
  constexpr int smem_pipe = (NSA * (NT >= 5 ? 3 : 2) * BM + NSB * (NT >= 6 ? 3 : 2) * BN) * KT * 2, smem_epi = NW * 32 * (WN + 4) * 4;
  constexpr int smem = smem_pipe > smem_epi ? smem_pipe : smem_epi;
  static_assert(smem <= 160 * 1024, "LDS");
  if (hipError_t e = once.lds_limit((const void*)kern, smem); e != hipSuccess) return e;
  const dim3 grid((unsigned)((int64_t)((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN)), (unsigned)nb, (unsigned)ks);
  hipLaunchKernelGGL(kern, grid, dim3(NW * 64), smem, st, p);
  return hipGetLastError();
}

// Tiles (index of the table of the launcher).
enum { LIN_64x64, LIN_64x128, LIN_128x64, LIN_128x96, LIN_128x128, LIN_128x192, LIN_128x256, LIN_CFGS };

// Products with low-order terms: nt = 5 or 6 operand tiles.
hipError_t launch_linear_lo(int cfg, int nt, int transB, const LinP& p, int nb, int ks, hipStream_t st);

}  // namespace hf
