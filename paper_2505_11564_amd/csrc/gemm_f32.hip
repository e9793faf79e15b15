// fp32 matrix products on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32): every product of the
// Hessian-vector product when the parameters are fp32.
//
//   C = alpha (A0 op B0 + A1 op B1 + A2 op B2) + bias + bias_t + Cadd        fp32 throughout
//
// What bounds it: the fp32 matrix pipe, 256 flops per clock and CU (157 TFLOP/s), a sixteenth of the
// bf16 one, so operand delivery is never the limit (a 64 x 64 tile reads 128 B of operands per k for
// 8192 flops, 13 % of what L2 delivers).  What costs time instead is a chip that is not full and a
// wave that waits for its operands, and the design is about those two:
//   * a launch takes up to four products (a primal product with its tangent, or the
//     weight-gradient products of a layer), longest blocks first, so their tiles fill the CUs together;
//   * k (over the slabs of all terms) is cut into parts where the tiles alone leave CUs idle.  Each
//     block leaves its partial tile in the workspace and the last block of a tile to arrive adds the parts in
//     their order, so the result does not depend on which one that was, and no second launch is needed;
//   * operands are two slabs ahead in registers and one in LDS (two stages, one barrier per slab).
// LDS layouts: a k-contiguous operand is kept [row][BK + 4], and a lane's 16-byte read holds four k of
// its row; a row-contiguous one is kept [k][R + 8] and read one float at a time.  The k index of a
// matrix instruction is free as long as both operands agree, so step j of a group of eight takes
// k = j and k = 4 + j (lane halves), which is what the 16-byte reads deliver.  Both strides put the
// lanes of a read on different banks.
// Measured: 120 to 125 TFLOP/s from 16000 x 768 x 1024 on, 80 to 105 at 1024 tokens of a 768-wide model (a vector-FMA
// kernel with 64 x 64 tiles before it: 13).
#include "hf_internal.h"
#include "gemm_params.h"

#include <algorithm>

namespace hf {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct F32Group {
  GemmP g[F32_GROUP_MAX];
  int first[F32_GROUP_MAX + 1];  // first block of each product (a multiple of 8); first[n] = number of blocks
  int tiles[F32_GROUP_MAX];      // tiles of one batch entry
  int blocks[F32_GROUP_MAX];     // tiles * batch entries
  int nks[F32_GROUP_MAX];        // parts of k
  int part0[F32_GROUP_MAX];      // first partial tile (of BM x BN floats) of a split product in the workspace
  int cnt0[F32_GROUP_MAX];       // and its first arrival counter
  int n;
  float* part;
  int* counters;  // zero between launches: the last block of a tile clears its own
};

// One operand's slab of R rows x BK: R * BK / 1024 chunks of four elements per thread, along k (KC) or along the rows.
template <int R, bool KC, int BK>
struct F32Tile {
  static constexpr int NI = R * BK / 1024;
  static constexpr int LD = KC ? BK + 4 : R + 8;
  static constexpr int FLOATS = KC ? R * LD : BK * LD;
  static __device__ __forceinline__ int row(int c) { return KC ? c / (BK / 4) : (c % (R / 4)) * 4; }
  static __device__ __forceinline__ int kk(int c) { return KC ? (c % (BK / 4)) * 4 : c / (R / 4); }
  // Element offsets of the thread's chunks from the slab's (block-uniform) base.  Rows beyond the operand are replaced
  // by its last ones (they only feed results that are never stored), so the loads need no guard; without VEC the
  // elements of a chunk are clamped one by one.
  template <bool VEC>
  static __device__ __forceinline__ void offsets(uint32_t (&o)[VEC ? NI : 4 * NI], int64_t ld, int r0, int rmax, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = t + i * 256;
#pragma unroll
      for (int q = 0; q < (VEC ? 1 : 4); ++q) {
        const int r = r0 + row(c) + (KC ? 0 : q), k = kk(c) + (KC ? q : 0);
        const int rc = (VEC && !KC ? min(r, ((rmax - 1) >> 2) << 2) : min(r, rmax - 1)) - r0;
        o[VEC ? i : 4 * i + q] = (uint32_t)(KC ? (int64_t)rc * ld + k : (int64_t)k * ld + rc);
      }
    }
  }
  template <bool VEC>
  static __device__ __forceinline__ void fetch(float4 (&v)[NI], const float* base, const uint32_t (&o)[VEC ? NI : 4 * NI]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if constexpr (VEC) v[i] = *(const float4*)(base + o[i]);
      else v[i] = make_float4(base[o[4 * i]], base[o[4 * i + 1]], base[o[4 * i + 2]], base[o[4 * i + 3]]);
    }
  }
  // The ragged last slab: zeros for k in [kend, k0 + BK); every load is in bounds (clamped) and none is conditional.
  static __device__ __forceinline__ void fetch_tail(float4 (&v)[NI], const float* X, int64_t ld, int r0, int rmax, int k0, int kend, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = t + i * 256;
      float e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = min(r0 + row(c) + (KC ? 0 : q), rmax - 1), k = k0 + kk(c) + (KC ? q : 0), kc = min(k, kend - 1);
        const float x = X[KC ? (int64_t)r * ld + kc : (int64_t)kc * ld + r];
        e[q] = k < kend ? x : 0.f;
      }
      v[i] = make_float4(e[0], e[1], e[2], e[3]);
    }
  }
  static __device__ __forceinline__ void store(const float4 (&v)[NI], float* lds, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = t + i * 256;
      *(float4*)(KC ? lds + row(c) * LD + kk(c) : lds + kk(c) * LD + row(c)) = v[i];
    }
  }
  // k = g*8 + (lane/32)*4 + 0..3 of row `r`
  static __device__ __forceinline__ float4 read(const float* lds, int r, int g, int half) {
    if (KC) return *(const float4*)(lds + r * LD + g * 8 + half * 4);
    const float* p = lds + (g * 8 + half * 4) * LD + r;
    return make_float4(p[0], p[LD], p[2 * LD], p[3 * LD]);
  }
};

// Four waves of WM x WN; where that covers the tile WK times over, each set of waves multiplies its share of a slab's k
// and the sums meet in LDS.  VEC: both operands' rows are 16-byte aligned.
template <int BM, int BN, int BK, int WM, int WN, bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_f32_mfma_kernel(F32Group gg) {
  constexpr int WK = 4 / ((BM / WM) * (BN / WN));
  static_assert((BM / WM) * (BN / WN) * WK == 4 && BK % (16 * WK) == 0, "four waves, pairs of groups of eight k");
  static_assert(WK == 1 || (WK == 4 && WM == 32 && WN == 32), "k shared by all four waves or by none");
  using TileA = F32Tile<BM, !TA, BK>;
  using TileB = F32Tile<BN, TB, BK>;
  constexpr int STAGE = TileA::FLOATS + TileB::FLOATS;
  __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
  __shared__ int last_block;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int col = lane & 31, half = lane >> 5;
  int g = 0;
  while (g + 1 < gg.n && (int)blockIdx.x >= gg.first[g + 1]) ++g;
  const GemmP& p = gg.g[g];
  // blocks go round-robin to the 8 XCDs: XCD x takes the x-th run of consecutive tiles, which share operand rows in
  // its L2 (parts of k outermost: neighbours work on the same k)
  const int nks = gg.nks[g], nblk = gg.blocks[g] * nks;
  int b = blockIdx.x - gg.first[g];
  b = (b & 7) * ((nblk + 7) >> 3) + (b >> 3);
  if (b >= nblk) return;
  const int ks = b / gg.blocks[g], zt = b - ks * gg.blocks[g];
  const int z = zt / gg.tiles[g], tile = zt - z * gg.tiles[g];
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tm, tn;
  {  // bands of 8 tile rows
    const int band = 8 * tiles_n, gi = tile / band, in = tile - gi * band;
    const int rows = min(8, tiles_m - gi * 8);
    tn = in / rows;
    tm = gi * 8 + in - tn * rows;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  if (p.skip_upper && n0 > m0 + BM - 1) return;
  const int z1 = z / p.nb2, z2 = z - z1 * p.nb2;
  const int64_t offA = z1 * p.sA1 + z2 * p.sA2, offB = z1 * p.sB1 + (z2 / p.divB) * p.sB2, offC = z1 * p.sC1 + z2 * p.sC2;
  int kbeg = 0, kend = p.K;
  if (p.klimit == 1) kend = min(p.K, m0 + BM);
  if (p.klimit == 2) kbeg = (m0 / BK) * BK;
  // whole slabs of all terms, dealt to the parts; the ragged remainder of each term goes to the last part
  const int nk = (kend - kbeg) / BK, total = nk * p.nterm;
  const int it0 = (int)((int64_t)total * ks / nks), it1 = (int)((int64_t)total * (ks + 1) / nks);

  const int wm0 = WK > 1 ? 0 : (wave / (BN / WN)) * WM, wn0 = WK > 1 ? 0 : (wave % (BN / WN)) * WN;
  constexpr int TM = WM / 32, TN = WN / 32, NG = BK / 8 / WK;
  const int g0 = WK > 1 ? wave * NG : 0;  // first group of eight k of this wave
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  float4 ra[2][TileA::NI], rb[2][TileB::NI];
  uint32_t oa[VEC ? TileA::NI : 4 * TileA::NI], ob[VEC ? TileB::NI : 4 * TileB::NI];
  TileA::template offsets<VEC>(oa, p.lda, m0, p.M, t);
  TileB::template offsets<VEC>(ob, p.ldb, n0, p.N, t);
  const int64_t stepA = TA ? BK * p.lda : BK, stepB = TB ? BK : BK * p.ldb;
  auto base_a = [&](int term, int k0) { return (const float*)p.A[term] + offA + (TA ? (int64_t)k0 * p.lda + m0 : (int64_t)m0 * p.lda + k0); };
  auto base_b = [&](int term, int k0) { return (const float*)p.B[term] + offB + (TB ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0); };
  int f_term = nk > 0 ? it0 / nk : 0, f_slab = nk > 0 ? it0 - f_term * nk : 0;
  const float *fa = nullptr, *fb = nullptr;
  auto fetch = [&](auto& va, auto& vb) {
    TileA::template fetch<VEC>(va, fa, oa);
    TileB::template fetch<VEC>(vb, fb, ob);
    fa += stepA;
    fb += stepB;
    if (++f_slab == nk && ++f_term < p.nterm) {
      f_slab = 0;
      fa = base_a(f_term, kbeg);
      fb = base_b(f_term, kbeg);
    }
  };
  auto store = [&](const auto& va, const auto& vb, int s) {
    TileA::store(va, smem + s * STAGE, t);
    TileB::store(vb, smem + s * STAGE + TileA::FLOATS, t);
  };
  // The matrix instructions of the slab in stage s; a group's fragments are read while the group before it is multiplied.
  float4 xa[2][TM], xb[2][TN];
  auto read_group = [&](int s, int gk) {
    const float* As = smem + s * STAGE;
    const float* Bs = As + TileA::FLOATS;
#pragma unroll
    for (int i = 0; i < TM; ++i) xa[gk & 1][i] = TileA::read(As, wm0 + i * 32 + col, g0 + gk, half);
#pragma unroll
    for (int j = 0; j < TN; ++j) xb[gk & 1][j] = TileB::read(Bs, wn0 + j * 32 + col, g0 + gk, half);
  };
  auto multiply = [&](int s) {
    read_group(s, 0);
#pragma unroll
    for (int gk = 0; gk < NG; ++gk) {
      if (gk + 1 < NG) read_group(s, gk + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(((const float*)&xa[gk & 1][i])[q], ((const float*)&xb[gk & 1][j])[q],
                                                             acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const int nit = it1 - it0;
  if (nit > 0) {
    fa = base_a(f_term, kbeg + f_slab * BK);
    fb = base_b(f_term, kbeg + f_slab * BK);
    fetch(ra[0], rb[0]);
    if (nit > 1) fetch(ra[1], rb[1]);
    store(ra[0], rb[0], 0);
    // pairs of iterations: slab i is in LDS stage 0, slab i + 1 in (or on its way to) register set 1
    int i = 0;
    for (; i + 4 <= nit; i += 2) {
      __syncthreads();
      fetch(ra[0], rb[0]);
      multiply(0);
      store(ra[1], rb[1], 1);
      __syncthreads();
      fetch(ra[1], rb[1]);
      multiply(1);
      store(ra[0], rb[0], 0);
    }
    // one to three slabs left
    __syncthreads();
    if (i + 2 < nit) fetch(ra[0], rb[0]);
    multiply(0);
    if (i + 1 < nit) {
      store(ra[1], rb[1], 1);
      __syncthreads();
      multiply(1);
      if (i + 2 < nit) {
        store(ra[0], rb[0], 0);
        __syncthreads();
        multiply(0);
      }
    }
  }
  if (kbeg + nk * BK < kend && ks == nks - 1) {
    for (int term = 0; term < p.nterm; ++term) {
      TileA::fetch_tail(ra[0], (const float*)p.A[term] + offA, p.lda, m0, p.M, kbeg + nk * BK, kend, t);
      TileB::fetch_tail(rb[0], (const float*)p.B[term] + offB, p.ldb, n0, p.N, kbeg + nk * BK, kend, t);
      __syncthreads();
      store(ra[0], rb[0], 0);
      __syncthreads();
      multiply(0);
    }
  }

  if constexpr (WK > 1) {  // (k is not cut over blocks as well)
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) smem[(wave * 16 + r) * 64 + lane] = acc[0][0][r];
    __syncthreads();
    const int gn = n0 + col;
    float bsum = 0.f;
    if (gn < p.N) {
      if (p.bias) bsum += ((const float*)p.bias)[gn];
      if (p.bias_t) bsum += p.bias_t[gn];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // wave w finishes rows 8w + 0..7
      const int r = wave * 4 + q, gm = m0 + wave * 8 + half * 4 + q;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += smem[(w * 16 + r) * 64 + lane];
      if (gm >= p.M || gn >= p.N) continue;
      const int64_t ci = offC + (int64_t)gm * p.ldc + gn;
      v = p.alpha * v + bsum;
      if (p.Cadd) v += p.Cadd[ci];
      ((float*)p.C)[ci] = v;
    }
    return;
  }

  if (nks > 1) {
    // partial tiles in accumulator order (thread t of every block of a tile owns the same elements)
    constexpr int NACC = TM * TN * 16;
    float* const base = gg.part + ((int64_t)gg.part0[g] + (int64_t)zt * nks) * (BM * BN);
    float* mine = base + (int64_t)ks * (BM * BN) + t;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          __hip_atomic_store(mine + ((i * TN + j) * 16 + r) * 256, acc[i][j][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // The parts are stored and loaded as agent-scope atomics, which pass the XCDs' L2s on their own: once the stores
    // are acknowledged the counter may follow.  (A fence instead would write back the whole L2 in every block: 580
    // against 130 us for 1024 x 2304 x 768.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
      int* cnt = gg.counters + gg.cnt0[g] + zt;
      const int arrived = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_block = arrived == nks - 1;
      if (arrived == nks - 1) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last_block) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int s = 0; s < nks; ++s) {
      float* src = base + (int64_t)s * (BM * BN) + t;
#pragma unroll
      for (int e = 0; e < NACC; ++e)
        acc[e / (TN * 16)][(e / 16) % TN][e % 16] += __hip_atomic_load(src + e * 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // accumulator tile: column lane & 31, rows 8*(r/4) + 4*(lane/32) + r%4
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int gn = n0 + wn0 + j * 32 + col;
    if (gn >= p.N) continue;
    float bsum = 0.f;
    if (p.bias) bsum += ((const float*)p.bias)[gn];
    if (p.bias_t) bsum += p.bias_t[gn];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int gm = m0 + wm0 + i * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        if (gm >= p.M) continue;
        const int64_t ci = offC + (int64_t)gm * p.ldc + gn;
        float v = p.alpha * acc[i][j][r] + bsum;
        if (p.Cadd) v += p.Cadd[ci];
        ((float*)p.C)[ci] = v;
      }
  }
}

template <int BM, int BN, int BK, int WM, int WN, bool VEC>
static hipError_t launch_f32_vec(const F32Group& gg, int grid, hipStream_t st) {
  const GemmP& p = gg.g[0];
  if (!p.transA && !p.transB) hipLaunchKernelGGL((gemm_f32_mfma_kernel<BM, BN, BK, WM, WN, false, false, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else if (!p.transA) hipLaunchKernelGGL((gemm_f32_mfma_kernel<BM, BN, BK, WM, WN, false, true, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else if (!p.transB) hipLaunchKernelGGL((gemm_f32_mfma_kernel<BM, BN, BK, WM, WN, true, false, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else hipLaunchKernelGGL((gemm_f32_mfma_kernel<BM, BN, BK, WM, WN, true, true, VEC>), dim3(grid), dim3(256), 0, st, gg);
  return hipGetLastError();
}
template <int BM, int BN, int BK, int WM, int WN>
static hipError_t launch_f32_cfg(const F32Group& gg, int grid, bool vec, hipStream_t st) {
  return vec ? launch_f32_vec<BM, BN, BK, WM, WN, true>(gg, grid, st) : launch_f32_vec<BM, BN, BK, WM, WN, false>(gg, grid, st);
}

// Tiles, and the clocks a CU's matrix pipes need per slab as they run (the 64-float deep slabs of the small tile share
// their k over the waves and pay a wait per 512 clocks).
struct F32Cfg { int bm, bn, bk; double slab_clk; };
static const F32Cfg kF32Cfg[] = {{64, 64, 32, 930.}, {128, 64, 32, 1720.}, {32, 32, 64, 665.}};

// Estimated clocks of a launch whose products have cnt[i] blocks of len[i] clocks, longest first.  Up to four blocks of the
// two small tiles are resident per CU (35 and 37 KB of LDS each), dealt to the CUs in turn, and their matrix pipes are
// busy 68, 79, 92 and 99 % of the time with one to four of them: launches of up to four blocks per CU last as
// long as the fullest CU, others as long as the average and about two blocks more.  The 128 x 64 tile (53 to 55 KB) has room
// for two or three: there the busy share of the last ones, and the limit of four, flatter it.
static double f32_estimate(const int64_t* cnt, const double* len, int n) {
  static const double kBusy[] = {1., 0.68, 0.79, 0.92, 0.99};
  int64_t blocks = 0;
  double sum = 0.;
  for (int i = 0; i < n; ++i) { blocks += cnt[i]; sum += (double)cnt[i] * len[i]; }
  if (blocks == 0) return 0.;
  if (blocks > 1024) return sum / 256. / kBusy[4] + 1.9 * sum / (double)blocks;
  double worst = 0.;
  int64_t start = 0;
  for (int i = 0; i <= n; ++i) {  // the first CU that gets one block of product i - 1 less
    const int64_t cu = i == 0 ? 0 : start % 256;
    double load = 0.;
    int held = 0;
    for (int64_t b = cu; b < blocks; b += 256, ++held) {
      int64_t e = 0;
      int k = 0;
      while (b >= (e += cnt[k])) ++k;
      load += len[k];
    }
    worst = std::max(worst, load / kBusy[held]);
    if (i < n) start += cnt[i];
  }
  return worst;
}

// All products have the same transposes and nb batch entries.  ws / counters nullptr: k is never cut.
hipError_t launch_gemm_f32_group(const GemmP* ps, int n, int nb, float* ws, int64_t ws_elems, int* counters, int force_cfg,
                                 int force_ks, hipStream_t st) {
  if (n < 1 || n > F32_GROUP_MAX) return hipErrorInvalidValue;
  for (int i = 1; i < n; ++i)
    if (ps[i].transA != ps[0].transA || ps[i].transB != ps[0].transB) return hipErrorInvalidValue;
  auto tiles_of = [&](const GemmP& p, const F32Cfg& c) {
    return ((int64_t)p.M + c.bm - 1) / c.bm * (((int64_t)p.N + c.bn - 1) / c.bn);
  };
  auto slabs_of = [&](const GemmP& p, const F32Cfg& c) { return (int64_t)p.nterm * ((p.K + c.bk - 1) / c.bk); };
  int order[F32_GROUP_MAX];
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order, order + n, [&](int a, int b) { return (int64_t)ps[a].nterm * ps[a].K > (int64_t)ps[b].nterm * ps[b].K; });
  // Tile and parts of k (the same for all products): the pair with the shortest estimated launch.  (Under klimit the blocks
  // are priced with the whole k, about twice their average: only the tile is chosen there, and all tiles are priced alike.)  A cut costs each block
  // about 2000 clocks (partial tile out; twice that with the twice as large tile) and the launch 8000 (arrivals, sums).
  // Measured (us; uncut 64 x 64, uncut 32 x 32, best and its tile / parts, chosen): primal product and tangent
  // 1024x768x768 45.8 46.5 41.7 64/2 41.7, 1024x2304x768 118 115 106 64/3 106, 1024x3072x768 135 149 135 64/1 137,
  // 1024x768x3072 167 161 141 64/2 148, 512x128x512 25.0 11.1 11.1 32/1 11.1, 512x384x128 10.4 7.1 7.1 32/1 7.1; A^T B
  // 768x768x1024 43.8 37 32.3 64/3 35.3.
  int cfg = 0, parts = 1;
  double best = 1e300;
  for (int ci = 0; ci < 3; ++ci) {
    if (force_cfg >= 0 && ci != force_cfg) continue;
    const F32Cfg& c = kF32Cfg[ci];
    const bool cut = ci != 2 && ws && counters && !ps[0].klimit;
    for (int k = 1; k <= (cut ? 12 : 1); ++k) {
      if (k > 1 && slabs_of(ps[order[0]], c) / k < 4) break;
      int64_t cnt[F32_GROUP_MAX];
      double len[F32_GROUP_MAX];
      for (int i = 0; i < n; ++i) {
        const GemmP& p = ps[order[i]];
        const int64_t slabs = slabs_of(p, c), nks = std::min<int64_t>(k, slabs);
        cnt[i] = tiles_of(p, c) * nb * nks;
        len[i] = c.slab_clk * (double)slabs / (double)nks + (nks > 1 ? (2000. + 60. * (double)nks) * (c.bm * c.bn) / 4096. : 0.);
      }
      const double t = f32_estimate(cnt, len, n) + (k > 1 ? 8000. : 0.);
      if (t < best) { best = t; cfg = ci; parts = k; }
    }
  }
  const F32Cfg& c = kF32Cfg[cfg];
  F32Group gg = {};
  gg.n = n;
  int64_t first = 0, part = 0, cnt = 0;
  for (int k = 0; k < n; ++k) {
    gg.g[k] = ps[order[k]];
    const GemmP& p = gg.g[k];
    const int64_t tiles = tiles_of(p, c), blocks = tiles * nb;
    int64_t nks = 1;
    if (cfg != 2 && ws && counters && !p.klimit) {
      nks = force_ks > 0 ? force_ks : parts;
      nks = std::max<int64_t>(1, std::min<int64_t>(nks, p.nterm * (p.K / c.bk)));
      while (nks > 1 && ((part + blocks * nks) * c.bm * c.bn > ws_elems || cnt + blocks > F32_COUNTERS)) --nks;
    }
    gg.tiles[k] = (int)tiles;
    gg.blocks[k] = (int)blocks;
    gg.nks[k] = (int)nks;
    gg.part0[k] = (int)part;
    gg.cnt0[k] = (int)cnt;
    if (nks > 1) { part += blocks * nks; cnt += blocks; }
    gg.first[k] = (int)first;
    first += (blocks * nks + 7) / 8 * 8;
    if (first > (int64_t)1 << 30) return hipErrorInvalidValue;
  }
  gg.first[n] = (int)first;
  gg.part = ws;
  gg.counters = counters;
  bool vec = true;
  for (int i = 0; i < n; ++i) vec = vec && ps[i].vecA && ps[i].vecB;
  if (cfg == 0) return launch_f32_cfg<64, 64, 32, 32, 32>(gg, (int)first, vec, st);
  if (cfg == 1) return launch_f32_cfg<128, 64, 32, 64, 32>(gg, (int)first, vec, st);
  return launch_f32_cfg<32, 32, 64, 32, 32>(gg, (int)first, vec, st);
}

}  // namespace hf
