// fp32 matrix products on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32): every product of the
// Hessian-vector product when the parameters are fp32.
//
//   C = alpha (A0 op B0 + A1 op B1 + A2 op B2) + bias + bias_t + Cadd        fp32 throughout
//
// The fp32 matrix pipe does 256 flops per clock and CU (157 TFLOP/s), a sixteenth of the bf16 one, so the larger tiles take their
// operands apart into three bf16 numbers each and multiply those (gemm_f32_split_kernel below); products too small for
// that to matter stay with the fp32 instructions (gemm_f32_mfma_kernel, 32 x 32 tiles), where the time goes into waits.  Both:
//   * a launch takes up to four products (a primal product with its tangent, or the weight-gradient products of a layer), longest
//     blocks first, so their tiles fill the CUs together;
//   * operands are two slabs ahead in registers and one in LDS (two stages, one barrier per slab).
// The split kernel also cuts k (over the slabs of all terms) into parts where the tiles alone leave CUs idle.  Each block leaves its
// partial tile in the workspace and the last block of a tile to arrive adds the parts in their order, so the result does
// not depend on which one that was, and no second launch is needed.
// fp32 LDS layouts: a k-contiguous operand is kept [row][BK + 4], and a lane's 16-byte read holds four k of its row; a
// row-contiguous one is kept [k][R + 8] and read one float at a time.  The k index of a matrix instruction is free as long as
// both operands agree, so step j of a group of eight takes k = j and k = 4 + j (lane halves), which is what the 16-byte reads
// deliver.  Both strides put the lanes of a read on different banks.
#include "gemm_linear.h"

#include <algorithm>

namespace hf {

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
template <int R, bool KC, int BK, int NTHR>
struct F32Tile {
  static constexpr int NI = R * BK / (4 * NTHR);
  static constexpr int LD = KC ? BK + 4 : R + 8;
  static constexpr int FLOATS = KC ? R * LD : BK * LD;
  static __device__ __forceinline__ int row(int c) { return KC ? c / (BK / 4) : (c % (R / 4)) * 4; }
  static __device__ __forceinline__ int kk(int c) { return KC ? (c % (BK / 4)) * 4 : c / (R / 4); }
  // Element offsets of the thread's chunks from the slab's (block-uniform) base.  Rows beyond the operand are replaced
  // by its last ones (they only feed results that are never stored), so the loads need no guard; without VEC the
  // elements of a chunk along the rows are clamped one by one.
  template <bool VEC> static constexpr int PER = VEC || KC ? 1 : 4;  // offsets a chunk
  template <bool VEC>
  static __device__ __forceinline__ void offsets(uint32_t (&o)[PER<VEC> * NI], int64_t ld, int r0, int rmax, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = t + i * NTHR;
#pragma unroll
      for (int q = 0; q < PER<VEC>; ++q) {
        const int r = r0 + row(c) + q;
        const int rc = (VEC && !KC ? min(r, ((rmax - 1) >> 2) << 2) : min(r, rmax - 1)) - r0;
        o[PER<VEC> * i + q] = (uint32_t)(KC ? (int64_t)rc * ld + kk(c) : (int64_t)kk(c) * ld + rc);
      }
    }
  }
  template <bool VEC>
  static __device__ __forceinline__ float4 fetch_one(const float* base, const uint32_t* o, int i) {
    if constexpr (VEC) return *(const float4*)(base + o[i]);
    else if constexpr (KC) {
      const float* const p = base + o[i];
      return make_float4(p[0], p[1], p[2], p[3]);
    }
    else return make_float4(base[o[4 * i]], base[o[4 * i + 1]], base[o[4 * i + 2]], base[o[4 * i + 3]]);
  }
  template <bool VEC>
  static __device__ __forceinline__ void fetch(float4 (&v)[NI], const float* base, const uint32_t (&o)[PER<VEC> * NI]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) v[i] = fetch_one<VEC>(base, o, i);
  }
  // The ragged last slab: zeros for k in [kend, k0 + BK); every load is in bounds (clamped) and none is conditional.
  static __device__ __forceinline__ void fetch_tail(float4 (&v)[NI], const float* X, int64_t ld, int r0, int rmax, int k0, int kend, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = t + i * NTHR;
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
      const int c = t + i * NTHR;
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

// 32 x 32 tiles: each of the four waves multiplies its share of a slab's k for the whole tile, and the sums meet in LDS.
// VEC: both operands' rows are 16-byte aligned.
template <bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_f32_mfma_kernel(F32Group gg) {
  constexpr int BM = 32, BN = 32, BK = 64, WAVES = 4;
  using TileA = F32Tile<BM, !TA, BK, 256>;
  using TileB = F32Tile<BN, TB, BK, 256>;
  constexpr int STAGE = TileA::FLOATS + TileB::FLOATS;
  __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int col = lane & 31, half = lane >> 5;
  int g = 0;
  while (g + 1 < gg.n && (int)blockIdx.x >= gg.first[g + 1]) ++g;
  const GemmP& p = gg.g[g];
  // blocks go round-robin to the 8 XCDs: XCD x takes the x-th run of consecutive tiles, which share operand rows in its L2
  const int nblk = gg.blocks[g];
  int b = blockIdx.x - gg.first[g];
  b = (b & 7) * ((nblk + 7) >> 3) + (b >> 3);
  if (b >= nblk) return;
  const int z = b / gg.tiles[g], tile = b - z * gg.tiles[g];
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
  const int nk = (kend - kbeg) / BK, nit = nk * p.nterm;  // whole slabs of a term and of all

  constexpr int NG = BK / 8 / WAVES;
  const int g0 = wave * NG;  // first group of eight k of this wave
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  float4 ra[2][TileA::NI], rb[2][TileB::NI];
  uint32_t oa[TileA::template PER<VEC> * TileA::NI], ob[TileB::template PER<VEC> * TileB::NI];
  TileA::template offsets<VEC>(oa, p.lda, m0, p.M, t);
  TileB::template offsets<VEC>(ob, p.ldb, n0, p.N, t);
  const int64_t stepA = TA ? BK * p.lda : BK, stepB = TB ? BK : BK * p.ldb;
  auto base_a = [&](int term, int k0) { return (const float*)p.A[term] + offA + (TA ? (int64_t)k0 * p.lda + m0 : (int64_t)m0 * p.lda + k0); };
  auto base_b = [&](int term, int k0) { return (const float*)p.B[term] + offB + (TB ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0); };
  int f_term = 0, f_slab = 0;
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
  float4 xa[2], xb[2];
  auto read_group = [&](int s, int gk) {
    const float* As = smem + s * STAGE;
    const float* Bs = As + TileA::FLOATS;
    xa[gk & 1] = TileA::read(As, col, g0 + gk, half);
    xb[gk & 1] = TileB::read(Bs, col, g0 + gk, half);
  };
  auto multiply = [&](int s) {
    read_group(s, 0);
#pragma unroll
    for (int gk = 0; gk < NG; ++gk) {
      if (gk + 1 < NG) read_group(s, gk + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(((const float*)&xa[gk & 1])[q], ((const float*)&xb[gk & 1])[q], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (nit > 0) {
    fa = base_a(0, kbeg);
    fb = base_b(0, kbeg);
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
  if (kbeg + nk * BK < kend) {
    for (int term = 0; term < p.nterm; ++term) {
      TileA::fetch_tail(ra[0], (const float*)p.A[term] + offA, p.lda, m0, p.M, kbeg + nk * BK, kend, t);
      TileB::fetch_tail(rb[0], (const float*)p.B[term] + offB, p.ldb, n0, p.N, kbeg + nk * BK, kend, t);
      __syncthreads();
      store(ra[0], rb[0], 0);
      __syncthreads();
      multiply(0);
    }
  }

  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) smem[(wave * 16 + r) * 64 + lane] = acc[r];
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
    for (int w = 0; w < WAVES; ++w) v += smem[(w * 16 + r) * 64 + lane];
    if (gm >= p.M || gn >= p.N) continue;
    const int64_t ci = offC + (int64_t)gm * p.ldc + gn;
    v = p.alpha * v + bsum;
    if (p.Cadd) v += p.Cadd[ci];
    ((float*)p.C)[ci] = v;
  }
}

// ---- larger tiles: fp32 operands as three bf16 parts each ------------------------------------------------------------------
// A float times 2^24 is the exact sum of three bf16 numbers x0 + x1 + x2 (8 significant bits each, each the rounding of what is left).
// The factor keeps the last bit of every float, the smallest subnormal one too, within bf16's normal range: without it operands lost
// bits below 2^-110 (relative error of a product 2.7e-6 at 1e-35 and 2.6e-4 at 1e-37).  It is taken out of the finished sums.  So
//   x y = x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0) + ...
// in exact bf16 products with fp32 accumulation.  The terms left out (x1 y2, x2 y1, x2 y2) are up to 2^-24 of |x y| where both mantissas
// lie just above 1 (2^-27.5 on average), as much as one rounding of an fp32 sum.  In return the large products x0 y0 have sums of their
// own, which round once for 16 of them; the five small ones go to others, 2^-8 of their size.
// Relative error against 64 bits, fp32 instructions (64 x 64 tiles; 32 x 32) / this: k = 16 7.4e-8 7.4e-8 / 3.2e-8, 128 2.0e-7 1.1e-7 /
// 6.5e-8, 512 4.1e-7 2.1e-7 / 1.3e-7, 4096 1.2e-6 5.8e-7 / 1.9e-7, 50257 4.0e-6 2.0e-6 / 2.3e-7; mantissas between 1 and 1.02 k = 512
// 3.1e-7 9.0e-8 / 3.4e-8; every product losing most 5.9e-8 5.9e-8 / 6.0e-8 (k = 4096 1.9e-5 1.5e-5 / 6.0e-8).
// What bounds it: six bf16 matrix instructions take 3/8 of the time of the fp32 ones they replace; a slab of 128 x 128 x 32 takes
// 1.3 us with all CUs busy, of which they are 0.75 and the taking apart (104 vector instructions a wave, dealt out between them) 0.4:
// 199 TFLOP/s at 4096^3 (fp32 instructions 129), with a tangent 150 at 1024 x 3072 x 768 (106).
// An operand that is infinite or at least 2^104 makes every result that it takes part in a NaN here, and sums of 2^80 (1.2e24) and
// more, or nearly that when the first parts are rounded up by as much as 2^-8 of them, are infinite: blocks that find a result that
// is not finite compute theirs again with the fp32 instructions (150 x 145 x 30000 with an infinity in each block: 2.6 instead of
// 0.85 ms with 64 x 64 tiles, 4.8 instead of 1.65 with 128 x 128; 4096^3 with one in every row 2.4 times as long).
struct F32Parts { uint2 p[3]; };
__device__ __forceinline__ unsigned f32_round_pair(float a, float b) {
  typedef float f32v2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector((f32v2){a, b}, bf16x2));
  asm("" : "+v"(u));  // (the compiler would round again, one number at a time, where the parts are unpacked)
  return u;
}
constexpr float F32_PARTS_SCALE = 16777216.f;  // 2^24
__device__ __forceinline__ F32Parts f32_split(const float4 v) {
  float x = v.x * F32_PARTS_SCALE, y = v.y * F32_PARTS_SCALE, z = v.z * F32_PARTS_SCALE, w = v.w * F32_PARTS_SCALE;
  F32Parts o;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    o.p[q] = make_uint2(f32_round_pair(x, y), f32_round_pair(z, w));
    if (q == 2) break;
    x -= __uint_as_float(o.p[q].x << 16); y -= __uint_as_float(o.p[q].x & 0xffff0000u);
    z -= __uint_as_float(o.p[q].y << 16); w -= __uint_as_float(o.p[q].y & 0xffff0000u);
  }
  return o;
}

// LDS: three planes of R x BK bf16 per operand and stage, in the layouts of the bf16 kernels (LinTile).
template <int R, bool KC, int BK>
struct SplitTile {
  using L = LinTile<R, KC, BK>;
  static constexpr int PLANE = R * BK;  // elements
  // chunk of four elements number c of the slab: along k (KC) or along the rows
  static __device__ __forceinline__ int at(int c) {
    const int line = KC ? c / (BK / 4) : c / (R / 4), e = (KC ? c % (BK / 4) : c % (R / 4)) * 4;
    return line * (L::CPL * 8) + L::swz(line, e >> 3) * 8 + (e & 4);
  }
};

template <int BM, int BN, int WM, int WN, bool TA, bool TB, bool VEC>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, 2) void gemm_f32_split_kernel(F32Group gg) {
  constexpr int BK = 32, NTHR = (BM / WM) * (BN / WN) * 64;
  constexpr bool AKC = !TA, BKC = TB;
  using TileA = F32Tile<BM, AKC, BK, NTHR>;
  using TileB = F32Tile<BN, BKC, BK, NTHR>;
  using SA = SplitTile<BM, AKC, BK>;
  using SB = SplitTile<BN, BKC, BK>;
  constexpr int STAGE = 3 * (SA::PLANE + SB::PLANE);  // elements
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  HF_LDS bf16* const smem = (HF_LDS bf16*)(HF_LDS void*)smem_raw;
  __shared__ int last_block, again;
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

  const int wm0 = (wave / (BN / WN)) * WM, wn0 = (wave % (BN / WN)) * WN;
  constexpr int TM = WM / 32, TN = WN / 32;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  float4 ra[2][TileA::NI], rb[2][TileB::NI];
  uint32_t oa[TileA::template PER<VEC> * TileA::NI], ob[TileB::template PER<VEC> * TileB::NI];
  TileA::template offsets<VEC>(oa, p.lda, m0, p.M, t);
  TileB::template offsets<VEC>(ob, p.ldb, n0, p.N, t);
  const int64_t stepA = TA ? BK * p.lda : BK, stepB = TB ? BK : BK * p.ldb;
  auto base_a = [&](int term, int k0) { return (const float*)p.A[term] + offA + (TA ? (int64_t)k0 * p.lda + m0 : (int64_t)m0 * p.lda + k0); };
  auto base_b = [&](int term, int k0) { return (const float*)p.B[term] + offB + (TB ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0); };
  int f_term = nk > 0 ? it0 / nk : 0, f_slab = nk > 0 ? it0 - f_term * nk : 0;
  const float *fa = nullptr, *fb = nullptr;
  auto advance = [&]() {
    if (f_slab + 1 < nk) {
      ++f_slab;
      fa += stepA;
      fb += stepB;
    } else if (f_term + 1 < p.nterm) {
      ++f_term;
      f_slab = 0;
      fa = base_a(f_term, kbeg);
      fb = base_b(f_term, kbeg);
    }  // else the last slab again, for nobody: every iteration loads, so that none has to wait for its own loads
  };
  auto fetch = [&](auto& va, auto& vb) {
    TileA::template fetch<VEC>(va, fa, oa);
    TileB::template fetch<VEC>(vb, fb, ob);
    advance();
  };
  // (chunks NTHR apart lie 4 NTHR elements apart: that many lines leave the rotation as it is)
  static_assert(NTHR / (BK / 4) % 16 == 0 && NTHR / (BM / 4) % 16 == 0 && NTHR / (BN / 4) % 16 == 0, "lines per round of chunks");
  const int sA0 = SA::at(t), sB0 = SB::at(t);
  constexpr int NCH = TileA::NI + TileB::NI;  // chunks of four that a thread splits per slab
  // chunk c of the slab in registers is split and stored into stage s; with REFILL its registers then receive the chunk of the
  // slab at the cursor
  auto store_one = [&](auto& va, auto& vb, int s, auto c_c, auto refill_c) {
    constexpr int c = decltype(c_c)::value;
    constexpr bool onA = c < TileA::NI;
    constexpr int i = onA ? c : c - TileA::NI, PL = onA ? SA::PLANE : SB::PLANE;
    HF_LDS bf16* d = smem + s * STAGE + (onA ? sA0 : 3 * SA::PLANE + sB0) + i * (4 * NTHR);
    F32Parts x;
    if constexpr (onA) x = f32_split(va[i]);
    else x = f32_split(vb[i]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      *(HF_LDS u32x2*)(d + q * PL) = (u32x2){x.p[q].x, x.p[q].y};
    }
    if constexpr (decltype(refill_c)::value) {
      if constexpr (onA) va[i] = TileA::template fetch_one<VEC>(fa, oa, i);
      else vb[i] = TileB::template fetch_one<VEC>(fb, ob, i);
    }
  };
  auto store = [&](auto& va, auto& vb, int s) {
    static_for<NCH>([&](auto c_c) { store_one(va, vb, s, c_c, std::false_type{}); });
  };
  const int fA = (int)lin_frag_addr<BM, AKC, BK, 32>(wm0, 0, lane) / 2, fB = (int)lin_frag_addr<BN, BKC, BK, 32>(wn0, 0, lane) / 2;
  // fragment i of a plane in k-step kk (row blocks of a wave differ in one bit field of the address, as do k-steps of a
  // k-contiguous tile)
  static_assert((TM == 1 || WM == 64) && TN == 1, "row blocks of a wave");
  auto frag = [&](auto kc_c, auto r_c, const HF_LDS bf16* plane, int f0, int i, int kk) -> bf16x8 {
    constexpr bool KC = decltype(kc_c)::value;
    constexpr int R = decltype(r_c)::value;
    if constexpr (KC) {
      return *(const HF_LDS bf16x8*)(plane + (f0 ^ (kk * 16)) + i * 32 * BK);
    } else {
      const HF_LDS bf16* q0 = plane + (f0 ^ (i * 32)) + kk * 16 * R;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((HF_LDS bf16x4*)q0);
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((HF_LDS bf16x4*)(q0 + 4 * R));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  bf16x8 xa[2][3][TM], xb[2][3][TN];
  auto read_kk = [&](int s, auto kk_c) {
    constexpr int kk = decltype(kk_c)::value;
    const HF_LDS bf16* As = smem + s * STAGE;
    const HF_LDS bf16* Bs = As + 3 * SA::PLANE;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        xa[kk][q][i] = frag(std::integral_constant<bool, AKC>{}, std::integral_constant<int, BM>{}, As + q * SA::PLANE, fA, i, kk);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        xb[kk][q][j] = frag(std::integral_constant<bool, BKC>{}, std::integral_constant<int, BN>{}, Bs + q * SB::PLANE, fB, j, kk);
    }
  };
  // The matrix instructions of k-step kk, whose fragments are in registers: the small terms, then the large one; chunks [C0, C1) of the slab in
  // registers (va, vb) are split and stored into stage ds between them.
  f32x16 low[TM][TN], sum[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { low[i][j][r] = 0.f; sum[i][j][r] = 0.f; }
  // Vector instructions that take a chunk apart, and a few addresses where the B side is read row by row (us with 26 / 32: 1024 x 3072 x 768
  // 100.6 / 98.7, 4096^3 with a tangent 2108 / 2065; A B^T 1024 x 50257 x 768 1314 / 1342).
  constexpr int SPLIT_VALU = TB ? 26 : 32;
  constexpr int MQ = 6 * TM * TN, CH = NCH / 2, NFRAG = 3 * (TM * (AKC ? 1 : 2) + TN * (BKC ? 1 : 2));
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using IH = std::integral_constant<int, CH>;
  using IN = std::integral_constant<int, NCH>;
  auto multiply = [&](auto kk_c, auto c0_c, auto c1_c, int ds, auto& va, auto& vb) {
    constexpr int kk = decltype(kk_c)::value, C0 = decltype(c0_c)::value, C1 = decltype(c1_c)::value;
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    static_for<MQ>([&](auto q_c) {
      constexpr int q = decltype(q_c)::value, term = q / (TM * TN), i = q % (TM * TN) / TN, j = q % TN;
      f32x16& to = term == 5 ? acc[i][j] : low[i][j];
      to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[kk][PA[term]][i], xb[kk][PB[term]][j], to, 0, 0, 0);
      constexpr int c = C0 + q * (C1 - C0) / MQ, cn = C0 + (q + 1) * (C1 - C0) / MQ;
      static_assert(cn - c <= 1, "at most one chunk per matrix instruction");
      if constexpr (cn > c) store_one(va, vb, ds, std::integral_constant<int, c>{}, std::true_type{});
    });
    // A wave issues in order: one matrix instruction (32 clocks of the pipe), then what fits into its shadow
    if constexpr (C1 > C0) {
      static_for<MQ>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                // matrix instruction
        __builtin_amdgcn_sched_group_barrier(0x100, (NFRAG + MQ - 1) / MQ, 0);             // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x002, (SPLIT_VALU * (C1 - C0) + MQ - 1) / MQ, 0);    // arithmetic
        if constexpr (q % 2 == 1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);       // LDS write
        if constexpr (q % 3 == 1) __builtin_amdgcn_sched_group_barrier(0x020, VEC ? 1 : 4, 0);  // load
      });
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Long sums in two levels: every 32 slabs (1024 k of all terms) the running sums go to another one and start again, which
  // keeps the rounding of a sum of 50000 products near that of 1000 in a row.
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) { sum[i][j][r] += acc[i][j][r] + low[i][j][r]; acc[i][j][r] = 0.f; low[i][j][r] = 0.f; }
  };
  // Slab i, in LDS stage i % 2: the last k-step of the slab before it covers the reads of its first one, so that the barrier
  // between slabs exposes no LDS latency; slab i + 1 goes from registers to the other stage (the last time it is an old one that
  // nobody reads), and as each chunk has gone, that of slab i + 3 is loaded into its registers, two slabs before it is needed.
  const int nit = it1 - it0;
  auto slab = [&](int i, auto par_c) {
    constexpr int s = decltype(par_c)::value;
    __builtin_amdgcn_sched_barrier(0);
    read_kk(s, I0{});
    multiply(I1{}, I0{}, IH{}, 1 - s, ra[1 - s], rb[1 - s]);
    if ((i & 31) == 0) flush();
    read_kk(s, I1{});
    multiply(I0{}, IH{}, IN{}, 1 - s, ra[1 - s], rb[1 - s]);
    advance();
    __syncthreads();
  };
  if (nit > 0) {
    fa = base_a(f_term, kbeg + f_slab * BK);
    fb = base_b(f_term, kbeg + f_slab * BK);
    fetch(ra[0], rb[0]);
    fetch(ra[1], rb[1]);
    store(ra[0], rb[0], 0);
    fetch(ra[0], rb[0]);
    // the first slab has none before it: a k-step of zeros
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const bf16x8 zero = {};
#pragma unroll
      for (int i = 0; i < TM; ++i) xa[1][q][i] = zero;
#pragma unroll
      for (int j = 0; j < TN; ++j) xb[1][q][j] = zero;
    }
    __syncthreads();
    int i = 0;
    for (; i + 1 < nit; i += 2) {
      slab(i, I0{});
      slab(i + 1, I1{});
    }
    if (i < nit) slab(i, I0{});
    multiply(I1{}, I0{}, I0{}, 0, ra[0], rb[0]);
  }
  const bool tail = kbeg + nk * BK < kend && ks == nks - 1;
  if (tail) {
    for (int term = 0; term < p.nterm; ++term) {
      TileA::fetch_tail(ra[0], (const float*)p.A[term] + offA, p.lda, m0, p.M, kbeg + nk * BK, kend, t);
      TileB::fetch_tail(rb[0], (const float*)p.B[term] + offB, p.ldb, n0, p.N, kbeg + nk * BK, kend, t);
      __syncthreads();
      store(ra[0], rb[0], 0);
      __syncthreads();
      read_kk(0, I0{});
      read_kk(0, I1{});
      multiply(I0{}, I0{}, I0{}, 0, ra[0], rb[0]);
      multiply(I1{}, I0{}, I0{}, 0, ra[0], rb[0]);
    }
  }
  flush();
  // Only results that are stored count: a tile's rows and columns beyond the operand hold products of whatever lies in the
  // padding of its rows.  (0 times a number is zero or, if that is not finite, a NaN, which stays one; no branches.)
  float nans = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] = sum[i][j][r] * (1.f / F32_PARTS_SCALE / F32_PARTS_SCALE);
        nans = fmaf(m0 + wm0 + i * 32 + (r >> 2) * 8 + half * 4 + (r & 3) < p.M ? sum[i][j][r] : 0.f, 0.f, nans);
      }
  const bool bad = nans != 0.f && n0 + wn0 + col < p.N;
  if (t == 0) again = 0;
  __syncthreads();
  if (__any(bad) && lane == 0) again = 1;
  __syncthreads();
  if (__builtin_expect(again, 0)) {  // this block's share of k once more, for the whole tile
    float* const As = (float*)smem_raw;
    float* const Bs = As + TileA::FLOATS;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll 1
    for (int term = 0; term < p.nterm; ++term) {
      const float *A = (const float*)p.A[term] + offA, *B = (const float*)p.B[term] + offB;
      const int k0 = kbeg + min(max(it0 - term * nk, 0), nk) * BK, k1 = tail ? kend : kbeg + min(max(it1 - term * nk, 0), nk) * BK;
      auto load = [&](int k) {
        TileA::fetch_tail(ra[0], A, p.lda, m0, p.M, k, k1, t);
        TileB::fetch_tail(rb[0], B, p.ldb, n0, p.N, k, k1, t);
      };
      if (k0 < k1) load(k0);
#pragma unroll 1
      for (int k = k0; k < k1; k += BK) {
        __syncthreads();
        TileA::store(ra[0], As, t);
        TileB::store(rb[0], Bs, t);
        __syncthreads();
        if (k + BK < k1) load(k + BK);
#pragma unroll
        for (int gk = 0; gk < BK / 8; ++gk) {
          const float4 y = TileB::read(Bs, wn0 + col, gk, half);
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const float4 x = TileA::read(As, wm0 + i * 32 + col, gk, half);
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc[i][0], 0, 0, 0);
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc[i][0], 0, 0, 0);
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc[i][0], 0, 0, 0);
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc[i][0], 0, 0, 0);
          }
        }
      }
    }
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
          __hip_atomic_store(mine + ((i * TN + j) * 16 + r) * NTHR, acc[i][j][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
        acc[e / (TN * 16)][(e / 16) % TN][e % 16] += __hip_atomic_load(src + e * NTHR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // accumulator tile: column lane & 31, rows 8*(r/4) + 4*(lane/32) + r%4.  Blocks whose tile lies inside the result store without a
  // branch an element, which pays for the look at the results above (us with / without, 1024 x 2304 x 768 with its tangent 70 / 66,
  // A^T B 768 x 3072 x 1024 89 / 85).
  static_assert(TN == 1, "one column a lane");
  const int gn = n0 + wn0 + col, row0 = m0 + wm0 + half * 4;
  float bsum = 0.f;
  if (gn < p.N) {
    if (p.bias) bsum += ((const float*)p.bias)[gn];
    if (p.bias_t) bsum += p.bias_t[gn];
  }
  auto write_out = [&](auto whole_c, auto add_c) {
    constexpr bool WHOLE = decltype(whole_c)::value, ADD = decltype(add_c)::value;
    if (!WHOLE && gn >= p.N) return;
    float* const C = (float*)p.C + offC + (int64_t)row0 * p.ldc + gn;
    const float* const D = ADD ? p.Cadd + offC + (int64_t)row0 * p.ldc + gn : nullptr;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = i * 32 + (r >> 2) * 8 + (r & 3);
        if (!WHOLE && row0 + row >= p.M) continue;
        float v = p.alpha * acc[i][0][r] + bsum;
        if (ADD) v += D[row * p.ldc];
        C[row * p.ldc] = v;
      }
  };
  using F = std::false_type;
  using T = std::true_type;
  if (m0 + BM <= p.M && n0 + BN <= p.N) {
    if (p.Cadd) write_out(T{}, T{});
    else write_out(T{}, F{});
  } else if (p.Cadd) {
    write_out(F{}, T{});
  } else {
    write_out(F{}, F{});
  }
}

template <bool VEC>
static hipError_t launch_mfma(const F32Group& gg, int grid, hipStream_t st) {
  const GemmP& p = gg.g[0];
  if (!p.transA && !p.transB) hipLaunchKernelGGL((gemm_f32_mfma_kernel<false, false, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else if (!p.transA) hipLaunchKernelGGL((gemm_f32_mfma_kernel<false, true, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else if (!p.transB) hipLaunchKernelGGL((gemm_f32_mfma_kernel<true, false, VEC>), dim3(grid), dim3(256), 0, st, gg);
  else hipLaunchKernelGGL((gemm_f32_mfma_kernel<true, true, VEC>), dim3(grid), dim3(256), 0, st, gg);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, bool TA, bool TB, bool VEC>
static hipError_t launch_split_one(const F32Group& gg, int grid, hipStream_t st) {
  static OncePerDevice once;
  auto kern = gemm_f32_split_kernel<BM, BN, WM, WN, TA, TB, VEC>;
  constexpr int smem = 2 * 3 * (BM + BN) * 32 * 2;
  if (hipError_t e = once.lds_limit((const void*)kern, smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3((BM / WM) * (BN / WN) * 64), smem, st, gg);
  return hipGetLastError();
}
template <int BM, int BN, int WM, int WN, bool VEC>
static hipError_t launch_split_vec(const F32Group& gg, int grid, hipStream_t st) {
  const GemmP& p = gg.g[0];
  if (!p.transA && !p.transB) return launch_split_one<BM, BN, WM, WN, false, false, VEC>(gg, grid, st);
  if (!p.transA) return launch_split_one<BM, BN, WM, WN, false, true, VEC>(gg, grid, st);
  if (!p.transB) return launch_split_one<BM, BN, WM, WN, true, false, VEC>(gg, grid, st);
  return launch_split_one<BM, BN, WM, WN, true, true, VEC>(gg, grid, st);
}
template <int BM, int BN, int WM, int WN>
static hipError_t launch_split(const F32Group& gg, int grid, bool vec, hipStream_t st) {
  return vec ? launch_split_vec<BM, BN, WM, WN, true>(gg, grid, st) : launch_split_vec<BM, BN, WM, WN, false>(gg, grid, st);
}
// Tiles, the clocks a slab takes a CU that has enough blocks of them, and how much of that rate one to four resident blocks
// reach: 64 x 64 has room for three (48 KB of LDS each; 1120 clocks a slab alone), 128 x 128 for one, 32 x 32 (64-deep slabs
// whose k its waves share) for four.
struct F32Cfg { int bm, bn, bk, resident; double slab_clk, busy[5]; };
static const F32Cfg kF32Cfg[] = {{64, 64, 32, 3, 870., {1., 0.78, 0.92, 1., 1.}}, {128, 128, 32, 1, 2500., {1., 1., 1., 1., 1.}},
                                  {32, 32, 64, 4, 665., {1., 0.68, 0.79, 0.92, 0.99}}};

// Estimated clocks of a launch whose products have cnt[i] blocks of len[i] clocks, longest first.  With one resident block a CU
// takes the next when it has finished one.  Of the small tiles, four a CU are dealt in turn at the start: launches of no more last as long as the fullest CU, others as long as the average and a block more.
static double f32_estimate(const int64_t* cnt, const double* len, int n, const F32Cfg& c) {
  const double* const busy = c.busy;
  int64_t blocks = 0;
  double sum = 0.;
  for (int i = 0; i < n; ++i) { blocks += cnt[i]; sum += (double)cnt[i] * len[i]; }
  if (blocks == 0) return 0.;
  if (c.resident == 1) {
    if (blocks > 16 * 256) return sum / 256. + 0.5 * len[n - 1];
    // CUs by the time at which they are free, as groups of equal times
    double at[64] = {0.};
    int64_t cus[64] = {256};
    int groups = 1;
    double end = 0.;
    for (int i = 0; i < n; ++i)
      for (int64_t left = cnt[i]; left > 0;) {
        int m = 0;
        for (int k = 1; k < groups; ++k)
          if (cus[k] > 0 && (cus[m] == 0 || at[k] < at[m])) m = k;
        const int64_t take = std::min(left, cus[m]);
        const double done = at[m] + len[i];
        end = std::max(end, done);
        left -= take;
        cus[m] -= take;
        int to = 0;
        while (to < groups && cus[to] > 0 && at[to] != done) ++to;
        if (to == 64) return std::max(end, sum / 256. + 0.5 * len[n - 1]);
        if (to == groups) { ++groups; cus[to] = 0; }
        at[to] = done;
        cus[to] += take;
      }
    return end;
  }
  if (blocks > 1024) return sum / 256. / busy[4] + sum / (double)blocks;
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
    worst = std::max(worst, load / busy[held]);
    if (i < n) start += cnt[i];
  }
  return worst;
}

// The choice of tile and parts: fills gg but for its pointers, with products in launch order (order[k]: position in ps).  Returns the tile's
// index, -1 for products that no launch takes.  scratch: there is a workspace (ws_elems floats) and counters, so k may be cut.
static int plan_group(const GemmP* ps, int n, int nb, bool scratch, int64_t ws_elems, int force_cfg, int force_ks, F32Group& gg, int* order) {
  if (n < 1 || n > F32_GROUP_MAX) return -1;
  for (int i = 1; i < n; ++i)
    if (ps[i].transA != ps[0].transA || ps[i].transB != ps[0].transB) return -1;
  auto tiles_of = [&](const GemmP& p, const F32Cfg& c) {
    return ((int64_t)p.M + c.bm - 1) / c.bm * (((int64_t)p.N + c.bn - 1) / c.bn);
  };
  auto slabs_of = [&](const GemmP& p, const F32Cfg& c) { return (int64_t)p.nterm * ((p.K + c.bk - 1) / c.bk); };
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order, order + n, [&](int a, int b) { return (int64_t)ps[a].nterm * ps[a].K > (int64_t)ps[b].nterm * ps[b].K; });
  // Tile and parts of k (the same for all products): the pair with the shortest estimated launch.  (Under klimit the blocks are
  // priced with the whole k, about twice their average: only the tile is chosen there, and all tiles are priced alike.)  A cut
  // costs each block 1500 clocks a 64 x 64 part (partial tile out) and the launch 6000 and 1500 or 10000 a part (sums of small or large ones).
  // Measured (us; 64 x 64 whole and in its best parts, 128 x 128 the same, 32 x 32, chosen): primal product and tangent
  // 1024x768x768 41 36/2 53 37/2 45, 37; 1024x2304x768 81 - 68 - 114, 68; 1024x3072x768 104 - 96 - 149, 97; 1024x768x3072 122
  // 108/3 188 92/3 163, 92; 1024x50257x768 1624 - 1261 - 2313, 1293; 1024x768x50257 1980 1641/4 3031 1305/8 3107, 1270; 512x128x128
  // 9.8 - 14 - 6.1, 6.1; 512x128x512 23 13/6 36 20/6 10.9, 11.0; A^T B 768x3072x1024 92 82/3 72 70/3 102, 75.
  int cfg = 0, parts = 1;
  double best = 1e300;
  for (int ci = 0; ci < 3; ++ci) {
    if (force_cfg >= 0 && ci != force_cfg) continue;
    const F32Cfg& c = kF32Cfg[ci];
    const bool cut = ci != 2 && scratch && !ps[0].klimit;
    const double tile = c.bm * c.bn / 4096.;
    int64_t all = 0;
    for (int i = 0; i < n; ++i) all += tiles_of(ps[i], c) * nb;
    for (int k = 1; k <= (cut ? 12 : 1); ++k) {
      if (k > 1 && slabs_of(ps[order[0]], c) / k < 4) break;
      if (k > 1 && (all * k * c.bm * c.bn > ws_elems || all > F32_COUNTERS)) break;
      int64_t cnt[F32_GROUP_MAX];
      double len[F32_GROUP_MAX];
      for (int i = 0; i < n; ++i) {
        const GemmP& p = ps[order[i]];
        const int64_t slabs = slabs_of(p, c), nks = std::min<int64_t>(k, slabs);
        cnt[i] = tiles_of(p, c) * nb * nks;
        len[i] = c.slab_clk * (double)slabs / (double)nks + (nks > 1 ? 1500. * tile : 0.);
      }
      const double t = f32_estimate(cnt, len, n, c) + (k > 1 ? 6000. + (ci == 0 ? 1500. : 10000.) * k : 0.);
      if (t < best) { best = t; cfg = ci; parts = k; }
    }
  }
  const F32Cfg& c = kF32Cfg[cfg];
  gg = {};
  gg.n = n;
  int64_t first = 0, part = 0, cnt = 0;
  for (int k = 0; k < n; ++k) {
    gg.g[k] = ps[order[k]];
    const GemmP& p = gg.g[k];
    const int64_t tiles = tiles_of(p, c), blocks = tiles * nb;
    int64_t nks = 1;
    if (cfg != 2 && scratch && !p.klimit) {
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
    if (first > (int64_t)1 << 30) return -1;
  }
  gg.first[n] = (int)first;
  return cfg;
}

int f32_plan(const GemmP* ps, int n, int nb, int64_t ws_elems, int* parts) {
  F32Group gg;
  int order[F32_GROUP_MAX];
  const int cfg = plan_group(ps, n, nb, ws_elems > 0, ws_elems, -1, 0, gg, order);
  for (int k = 0; cfg >= 0 && k < n; ++k) parts[order[k]] = gg.nks[k];
  return cfg;
}

// All products have the same transposes and nb batch entries.  ws / counters nullptr: k is never cut.
hipError_t launch_gemm_f32_group(const GemmP* ps, int n, int nb, float* ws, int64_t ws_elems, int* counters, int force_cfg,
                                 int force_ks, hipStream_t st) {
  F32Group gg;
  int order[F32_GROUP_MAX];
  const int cfg = plan_group(ps, n, nb, ws && counters, ws_elems, force_cfg, force_ks, gg, order);
  if (cfg < 0) return hipErrorInvalidValue;
  gg.part = ws;
  gg.counters = counters;
  const int grid = gg.first[n];
  bool vec = true;
  for (int i = 0; i < n; ++i) vec = vec && ps[i].vecA && ps[i].vecB;
  if (cfg == 0) return launch_split<64, 64, 32, 32>(gg, grid, vec, st);
  if (cfg == 1) return launch_split<128, 128, 64, 32>(gg, grid, vec, st);
  return vec ? launch_mfma<true>(gg, grid, st) : launch_mfma<false>(gg, grid, st);
}

}  // namespace hf
