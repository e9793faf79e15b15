// The Lanczos update of short vectors by one block of 16 waves: device code shared by the kernel of lanczos.hip and by the one that adds
// up an MLP product (mlp.hip).
#pragma once
#include "hf_internal.h"
#include "lanczos.h"

namespace hf {

// v of the lane O away inside the wave: halves and odd / even rows of 16 lanes trade places, inside a row lanes rotate (so that steps
// 8, 4, 2, 1 in that order add up a row).  In registers: a shuffle through LDS takes ten times as long, and short runs wait for little else.
template <int O>
__device__ __forceinline__ float lane_across(float v) {
  const int x = __builtin_bit_cast(int, v);
  if constexpr (O >= 16) {
    const auto y = O == 32 ? __builtin_amdgcn_permlane32_swap(x, x, false, false) : __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & O) ? y[0] : y[1]);
  } else {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, 0x120 + O, 0xf, 0xf, false));  // row_ror
  }
}
template <int O>
__device__ __forceinline__ double lane_across(double v) {
  typedef float f32v2 __attribute__((ext_vector_type(2)));
  const f32v2 x = __builtin_bit_cast(f32v2, v);
  return __builtin_bit_cast(double, (f32v2){lane_across<O>(x.x), lane_across<O>(x.y)});
}
// Sum over the lanes that agree in lane % PER, in all of them.
template <int PER, typename T>
__device__ __forceinline__ T lanes_sum(T v) {
  if constexpr (PER <= 32) v += lane_across<32>(v);
  if constexpr (PER <= 16) v += lane_across<16>(v);
  if constexpr (PER <= 8) v += lane_across<8>(v);
  if constexpr (PER <= 4) v += lane_across<4>(v);
  if constexpr (PER <= 2) v += lane_across<2>(v);
  if constexpr (PER <= 1) v += lane_across<1>(v);
  return v;
}
__device__ __forceinline__ float wave_max_f(float v) {
  v = fmaxf(v, lane_across<32>(v));
  v = fmaxf(v, lane_across<16>(v));
  v = fmaxf(v, lane_across<8>(v));
  v = fmaxf(v, lane_across<4>(v));
  v = fmaxf(v, lane_across<2>(v));
  return fmaxf(v, lane_across<1>(v));
}
__device__ __forceinline__ double wave_sum_d(double v) { return lanes_sum<1>(v); }

__device__ __forceinline__ double block16_sum_d(double v, double* red /* [16] */) {
  v = wave_sum_d(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) s += red[i];
  return s;
}

// <a, b> over n elements by one wave
__device__ __forceinline__ double wave_dot(const float* a, const float* b, int n) {
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x & 63; i < n; i += 64) s += (double)a[i] * (double)b[i];
  return wave_sum_d(s);
}

// The iteration's scalars, on the device and in the host's array.  chained: the host enqueues iterations ahead of their
// results, so one that may not advance stops those behind it.
__device__ __forceinline__ void small_scalars(const LzSmall& u, double alpha, double beta, double f0, double f1, bool ok) {
  double *scal = u.scal, *host = u.host;
  scal[S_ALPHA] = alpha; scal[S_BETA] = beta; scal[S_REDO] = 0.0; scal[S_FLAG0] = f0; scal[S_FLAG1] = f1;
  host[S_ALPHA] = alpha; host[S_BETA] = beta; host[S_FLAG0] = f0; host[S_FLAG1] = f1;
  if (u.chained && !ok) scal[S_STOP] = 1.0;
}

// Full orthogonalisation against an fp32 basis of nq = k + 1 rows: the first Gram-Schmidt pass on w = H q_k itself, a
// second one where it shrank the norm below 1/sqrt(2), q_{k+1} = r / beta_k into any of row, spill, vb.  w: in LDS, complete;
// f0, f1: error bits and valid labels of the product.
__device__ __forceinline__ void lz_small_full_block(const LzSmall& u, float* w, double* sm_c /* [nq + 1] */, double* red, int f0, int f1) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = u.n, nq = u.nq;
  const float* const Q = u.Q;
  double alpha = 0.0, before = 0.0, beta = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int j = wave; j <= nq; j += 16) {
      const double d = wave_dot(j < nq ? Q + (int64_t)j * u.ldq : w, w, n);
      if (lane == 0) sm_c[j] = d;
    }
    __syncthreads();
    if (pass == 0) {  // as lz_first_plan, with what three terms would leave for beta_k
      alpha = sm_c[nq - 1];
      const double p = nq >= 2 ? sm_c[nq - 2] : 0.0, ww = sm_c[nq], rest = ww - alpha * alpha - p * p;
      bool grows = false;
      if (alpha * alpha > 4.0 * rest)
        for (int j = 0; j < nq - 2; ++j) grows = grows || sm_c[j] * sm_c[j] > 1e-10 * ww;
      before = rest > 1e-5 * ww && !grows ? sqrt(rest) : INFINITY;
    }
    double s = 0.0;
    for (int i = t; i < n; i += 1024) {
      float x = w[i];
#pragma unroll 8
      for (int j = 0; j < nq; ++j) x = fmaf(-(float)sm_c[j], Q[(int64_t)j * u.ldq + i], x);
      w[i] = x;
      s += (double)x * (double)x;
    }
    beta = sqrt(block16_sum_d(s, red));
    if (pass == 1 || !(beta < before * 0.70710678118654752)) break;
  }
  const bool ok = beta >= u.tol && beta > 0.0 && f0 == 0 && f1 != 0;
  const float inv = (float)(1.0 / beta);
  for (int i = t; i < n; i += 1024) {
    const float x = w[i];
    u.r[i] = x;
    if (!ok) continue;
    const float q = x * inv;
    if (u.row) u.row[i] = q;
    if (u.spill) u.spill[i] = q;
    if (u.vb) u.vb[i] = (bf16)q;
  }
  if (t == 0) small_scalars(u, alpha, beta, (double)f0, (double)f1, ok);
}

// Three-term recurrence: alpha_k, beta_k, and q_{k+1} over qp; r (may be NULL) takes a copy of w = H q_k.
__device__ __forceinline__ void lz_small_three_block(const LzSmall& u, float* w, double* red, int f0, int f1) {
  const int t = threadIdx.x, n = u.n;
  const float* const q = u.q;
  const float bprev = u.chained ? (float)u.scal[S_BETA] : u.bprev;  // of the iteration before, whose result the host may not have seen
  double s = 0.0;
  for (int i = t; i < n; i += 1024) {
    float x = w[i];
    if (u.r) u.r[i] = x;
    if (u.use_prev) x = fmaf(-bprev, u.qp[i], x);
    w[i] = x;
    s += (double)x * (double)q[i];
  }
  const double alpha = block16_sum_d(s, red);
  const float al = (float)alpha;
  s = 0.0;
  for (int i = t; i < n; i += 1024) {
    const float x = fmaf(-al, q[i], w[i]);
    w[i] = x;
    s += (double)x * (double)x;
  }
  const double beta = sqrt(block16_sum_d(s, red));
  const bool ok = beta >= u.tol && beta > 0.0 && f0 == 0 && f1 != 0;
  if (ok) {
    const float inv = (float)(1.0 / beta);
    for (int i = t; i < n; i += 1024) {
      const float x = w[i] * inv;
      u.qp[i] = x;
      if (u.vb) u.vb[i] = (bf16)x;
    }
  }
  if (t == 0) small_scalars(u, alpha, beta, (double)f0, (double)f1, ok);
}

}  // namespace hf
