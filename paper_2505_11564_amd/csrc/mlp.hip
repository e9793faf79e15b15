// The Hessian-vector product of the tanh MLP as one launch and a sum, for fp32 models whose weights fit a CU's LDS.
//
// What bounds it: nothing but latency (the 32-32-10 model at 256 samples is 5 MFLOP and 11 KB of weights): as a
// chain of products and pointwise kernels it was 15 launches of 1.5 to 13 us, each waiting for the one before.  The samples
// are independent, so a block takes its own through the forward, loss and backward sweeps with their tangents in LDS and
// leaves its share of H v (n floats) in the workspace; a second kernel adds the blocks' shares in a fixed order.
// In a run of few samples that sum is part of the Lanczos update behind it (mlp_sum_update_kernel), one launch less.
// Measured at that shape: 62 us of kernels in 15 launches (with the products of gemm_f32.hip); 13 + 4 us with 256 threads a block and
// the update, 6.5, behind them; 11.7 + 8 us now, at n = 4204 (16-200-4) 19 us (27).  Of the 11.7 most is the same at n = 90 (9): what a launch
// takes to fetch 10 KB of instructions and go through a dozen barriers.
// Blocks: one per eight samples up to one per CU (the largest weights take a CU's LDS), then several turns each.  With at most
// 64 blocks, whatever the batch, a large one lost to the chain of products.  hf_hvp, us (chain / 64 blocks / 256 blocks and the
// sum spread over eight groups of lanes): 128-64-10 at 256 samples 97 / 55 / 54, 2048 138 / 134 / 62, 16384 451 / 839 / 250, 65536
// 1553 / - / 917; 32-32-10 88 / 34 / 33, 124 / 58 / 34, 428 / 269 / 94, 1493 / - / 292; 100-70-31 118 / 64 / 62, 202 / 159 /
// 68, 852 / 1029 / 297, 3093 / - / 1102.  256 threads and 32 lanes a sample / sixteen waves: 32-32-10 at 3000 samples 41 / 36, 16384 89 / 68;
// 64-64-10 62 / 44, 165 / 94; 16-200-4 85 / 49, 250 / 114; 8-8-2 32 / 32, 57 / 58.  Larger batches (MLP_FUSED_MAX_BATCH) have not been measured and take the chain.
//   f = x W1 + b1, g = tanh f, z = g W2 + b2, p = softmax z, and along v:
//   f_t = x W1_t + b1_t, g_t = g' f_t, z_t = g_t W2 + g W2_t + b2_t
//   dz = (p - onehot) s, dz_t = p (z_t - <p, z_t>) s;  dg = dz W2^T, dg_t = dz_t W2^T + dz W2_t^T
//   da_t = g' dg_t + g'' f_t dg,  g' = 1 - g^2, g'' = -2 g g'
//   (Hv)_W2 = g_t^T dz + g^T dz_t, (Hv)_b2 = sum dz_t, (Hv)_W1 = x^T da_t, (Hv)_b1 = sum da_t
#include "engine.h"
#include "lanczos_small.h"

#include <algorithm>
#include <cmath>

namespace hf {

constexpr int MLP_ROWS = 8, MLP_THREADS = 1024;  // samples a block works on at a time: two waves each
constexpr int64_t MLP_ADD_IN_UPDATE = 65536;      // most floats of shares that the one block of an update adds

struct MlpP {
  const float *params, *v, *x;
  const int32_t* labels;
  int B, I, H, O;
  float seed;
  int accumulate;
  float* part;        // [blocks][n]
  double* part_loss;  // [blocks]
  int* flags;
};

// LDS floats: W1, W1_t, b1, b1_t; W2, W2_t with rows of LO = O | 1 floats (lanes that walk down a column then
// hit different banks); b2, b2_t; the block's share of H v; the rows' buffers.
__host__ __device__ inline int64_t mlp_lds_floats(int64_t I, int64_t H, int64_t O, int rows) {
  const int64_t LO = O | 1;
  return 2 * (I * H + H + H * LO + O) + (I * H + H + H * O + O) + rows * (I + 4 * H + 4 * LO);
}

// Sum over k = k0, k0 + step, .. < K of a[k] u[k st], and of b[k] w[k st] if there is a b.
__device__ __forceinline__ float lds_dot(const float* a, const float* u, const float* b, const float* w, int st, int k0, int step, int K) {
  float s = 0.f;
  if (!b) {
#pragma unroll 4
    for (int k = k0; k < K; k += step) s = fmaf(a[k], u[k * st], s);
  } else {
#pragma unroll 4
    for (int k = k0; k < K; k += step) s = fmaf(b[k], w[k * st], fmaf(a[k], u[k * st], s));
  }
  return s;
}

// Two waves a sample (WPS), one for the primal of each sum and one for the tangent, or one for both.  The three matrix-vector products share their code, as do
// the blocks of H v: a launch fetches its instructions anew and runs through them once, so that a kernel waits for its own size.
template <int WPS>
__global__ __launch_bounds__(MLP_THREADS) void mlp_hvp_kernel(MlpP p) {
  constexpr int MLP_ROWS = MLP_THREADS / 64 / WPS;
  extern __shared__ float sm[];
  const int t = threadIdx.x, I = p.I, H = p.H, O = p.O, LO = O | 1, IH = I * H, HO = H * O, n = IH + H + HO + O;
  float* w1 = sm;        float* w1t = w1 + IH;
  float* b1 = w1t + IH;  float* b1t = b1 + H;
  float* w2 = b1t + H;   float* w2t = w2 + H * LO;
  float* b2 = w2t + H * LO; float* b2t = b2 + O;
  float* acc = b2t + O;
  float* X = acc + n;                                              // [rows][I]
  float* G = X + MLP_ROWS * I;    float* Ft = G + MLP_ROWS * H;    // g, f_t
  float* E = Ft + MLP_ROWS * H;   float* Et = E + MLP_ROWS * H;    // g_t, then dg, then g_t again; dg_t, then da_t
  float* Z = Et + MLP_ROWS * H;   float* Zt = Z + MLP_ROWS * LO;   // z, z_t
  float* D = Zt + MLP_ROWS * LO;  float* Dt = D + MLP_ROWS * LO;   // dz, dz_t
  __shared__ int cnt[MLP_THREADS / 64], bad[MLP_THREADS / 64];
  __shared__ double rowloss[MLP_ROWS];
  __shared__ float one;

  const int wave = t >> 6, lane = t & 63, row = wave / WPS, lane_r = t % (64 * WPS);
  const bool first_wave = wave % WPS == 0;
  // all loads of the start are independent and in flight together: weights, direction, labels, the first samples
  const int r_first = blockIdx.x * MLP_ROWS;
  for (int i = lane_r; i < I; i += 64 * WPS) X[row * I + i] = r_first + row < p.B ? p.x[(int64_t)(r_first + row) * I + i] : 0.f;
#pragma unroll 4
  for (int j = t; j < n; j += MLP_THREADS) {
    const float w = p.params[j], d = p.v[j];
    int at = j, gap = IH;  // the weight's place, and how far behind it its tangent lies
    if (j >= IH) {
      const int q = j - IH - H;
      at = j + IH;
      gap = H;
      if (q >= HO) { at += H + 2 * H * LO - HO; gap = O; }
      else if (q >= 0) { at += H + q / O * (LO - O); gap = H * LO; }
    }
    sm[at] = w;
    sm[at + gap] = d;
    acc[j] = 0.f;
  }
  // every block counts the valid labels of the whole batch itself
  int c = 0, b = 0;
  for (int i = t; i < p.B; i += MLP_THREADS) {
    const int y = p.labels[i];
    c += (y >= 0);
    b |= (y >= O);
  }
  c = (int)lanes_sum<1>((float)c);  // (at most MLP_FUSED_MAX_BATCH: exact)
  b = __any(b);
  if (lane == 0) { cnt[wave] = c; bad[wave] = b; }
  if (t == 0) one = 1.f;
  __syncthreads();
  int nv = 0, any_bad = 0;
  for (int w = 0; w < MLP_THREADS / 64; ++w) { nv += cnt[w]; any_bad |= bad[w]; }
  if (blockIdx.x == 0 && t == 0) {
    const int bits = (any_bad ? 2 : 0) | (nv == 0 ? 4 : 0);
    p.flags[0] = p.accumulate ? (p.flags[0] | bits) : bits;
    p.flags[1] = nv;
  }
  const float invN = p.seed / (float)max(1, nv);
  double loss = 0.0;
#pragma unroll 1
  for (int r0 = r_first; r0 < p.B; r0 += gridDim.x * MLP_ROWS) {
    const int gr = r0 + row;
    const bool in = gr < p.B;
    if (r0 != r_first) {
      __syncthreads();  // the products of the previous samples are done with the row buffers
      for (int i = lane_r; i < I; i += 64 * WPS) X[row * I + i] = in ? p.x[(int64_t)gr * I + i] : 0.f;
      __syncthreads();
    }
    // ph 0: f, f_t; 1: z, z_t and from them dz, dz_t; 2: dg, dg_t
#pragma unroll 1
    for (int ph = 0; ph < 3; ++ph) {
      const int J = ph == 1 ? O : H, K = ph == 0 ? I : ph == 1 ? H : O;
      const int sk = ph == 0 ? H : ph == 1 ? LO : 1, sj = ph == 2 ? LO : 1;
      const float* const a = ph == 0 ? X + row * I : ph == 1 ? G + row * H : D + row * LO;
      int per = 8;  // lanes of different j; where J leaves lanes over, several share the k of one
      while (per < J && per < 64) per <<= 1;
#pragma unroll 1
      for (int tang = WPS == 2 ? wave & 1 : 0; tang < (WPS == 2 ? (wave & 1) + 1 : 2); ++tang) {
        const float* const u = ph == 0 ? (tang ? w1t : w1) : (tang ? w2t : w2);
        const float* const a2 = !tang || ph == 0 ? nullptr : ph == 1 ? E + row * H : Dt + row * LO;
        const float* const bias = ph == 0 ? (tang ? b1t : b1) : (tang ? b2t : b2);
        float* const dst = ph == 0 ? (tang ? Ft : G) + row * H : ph == 1 ? (tang ? Zt : Z) + row * LO : (tang ? Et : E) + row * H;
        for (int j = lane & (per - 1); j < ((J + per - 1) & -per); j += per) {
          float s = 0.f;
          if (j < J) s = lds_dot(a, u + j * sj, a2, w2 + j * sj, sk, lane / per, 64 / per, K);
          if (per <= 32) s += lane_across<32>(s);
          if (per <= 16) s += lane_across<16>(s);
          if (per <= 8) s += lane_across<8>(s);
          if (lane < per && j < J) {
            if (ph < 2) s += bias[j];
            if (ph == 0 && !tang) s = tanhf(s);
            dst[j] = s;
          }
        }
      }
      __syncthreads();
      if (ph == 1) {
        if (first_wave) {
          const int y = in ? p.labels[gr] : -1;
          const bool valid = y >= 0 && y < O;
          const float *z = Z + row * LO, *zt = Zt + row * LO;
          float m = -INFINITY;
          for (int o = lane; o < O; o += 64) m = fmaxf(m, z[o]);
          m = wave_max_f(m);
          float se = 0.f, sd = 0.f;
          for (int o = lane; o < O; o += 64) {
            const float e = __expf(z[o] - m);
            se += e;
            sd = fmaf(e, zt[o], sd);
          }
          se = lanes_sum<1>(se);
          sd = lanes_sum<1>(sd);
          const float inv = 1.f / se, pz = sd * inv;
          for (int o = lane; o < O; o += 64) {
            const float pv = __expf(z[o] - m) * inv;
            D[row * LO + o] = valid ? (pv - (o == y ? 1.f : 0.f)) * invN : 0.f;
            Dt[row * LO + o] = valid ? pv * (zt[o] - pz) * invN : 0.f;
          }
          if (valid && lane == 0) loss += (double)(logf(se) + m - z[y]);
        }
      } else {
        for (int j = t; j < MLP_ROWS * H; j += MLP_THREADS) {
          const float g = G[j], g1 = 1.f - g * g, ft = Ft[j];
          if (ph == 2) Et[j] = g1 * Et[j] - 2.f * g * g1 * ft * E[j];
          E[j] = g1 * ft;
        }
      }
      __syncthreads();
    }
    // the blocks of H v as sums over the rows of x y (+ x' y')
#pragma unroll 1
    for (int j = t; j < n; j += MLP_THREADS) {
      const float *x = &one, *y, *x2 = nullptr, *y2 = nullptr;
      int sx = 0, sy = H;
      if (j < IH) {
        const int i = j / H;
        x = X + i; sx = I;
        y = Et + (j - i * H);
      } else if (j < IH + H) {
        y = Et + (j - IH);
      } else if (j < IH + H + HO) {
        const int q = j - IH - H, h = q / O, o = q - h * O;
        x = E + h; sx = H; y = D + o; sy = LO;
        x2 = G + h; y2 = Dt + o;
      } else {
        y = Dt + (j - IH - H - HO); sy = LO;
      }
      float s = acc[j];
#pragma unroll
      for (int r = 0; r < MLP_ROWS; ++r) s = fmaf(x[r * sx], y[r * sy], s);
      if (x2) {
#pragma unroll
        for (int r = 0; r < MLP_ROWS; ++r) s = fmaf(x2[r * H], y2[r * LO], s);
      }
      acc[j] = s;
    }
  }
  if (first_wave && lane == 0) rowloss[row] = loss;
  for (int j = t; j < n; j += MLP_THREADS) p.part[(int64_t)blockIdx.x * n + j] = acc[j];
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
    for (int r = 0; r < MLP_ROWS; ++r) s += rowloss[r];
    p.part_loss[blockIdx.x] = s;
  }
}

// The loss of a product, by one wave: the blocks' shares of it, and what the host reads.
__device__ __forceinline__ void mlp_loss(const double* part_loss, int nblk, const int* flags, double weight, int accumulate, double* loss, double* host) {
  const int lane = threadIdx.x & 63;
  double l = 0.0;
  for (int b = lane; b < nblk; b += 64) l += part_loss[b];
  l = wave_sum_d(l);
  if (lane == 0) {
    l = (accumulate ? loss[0] : 0.0) + weight * l / (double)max(1, flags[1]);
    loss[0] = l;
    host[0] = (double)flags[0]; host[1] = (double)flags[1]; host[2] = l;
  }
}

// H v = sum of the blocks' shares (+ what out holds); block 0 also the loss.  A block takes 32 elements; its eight groups of
// 32 lanes add every eighth share each and meet in LDS, always in the same order.
__global__ __launch_bounds__(256) void mlp_sum_kernel(const float* __restrict__ part, const double* __restrict__ part_loss, int nblk,
                                                      int n, const int* __restrict__ flags, double weight, int accumulate,
                                                      float* __restrict__ out, double* __restrict__ loss, double* __restrict__ host) {
  __shared__ double red[8][32];
  const int t = threadIdx.x, lane = t & 31, grp = t >> 5;
  const int j = blockIdx.x * 32 + lane;
  double s = 0.0;
  if (j < n) {
#pragma unroll 8
    for (int b = grp; b < nblk; b += 8) s += (double)part[(int64_t)b * n + j];
  }
  red[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && j < n) {
    s = accumulate ? (double)out[j] : 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) s += red[g][lane];
    out[j] = (float)s;
  }
  if (blockIdx.x == 0 && t >= 64 && t < 128) mlp_loss(part_loss, nblk, flags, weight, accumulate, loss, host);
}

// The sum of few shares and the Lanczos update behind it, by one block.
__global__ __launch_bounds__(1024) void mlp_sum_update_kernel(const float* __restrict__ part, const double* __restrict__ part_loss, int nblk,
                                                              const int* __restrict__ flags, double weight, double* __restrict__ loss,
                                                              double* __restrict__ host, LzSmall u) {
  extern __shared__ double sm_c[];  // [nq + 1] coefficients (full), then w
  float* const w = (float*)(sm_c + (u.full ? u.nq + 1 : 0));
  __shared__ double red[16];
  if (u.chained && u.scal[S_STOP] != 0.0) return;
  const int t = threadIdx.x, n = u.n, f0 = flags[0], f1 = flags[1];
  for (int j = t; j < n; j += 1024) {
    double g[8] = {}, s = 0.0;  // in the order of mlp_sum_kernel: runs and single steps agree bit for bit
    int b = 0;
#pragma unroll 2
    for (; b + 8 <= nblk; b += 8)
#pragma unroll
      for (int q = 0; q < 8; ++q) g[q] += (double)part[(int64_t)(b + q) * n + j];
#pragma unroll
    for (int q = 0; q < 7; ++q)
      if (b + q < nblk) g[q] += (double)part[(int64_t)(b + q) * n + j];
#pragma unroll
    for (int q = 0; q < 8; ++q) s += g[q];
    w[j] = (float)s;
  }
  if (t >= 960) mlp_loss(part_loss, nblk, flags, weight, 0, loss, host);
  __syncthreads();
  if (u.full) lz_small_full_block(u, w, sm_c, red, f0, f1);
  else lz_small_three_block(u, w, red, f0, f1);
}

int mlp_blocks(int B) { return std::min(MLP_BLOCKS, (B + MLP_ROWS - 1) / MLP_ROWS); }

// 150 of the 160 KB of LDS.
bool mlp_fused_fits(const hf_model_desc& d) {
  return d.param_dtype == HF_F32 && mlp_lds_floats(d.mlp_in, d.mlp_hidden, d.mlp_out, MLP_ROWS) * 4 <= 150 * 1024;
}

}  // namespace hf

using namespace hf;

int hf_ctx::hvp_mlp_fused(const float* params, const float* inputs, const int32_t* labels, int B, const float* v, float* out,
                          hipStream_t st) {
  MlpP p;
  p.params = params; p.v = v; p.x = inputs; p.labels = labels;
  p.B = B; p.I = desc.mlp_in; p.H = desc.mlp_hidden; p.O = desc.mlp_out;
  p.seed = seed; p.accumulate = acc_mode; p.part = mlp_part; p.part_loss = mlp_part_loss; p.flags = flags;
  const int nb = mlp_blocks(B);
  constexpr int LDS_MAX = 150 * 1024;
  // Several turns a block: one wave a sample where LDS has room for sixteen (figures above; with two waves 32-32-10 at 16384 samples 81, 64-64-10
  // 112, 8-8-2 67).
  const int64_t lds16 = mlp_lds_floats(p.I, p.H, p.O, 2 * MLP_ROWS) * 4, lds8 = mlp_lds_floats(p.I, p.H, p.O, MLP_ROWS) * 4;
  const bool one_wave = B > MLP_BLOCKS * MLP_ROWS && lds16 <= LDS_MAX;
  static OncePerDevice once1, once2;
  hipError_t e = one_wave ? once1.lds_limit((const void*)mlp_hvp_kernel<1>, LDS_MAX) : once2.lds_limit((const void*)mlp_hvp_kernel<2>, LDS_MAX);
  if (e == hipSuccess) {
    if (one_wave) hipLaunchKernelGGL(mlp_hvp_kernel<1>, dim3(nb), dim3(MLP_THREADS), (size_t)lds16, st, p);
    else hipLaunchKernelGGL(mlp_hvp_kernel<2>, dim3(nb), dim3(MLP_THREADS), (size_t)lds8, st, p);
    if (then_update && !acc_mode && nb * n <= MLP_ADD_IN_UPDATE) {
      hipLaunchKernelGGL(mlp_sum_update_kernel, dim3(1), dim3(1024), (size_t)then_update->lds(), st, mlp_part, mlp_part_loss, nb, flags,
                         (double)seed, loss_dev, host_hvp, *then_update);
      then_update = nullptr;
    } else
      hipLaunchKernelGGL(mlp_sum_kernel, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, mlp_part, mlp_part_loss, nb, (int)n, flags,
                       (double)seed, acc_mode, out, loss_dev, host_hvp);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return fail(HF_EDEVICE, std::string("hvp_mlp_fused: ") + hipGetErrorString(e));
  return HF_OK;
}
