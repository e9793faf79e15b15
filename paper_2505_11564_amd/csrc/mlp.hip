// The Hessian-vector product of the tanh MLP as one launch and a sum, for fp32 models whose weights fit a CU's LDS.
//
// What bounds it: nothing but latency (the 32-32-10 model at 256 samples is 5 MFLOP and 11 KB of weights): as a
// chain of products and pointwise kernels it was 15 launches of 1.5 to 13 us, each waiting for the one before.  The samples
// are independent, so a block takes its own through the forward, loss and backward sweeps with their tangents in LDS and
// leaves its share of H v (n floats) in the workspace; a second kernel adds the blocks' shares in a fixed order.
// Measured at that shape: 13 + 4 us for the two, against 62 us of kernels in 15 launches (with the products of
// gemm_f32.hip); an iteration of a run 33 us, 136 before.
// Blocks: one per eight samples up to one per CU (the largest weights take a CU's LDS), then several turns each.  With at most
// 64 blocks, whatever the batch, a large one lost to the chain of products.  hf_hvp, us (chain / 64 blocks / 256 blocks and the
// sum spread over eight groups of lanes): 128-64-10 at 256 samples 97 / 55 / 54, 2048 138 / 134 / 62, 16384 451 / 839 / 250, 65536
// 1553 / - / 917; 32-32-10 88 / 34 / 33, 124 / 58 / 34, 428 / 269 / 94, 1493 / - / 292; 100-70-31 118 / 64 / 62, 202 / 159 /
// 68, 852 / 1029 / 297, 3093 / - / 1102.  Larger batches (MLP_FUSED_MAX_BATCH) have not been measured and take the chain.
//   f = x W1 + b1, g = tanh f, z = g W2 + b2, p = softmax z, and along v:
//   f_t = x W1_t + b1_t, g_t = g' f_t, z_t = g_t W2 + g W2_t + b2_t
//   dz = (p - onehot) s, dz_t = p (z_t - <p, z_t>) s;  dg = dz W2^T, dg_t = dz_t W2^T + dz W2_t^T
//   da_t = g' dg_t + g'' f_t dg,  g' = 1 - g^2, g'' = -2 g g'
//   (Hv)_W2 = g_t^T dz + g^T dz_t, (Hv)_b2 = sum dz_t, (Hv)_W1 = x^T da_t, (Hv)_b1 = sum da_t
#include "engine.h"

#include <algorithm>
#include <cmath>

namespace hf {

constexpr int MLP_ROWS = 8;  // samples a block works on at a time: 32 lanes each

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
__host__ __device__ inline int64_t mlp_lds_floats(int64_t I, int64_t H, int64_t O) {
  const int64_t LO = O | 1;
  return 2 * (I * H + H + H * LO + O) + (I * H + H + H * O + O) + MLP_ROWS * (I + 4 * H + 4 * LO);
}

__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 32);
  return v;
}
__device__ __forceinline__ float half_max(float v) {
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 32));
  return v;
}

__global__ __launch_bounds__(256) void mlp_hvp_kernel(MlpP p) {
  extern __shared__ float sm[];
  const int t = threadIdx.x, I = p.I, H = p.H, O = p.O, LO = O | 1, IH = I * H, HO = H * O, n = IH + H + HO + O;
  float* w1 = sm;        float* w1t = w1 + IH;
  float* b1 = w1t + IH;  float* b1t = b1 + H;
  float* w2 = b1t + H;   float* w2t = w2 + H * LO;
  float* b2 = w2t + H * LO; float* b2t = b2 + O;
  float* acc = b2t + O;
  float* X = acc + n;                                              // [rows][I]
  float* G = X + MLP_ROWS * I;    float* Gt = G + MLP_ROWS * H;    // g, g_t
  float* Ft = Gt + MLP_ROWS * H;  float* At = Ft + MLP_ROWS * H;   // f_t, da_t
  float* Z = At + MLP_ROWS * H;   float* Zt = Z + MLP_ROWS * LO;   // z, z_t
  float* D = Zt + MLP_ROWS * LO;  float* Dt = D + MLP_ROWS * LO;   // dz, dz_t
  __shared__ int cnt[4], bad[4];
  __shared__ double rowloss[MLP_ROWS];

  const int row = t >> 5, lane = t & 31;  // each half wave owns one sample
  // all loads of the start are independent and in flight together: weights, direction, labels, the first samples
  const int r_first = blockIdx.x * MLP_ROWS;
  for (int i = lane; i < I; i += 32) X[row * I + i] = r_first + row < p.B ? p.x[(int64_t)(r_first + row) * I + i] : 0.f;
#pragma unroll 8
  for (int j = t; j < n; j += 256) {
    const float w = p.params[j], d = p.v[j];
    float *dst = w1 + j, *dst_t = w1t + j;
    if (j >= IH) {
      if (j < IH + H) { dst = b1 + (j - IH); dst_t = b1t + (j - IH); }
      else if (j < IH + H + HO) {
        const int q = j - IH - H, h = q / O, at = h * LO + q - h * O;
        dst = w2 + at; dst_t = w2t + at;
      } else { dst = b2 + (j - IH - H - HO); dst_t = b2t + (j - IH - H - HO); }
    }
    *dst = w;
    *dst_t = d;
    acc[j] = 0.f;
  }
  // every block counts the valid labels of the whole batch itself
  int c = 0, b = 0;
  for (int i = t; i < p.B; i += 256) {
    const int y = p.labels[i];
    c += (y >= 0);
    b |= (y >= O);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { c += __shfl_xor(c, o, 64); b |= __shfl_xor(b, o, 64); }
  if ((t & 63) == 0) { cnt[t >> 6] = c; bad[t >> 6] = b; }
  __syncthreads();
  const int nv = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  if (blockIdx.x == 0 && t == 0) {
    const int bits = ((bad[0] | bad[1] | bad[2] | bad[3]) ? 2 : 0) | (nv == 0 ? 4 : 0);
    p.flags[0] = p.accumulate ? (p.flags[0] | bits) : bits;
    p.flags[1] = nv;
  }
  const float invN = p.seed / (float)max(1, nv);
  double loss = 0.0;
  for (int r0 = r_first; r0 < p.B; r0 += gridDim.x * MLP_ROWS) {
    const int gr = r0 + row;
    const bool in = gr < p.B;
    if (r0 != r_first) {
      __syncthreads();  // the products of the previous samples are done with the row buffers
      for (int i = lane; i < I; i += 32) X[row * I + i] = in ? p.x[(int64_t)gr * I + i] : 0.f;
      __syncthreads();
    }
    for (int h = lane; h < H; h += 32) {
      float f = b1[h], ft = b1t[h];
#pragma unroll 8
      for (int i = 0; i < I; ++i) {
        const float xv = X[row * I + i];
        f = fmaf(xv, w1[i * H + h], f);
        ft = fmaf(xv, w1t[i * H + h], ft);
      }
      const float g = tanhf(f);
      G[row * H + h] = g;
      Ft[row * H + h] = ft;
      Gt[row * H + h] = (1.f - g * g) * ft;
    }
    __syncthreads();
    const int y = in ? p.labels[gr] : -1;
    const bool valid = y >= 0 && y < O;
    float m = -INFINITY;
    for (int o = lane; o < O; o += 32) {
      float z = b2[o], zt = b2t[o];
#pragma unroll 8
      for (int h = 0; h < H; ++h) {
        const float g = G[row * H + h], w = w2[h * LO + o];
        z = fmaf(g, w, z);
        zt = fmaf(Gt[row * H + h], w, zt);
        zt = fmaf(g, w2t[h * LO + o], zt);
      }
      Z[row * LO + o] = z;
      Zt[row * LO + o] = zt;
      m = fmaxf(m, z);
    }
    m = half_max(m);
    float se = 0.f, sd = 0.f;
    for (int o = lane; o < O; o += 32) {
      const float e = __expf(Z[row * LO + o] - m);
      se += e;
      sd = fmaf(e, Zt[row * LO + o], sd);
    }
    se = half_sum(se);
    sd = half_sum(sd);
    const float inv = 1.f / se, pz = sd * inv;
    for (int o = lane; o < O; o += 32) {
      const float pv = __expf(Z[row * LO + o] - m) * inv;
      D[row * LO + o] = valid ? (pv - (o == y ? 1.f : 0.f)) * invN : 0.f;
      Dt[row * LO + o] = valid ? pv * (Zt[row * LO + o] - pz) * invN : 0.f;
    }
    __syncthreads();
    if (valid && lane == 0) loss += (double)(logf(se) + m - Z[row * LO + y]);
    for (int h = lane; h < H; h += 32) {
      float dg = 0.f, dgt = 0.f;
#pragma unroll 8
      for (int o = 0; o < O; ++o) {
        const float d = D[row * LO + o], w = w2[h * LO + o];
        dg = fmaf(d, w, dg);
        dgt = fmaf(Dt[row * LO + o], w, dgt);
        dgt = fmaf(d, w2t[h * LO + o], dgt);
      }
      const float g = G[row * H + h], g1 = 1.f - g * g;
      At[row * H + h] = g1 * dgt - 2.f * g * g1 * Ft[row * H + h] * dg;
    }
    __syncthreads();
    for (int j = t; j < n; j += 256) {
      float s = acc[j];
      if (j < IH) {
        const int i = j / H, h = j - i * H;
#pragma unroll
        for (int r = 0; r < MLP_ROWS; ++r) s = fmaf(X[r * I + i], At[r * H + h], s);
      } else if (j < IH + H) {
#pragma unroll
        for (int r = 0; r < MLP_ROWS; ++r) s += At[r * H + j - IH];
      } else if (j < IH + H + HO) {
        const int q = j - IH - H, h = q / O, o = q - h * O;
#pragma unroll
        for (int r = 0; r < MLP_ROWS; ++r) {
          s = fmaf(Gt[r * H + h], D[r * LO + o], s);
          s = fmaf(G[r * H + h], Dt[r * LO + o], s);
        }
      } else {
#pragma unroll
        for (int r = 0; r < MLP_ROWS; ++r) s += Dt[r * LO + j - IH - H - HO];
      }
      acc[j] = s;
    }
  }
  if (lane == 0) rowloss[row] = loss;
  for (int j = t; j < n; j += 256) p.part[(int64_t)blockIdx.x * n + j] = acc[j];
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
    for (int r = 0; r < MLP_ROWS; ++r) s += rowloss[r];
    p.part_loss[blockIdx.x] = s;
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
  if (blockIdx.x == 0 && t >= 64 && t < 128) {
    double l = 0.0;
    for (int b = t - 64; b < nblk; b += 64) l += part_loss[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
    if (t == 64) {
      l = (accumulate ? loss[0] : 0.0) + weight * l / (double)max(1, flags[1]);
      loss[0] = l;
      host[0] = (double)flags[0]; host[1] = (double)flags[1]; host[2] = l;
    }
  }
}

int mlp_blocks(int B) { return std::min(MLP_BLOCKS, (B + MLP_ROWS - 1) / MLP_ROWS); }

// 150 of the 160 KB of LDS.
bool mlp_fused_fits(const hf_model_desc& d) {
  return d.param_dtype == HF_F32 && mlp_lds_floats(d.mlp_in, d.mlp_hidden, d.mlp_out) * 4 <= 150 * 1024;
}

}  // namespace hf

using namespace hf;

int hf_ctx::hvp_mlp_fused(const float* params, const float* inputs, const int32_t* labels, int B, const float* v, float* out,
                          hipStream_t st) {
  MlpP p;
  p.params = params; p.v = v; p.x = inputs; p.labels = labels;
  p.B = B; p.I = desc.mlp_in; p.H = desc.mlp_hidden; p.O = desc.mlp_out;
  p.seed = seed; p.accumulate = acc_mode; p.part = mlp_part; p.part_loss = mlp_part_loss; p.flags = flags;
  const int lds = (int)(mlp_lds_floats(p.I, p.H, p.O) * 4), nb = mlp_blocks(B);
  static OncePerDevice once;
  hipError_t e = once.lds_limit((const void*)mlp_hvp_kernel, 150 * 1024);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(mlp_hvp_kernel, dim3(nb), dim3(256), lds, st, p);
    hipLaunchKernelGGL(mlp_sum_kernel, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, mlp_part, mlp_part_loss, nb, (int)n, flags,
                       (double)seed, acc_mode, out, loss_dev, host_hvp);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return fail(HF_EDEVICE, std::string("hvp_mlp_fused: ") + hipGetErrorString(e));
  return HF_OK;
}
