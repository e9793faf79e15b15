// One matrix product as the engine launches it, the launchers' choices and those of an orthogonalisation, behind C entries: what the tests of
// single products and of rules call.
// Not part of the API.
#include "gemm_params.h"
#include "hf_internal.h"
#include "lanczos.h"

// ptr: A[3], B[3], C, C_lo, Cadd, At, Bt, Ct, Cadd_t, ws, counters (device memory; nullptr where absent).
// num: M, N, K, lda, ldb, ldc, transA, transB, in_bf16, out_bf16, klimit, elements of ws, force_cfg, force_ks.
// Returns the launch's hipError_t.
extern "C" __attribute__((visibility("default"))) int hf_internal_product(void* const* ptr, const int64_t* num, float alpha, void* stream) {
  if (!ptr || !num) return (int)hipErrorInvalidValue;
  for (int i = 0; i < 6; ++i)
    if (num[i] < 1 || num[i] > (int64_t)1 << 30) return (int)hipErrorInvalidValue;
  hf::Gemm g;
  for (int i = 0; i < 3; ++i) { g.A[i] = ptr[i]; g.B[i] = ptr[3 + i]; }
  g.C = ptr[6]; g.C_lo = ptr[7]; g.Cadd = (const float*)ptr[8];
  g.At = ptr[9]; g.Bt = ptr[10]; g.Ct = ptr[11]; g.Cadd_t = (const float*)ptr[12];
  g.ws = (float*)ptr[13]; g.counters = (int*)ptr[14];
  g.M = (int)num[0]; g.N = (int)num[1]; g.K = (int)num[2];
  g.lda = num[3]; g.ldb = num[4]; g.ldc = num[5];
  g.transA = (int)num[6]; g.transB = (int)num[7];
  g.in_bf16 = (int)num[8]; g.out_bf16 = (int)num[9]; g.klimit = (int)num[10];
  g.ws_elems = num[11]; g.force_cfg = (int)num[12]; g.force_ks = (int)num[13];
  g.alpha = alpha;
  if (g.lda < (g.transA ? g.M : g.K) || g.ldb < (g.transB ? g.K : g.N) || g.ldc < g.N) return (int)hipErrorInvalidValue;
  return (int)hf::launch_gemm(g, (hipStream_t)stream);
}

// Tile and parts of k of a bf16 product with its tangent: M, N, K, transA, transB, low-order terms (0, 1, 2), out_bf16, addends (0, 1),
// elements of ws.  Returns tile + 16 parts, -1 for two products of 256 x 256 tiles in one launch.
extern "C" __attribute__((visibility("default"))) int hf_internal_linear_plan(const int64_t* num) {
  static float none;
  hf::Gemm g;
  g.M = (int)num[0]; g.N = (int)num[1]; g.K = (int)num[2];
  g.transA = (int)num[3]; g.transB = (int)num[4];
  g.A[0] = &none;
  for (int i = 0; i < num[5] && i < 2; ++i) g.A[1 + i] = &none;
  g.in_bf16 = 1; g.out_bf16 = (int)num[6];
  if (num[7]) g.Cadd = g.Cadd_t = &none;
  g.ws_elems = num[8];
  if (num[8] > 0) g.ws = (float*)(uintptr_t)4096;  // (aligned; only looked at)
  int parts;
  const int tile = hf::linear_plan(g, &parts);
  return tile < 0 ? -1 : tile + 16 * parts;
}

// Tile of n fp32 products launched together (M, N, K, terms of each in num), and the parts of each one's k.
extern "C" __attribute__((visibility("default"))) int hf_internal_f32_plan(const int64_t* num, int n, int64_t ws_elems, int* parts) {
  if (n < 1 || n > hf::F32_GROUP_MAX) return -1;
  hf::GemmP ps[hf::F32_GROUP_MAX] = {};
  for (int i = 0; i < n; ++i) {
    ps[i].M = (int)num[4 * i]; ps[i].N = (int)num[4 * i + 1]; ps[i].K = (int)num[4 * i + 2]; ps[i].nterm = (int)num[4 * i + 3];
  }
  return hf::f32_plan(ps, n, 1, ws_elems, parts);
}

// What the first orthogonalisation pass decides: a, p, ww, others, sum, most, gkk, gpp, gkp of LzFirst and a tolerance; before and est into out.
extern "C" __attribute__((visibility("default"))) void hf_internal_lz_first_plan(const double* in, double* out) {
  const hf::LzFirst s = {in[0], in[1], in[2], in[3], in[4], in[5], in[6], in[7], in[8]};
  const hf::LzFirstPlan plan = hf::lz_first_plan(s, in[9]);
  out[0] = plan.before;
  out[1] = plan.est;
}
