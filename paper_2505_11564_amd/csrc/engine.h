// Context of libhessformer_hip: model description, canonical layout, device
// workspace, and the host-side schedules of the Hessian-vector product
// (Algorithm 1 of the paper, evaluated forward-over-reverse) and of the
// Lanczos iteration (Algorithm 2).
#pragma once

#include "hf_internal.h"
#include "lanczos.h"

namespace hf {

struct LayoutEntry {
  std::string name;
  int64_t offset;
  int64_t shape[2];
  int64_t count() const { return shape[0] * (shape[1] ? shape[1] : 1); }
};

// Fills `out` with the canonical flat order; returns HF_OK or HF_EINVAL.
int build_layout(const hf_model_desc& d, std::vector<LayoutEntry>& out, std::string* why);

// Offsets (elements) of one transformer layer's tensors in the flat vector.
struct LayerOff {
  int64_t n1g = -1, n1b = -1, wqkv = -1, bqkv = -1, wq = -1, wk = -1, wv = -1, wo = -1, bo = -1;
  int64_t n2g = -1, n2b = -1, wfc = -1, bfc = -1, wproj = -1, bproj = -1, wgate = -1, wup = -1, wdown = -1;
};

// Device buffers of one layer kept from the forward pass for the backward
// pass (each with its tangent twin `*_t`).
struct LayerBuf {
  float *x1, *x1_t, *x2, *x2_t, *st1, *st2;          // residual stream, norm statistics
  void *a, *a_t, *qkv, *qkv_t, *P, *P_t, *o, *o_t;   // attention branch
  void *m, *m_t, *f, *f_t, *g, *g_t;                 // MLP branch: norm out, pre-activation, activation out
  void *up, *up_t;                                   // LLAMA: up projection (f = gate)
  // streamed attention (bf16, head width 32 / 64 / 128): the backward sweep recomputes the scores,
  // so each layer keeps the low-order halves of q | k | v and of the attention output, and the
  // row statistics (m + log l, r) of its softmax
  void *qkv_lo, *o_lo;
  float* att_stat;
};

// Adjoints (with tangents) that the weight-gradient products of a layer read: of its output (x) and between its two branches
// (m; operand-type copies), of the activation's input(s), of the packed q | k | v, and of v apart from them (stored attention, grouped
// heads).  The products of several layers may run as one launch, so there are several of these (dw_layers).
struct AdjBuf {
  void *x, *x_t, *m, *m_t, *g, *g_t, *up, *up_t, *qkv, *qkv_t, *v, *v_t;
};

// mlp.hip: MLP products whose weights fit LDS run in one kernel of at most MLP_BLOCKS blocks, each of which leaves a
// partial result.
constexpr int MLP_BLOCKS = 256, MLP_FUSED_MAX_BATCH = 65536;
bool mlp_fused_fits(const hf_model_desc& d);
int mlp_blocks(int B);

}  // namespace hf

struct hf_ctx {
  hf_model_desc desc;
  int device = 0;
  int max_batch = 0, max_m = 0;
  int bf = 0;  // 1: bf16 parameters / operands
  int flash = 0;  // 1: attention runs in the streamed kernels (no S x S buffers are allocated)
  int pairs = 0;  // 1: bf16 primal activations are carried as (rounded value, remainder) pairs; the *_lo buffers exist
  int64_t n = 0;
  std::vector<hf::LayoutEntry> layout;
  std::vector<hf::LayerOff> loff;
  int64_t off_wte = -1, off_wpe = -1, off_nfg = -1, off_nfb = -1, off_head = -1;
  int64_t off_w1 = -1, off_b1 = -1, off_w2 = -1, off_b2 = -1;
  std::vector<std::pair<int64_t, int64_t>> zero_ranges;  // H v regions filled by atomics
  int64_t layers_begin = 0, layers_end = 0;  // the layers' parameters (through the final norm) in the flat vector
  int dw_prezeroed = 0;  // this product cleared [layers_begin, layers_end) of H v in one pass
  std::string err;

  // device memory
  char* arena = nullptr;
  int64_t arena_bytes = 0;
  std::vector<hf::LayerBuf> lb;
  hf::bf16* vb = nullptr;  // bf16 copy of the direction (bf16 mode)
  const float* vb_of = nullptr;  // the Lanczos vector whose bf16 copy vb_cur holds (written by the update), or nullptr
  const hf::bf16* vb_cur = nullptr;   // the bf16 copy the running product multiplies with: vb, or a row of a bf16 basis
  const hf::bf16* next_vb = nullptr;  // scratch of lanczos_update
  float *xL = nullptr, *xL_t = nullptr, *stf = nullptr;
  void *xf = nullptr, *xf_t = nullptr, *xf_lo = nullptr;
  // bf16 mode: low-order halves of the primal forward activations (reused by every layer)
  void *a_lo = nullptr, *qkv_lo = nullptr, *P_lo = nullptr, *o_lo = nullptr, *f_lo = nullptr, *up_lo = nullptr, *g_lo = nullptr;
  float *rq = nullptr, *rq_t = nullptr;  // LLAMA: fp32 q|k (or their adjoints) before the rotation
  float *rv = nullptr, *rv_t = nullptr;  // grouped-query attention: fp32 dV summed over the heads of a group
  float *z = nullptr, *z_t = nullptr;
  void *dz = nullptr, *dz_t = nullptr;
  int64_t ldz = 0;
  float* loss_rows = nullptr;
  float *sc = nullptr, *sc_t = nullptr;
  float* norm_part = nullptr;  // per-block column sums of the norm backward kernels
  float *att_part = nullptr, *att_rstat = nullptr;  // row statistics of the fused attention epilogues
  int64_t att_SS = 0;                                 // elements of one score-shaped buffer
  int att_zero_B = -1, att_zero_S = -1;               // shape for which the never-written score tiles were last cleared
  void *dS = nullptr, *dS_t = nullptr;
  float *dx = nullptr, *dx_t = nullptr, *tmpd = nullptr, *tmpd_t = nullptr;
  void *dob = nullptr, *dob_t = nullptr, *dy = nullptr, *dy_t = nullptr;
  std::vector<hf::AdjBuf> adj;  // layer l's are adj[l % adj.size()]; those beyond the first lie in adj_arena
  char* adj_arena = nullptr;
  int64_t adj_bytes = 0;
  void drop_waiting();  // back to one: weight-gradient products then never wait beyond their layer
  float* mlp_part = nullptr;  // MLP products in one kernel: the blocks' shares of H v and of the loss; nullptr = not that size
  double* mlp_part_loss = nullptr;
  void* xin = nullptr;  // MLP input in operand type (bf16 mode)
  int* flags = nullptr;  // [0] error bits, [1] number of valid labels
  double* loss_dev = nullptr;
  double* host_hvp = nullptr;  // pinned: error bits, number of valid labels and loss of the last product
  unsigned long long* stats_dev = nullptr;  // column statistics counters
  float* gemm_ws = nullptr;  // fp32 scratch of products with a cut k
  int64_t gemm_ws_elems = 0;
  int* gemm_cnt = nullptr;   // fp32 parameters: arrival counters of those products (F32_COUNTERS, zero between launches)
  int gemm_cnt_clear = 0;    // the first product has cleared them
  float* aux_vec = nullptr;  // n floats, allocated on first use (the unit vector of a Hessian column)
  int dw_layers() const;  // layers whose weight-gradient products may wait for a common launch
  int clear_padding(int T, hipError_t* er, hipStream_t st);
  int pad_T = -1;  // number of tokens behind which those rows are zero
  int ensure_aux();

  // Lanczos state
  // Working vectors.  With an fp32 basis and full orthogonalisation the basis rows k and k - 1 are
  // q_k and q_{k-1} themselves (cur_q / prev_q) and lz_vec holds only r and, once the basis is
  // full, the last q; otherwise lz_vec rotates q, q_prev and r.
  float* lz_vec[3] = {nullptr, nullptr, nullptr};
  float* lz_hq = nullptr;  // short vectors: the products of a run that the host enqueues ahead, so that r stays the last iteration's
  int iq = 0, iqp = 1, ir = 2;
  void* basis = nullptr;
  // bf16 copies of the rows of an fp32 basis, kept by contexts with bf16 parameters: row k is the
  // operand-type copy of q_k that the product multiplies with anyway, and the subtraction pass of
  // the orthogonalisation reads rows 0 .. k-2 from here at half the bytes (their coefficients are
  // at rounding level, so the rounding of the copies is below that of the fp32 result)
  hf::bf16* basis_bf = nullptr;
  int64_t ldq = 0;
  double *scal = nullptr, *cvec = nullptr, *partials = nullptr;
  double* host_scal = nullptr;  // pinned, LZ_AHEAD slots of S_COUNT doubles; host_hvp and host_stats follow
  unsigned long long* host_stats = nullptr;  // and the sums of the column statistics
  int host_slot = -1;           // its slot of the shared block, or -1: this context's own
  void release_host();
  hipEvent_t ahead_ev[hf::LZ_AHEAD] = {};  // one per slot, created by the first run with short vectors
  int lz_k = -1;                // iterations done; -1 = not initialised
  int lz_reorth = 0;
  int lz_done = 0;
  double lz_beta_prev = 0.0;    // beta_{k-1}
  bool lz_r_is_q = false;       // the last update left no r: it is beta_{k-1} q_k
  bool lz_rows_are_vectors() const { return lz_reorth == HF_REORTH_FULL && desc.basis_dtype == HF_F32; }
  float* cur_q() const;         // q_k
  float* prev_q() const;        // q_{k-1} (meaningful for k >= 1)

  int fail(int code, const std::string& m) { err = m; return code; }
  int plan_and_alloc();
  // out = seed_scale * H v, or out += seed_scale * H v when accumulate (the batch loop of Algorithm 1:
  // the weight of a batch multiplies the adjoint seeds, in which the backward sweep is linear)
  int hvp_enqueue(const void* params, const void* inputs, const int32_t* labels, int batch, int seq, const float* v,
                  float* out, hipStream_t st, float seed_scale = 1.f, int accumulate = 0);
  int acc_mode = 0;   // the product being enqueued adds to out
  float seed = 1.f;   // and scales its adjoint seeds by this
  int hvp_mlp(const void* params, const void* inputs, const int32_t* labels, int B, const float* v, float* out,
              hipStream_t st);
  int hvp_mlp_fused(const float* params, const float* inputs, const int32_t* labels, int B, const float* v, float* out,
                    hipStream_t st);
  int hvp_transformer(const void* params, const int32_t* tok, const int32_t* labels, int B, int S, const float* v,
                      float* out, hipStream_t st);
  int finish_hvp(double* loss_host, hipStream_t st);
  // Iterations 0 .. m-1 of a run with short vectors (lz_small), enqueued up to LZ_AHEAD ahead of their results; *done =
  // iterations finished.  HF_EBREAKDOWN as lanczos_update.
  int run_small(const void* params, const void* inputs, const int32_t* labels, int batch, int seq, int m, double tol, double* alpha,
                double* beta, int* done, hipStream_t st);
  // the small update of iteration lz_k (the residual, or without a basis H q_k itself, into r), scalars into slot `host`; false: vectors too long
  bool small_update(float* r, double tol, double* host, int chained, hf::LzSmall& u);
  const hf::LzSmall* then_update = nullptr;  // the update that follows the product being enqueued; taken (NULL again) by one that includes it
  // what a finished iteration k with norm bt leaves: true if the run goes on
  bool advance(int k, double bt, double tol);
  int flag_error(const double* host);
  // hvp_flags: the device flags of the product that made r (NULL when r came from the caller)
  int lanczos_update(float* r, double tol, double* alpha_k, double* beta_k, const int* hvp_flags, hipStream_t st);
};
