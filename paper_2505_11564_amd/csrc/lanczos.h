// Internal interface of the Lanczos vector kernels (lanczos.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "hf_internal.h"

namespace hf {

// Slots of the device-resident scalar array.
enum {
  S_ALPHA = 0,       // alpha_k
  S_BETA = 1,        // current ||r|| (beta_k once the iteration's updates are done)
  S_NRM_BEFORE = 3,  // ||r|| before the orthogonalisation pass in flight; -1.0 after a pass that wrote q_{k+1} itself: there is no r then
  S_REDO = 4,        // 1.0 when a second orthogonalisation pass is required
  S_Q0NORM = 5,      // ||q0|| before normalisation
  S_FLAG0 = 6,       // error bits and number of valid labels of the Hessian-vector product that made
  S_FLAG1 = 7,       //   w, copied here by the kernel that writes q_{k+1}
  S_STOP = 2,        // 1.0 once an iteration of a chained run (host ahead of the results) could not advance
  S_COUNT = 8,
  // device only
  S_EST = 8,         // > 0: the first orthogonalisation pass writes q_{k+1} itself, with this estimate of beta_k
  S_FIX = 9,         // what that q_{k+1} still has to be multiplied by; 1.0: nothing
  S_DEVICE = 10
};

constexpr int HF_MAX_M = 2000;  // most basis vectors a context may hold
constexpr int LZ_NBLK = 2048;  // upper bound on blocks (= partial sums per basis vector) of the re-orthogonalisation kernels
constexpr int LZ_NBLK_VEC = 16384;  // upper bound on blocks (= partial sums) of the read-only passes over one vector

hipError_t lz_norm_q0(const float* z, int64_t n, double* scal, double* partials, hipStream_t st);
// Iteration k of the three-term recurrence without a basis: alpha_k, beta_k into scal, and
// q_{k+1} = (w - beta_prev qp - alpha_k q) / beta_k written over qp (with its bf16 copy in vb, may be
// NULL) unless beta_k < tol or `flags` (device, may be NULL: [0] error bits, [1] valid labels)
// report a failed product.  partials: 3 * LZ_NBLK_VEC doubles.
hipError_t lz3_update(const float* w, const float* q, float* qp, bf16* vb, int64_t n, int use_prev, double beta_prev,
                      double tol, const int* flags, double* scal, double* partials, hipStream_t st);
// q_{k+1} = src / scal[idx] into dst (fp32, may be NULL), its basis row (may be NULL) and vb (bf16,
// may be NULL), under the same test.  idx = S_BETA after a pass that wrote q_{k+1} itself: only what S_FIX asks for.
hipError_t lz_scale(const float* src, float* dst, void* basis, int basis_bf16, bf16* vb, int64_t n, double* scal, int idx,
                    double tol, const int* flags, hipStream_t st);
// The second classical Gram-Schmidt pass, of r against Q[0..nq): a no-op unless the first set the redo flag.
// copies (optional, fp32 basis only): bf16 copies of the rows, same row stride; the subtraction
// reads rows 0 .. nq-3 from them.
hipError_t lz_gs_second_pass(const void* Q, int basis_bf16, const bf16* copies, int64_t ldq, float* r, int64_t n, int nq,
                             double* scal, double* c, double* partials, hipStream_t st);
// What the first orthogonalisation pass decides from c = Q^T w and a few products more (w = H q_k, Q = q_0 .. q_k).
struct LzFirst {
  double a, p;              // c_k = alpha_k, c_{k-1} (0 for k = 0)
  double ww;                // <w, w>
  double others, sum, most; // of the older rows: sum of c_j^2, sum of |c_j|, largest c_j^2
  double gkk, gpp, gkp;     // <q_k, q_k>; <q_{k-1}, q_{k-1}>, <q_k, q_{k-1}> (0 for k = 0)
};
// before: the norm that the three-term recurrence would have left, ||w - alpha_k q_k - c_{k-1} q_{k-1}||; the pass asks for a second one where it
// leaves less than 1 / sqrt(2) of that.  Where the difference has lost its digits (beta_k tiny against alpha_k) it is infinite, which makes
// the pass ask.  So it is where an older row has a coefficient above 1e-5 ||w|| and alpha_k > 2 beta_k: that may say that q_k has lost as much
// orthogonality, and what one pass leaves of it, alpha_k <q_k, q_j> / beta_k, then grows from iteration to iteration (a spectrum that
// keeps away from zero: 0.9 .. 1.0 lost the basis in five iterations).
// est: beta_k itself, ||w - Q c||, or 0.  ||w||^2 - sum c_j^2 (2 - <q_j, q_j>) + 2 c_k c_{k-1} <q_k, q_{k-1}> leaves out what the older rows' products with
// each other, with themselves beyond 1, and with q_k and q_{k-1} add: at most LZ_OFF times (sum |c_j|)^2 + 2 sum |c_j| (|c_k| + |c_{k-1}|), as no
// such product is off by more than LZ_OFF (rounding a row to bf16 moves it by 2^-9 of its length; rows of fp32 are a thousand times closer).
// In a run the c_j are rounding errors and the bound is far below the 1e-3 asked for.  Where beta_k less that bound is no small difference, and
// neither a second pass nor, with 1e-3 to spare for the fp32 sums in <w, w>, an end of the iteration is in sight, the pass divides by
// beta_k and writes q_{k+1} at once, over q_{k-1} if need be, which saves a vector's way to memory and back.
constexpr double LZ_OFF = 1.0 / 128.0;
struct LzFirstPlan { double before, est; };
__host__ __device__ inline LzFirstPlan lz_first_plan(const LzFirst& s, double tol) {
  const double rest = s.ww - s.a * s.a - s.p * s.p;
  const double b2 = s.ww - s.a * s.a * (2.0 - s.gkk) - s.others + 2.0 * s.a * s.p * s.gkp - s.p * s.p * (2.0 - s.gpp);
  const double low = b2 - LZ_OFF * s.sum * (s.sum + 2.0 * (fabs(s.a) + fabs(s.p)));
  const bool grows = s.most > 1e-10 * s.ww && s.a * s.a > 4.0 * b2;
  LzFirstPlan plan;
  plan.before = rest > 1e-5 * s.ww && !grows ? sqrt(rest) : INFINITY;
  const bool ok = low > 1e-3 * s.ww && sqrt(low) >= 0.7072 * plan.before && sqrt(low) >= 1.001 * tol;  // (false for NaN)
  plan.est = ok ? sqrt(b2) : 0.0;
  return plan;
}

// Where q_{k+1} goes (fp32; bf16, may be NULL), and the test that decides whether it may be written.
struct LzNext {
  float* q;
  bf16* qb;
  const int* flags;
  double tol;
};
// The first pass applied to w = H q_k itself against an fp32 basis holding q_0 .. q_k (nq = k + 1): also yields alpha_k.  Writes
// q_{k+1} instead of r where beta_k is known well enough beforehand (scal[S_EST] > 0).
// c: nq + 4 doubles, partials: (nq + 4) * LZ_NBLK.
hipError_t lz_gs_first_pass(const float* Q, const bf16* copies, int64_t ldq, float* r, int64_t n, int nq, const LzNext& next, double* scal,
                            double* c, double* partials, hipStream_t st);
// The same for a bf16 basis: q_k and q_{k-1} come from the fp32 working vectors, rows 0 .. k-2 from the basis.
hipError_t lz_gs_first_pass_bf16(const bf16* Q, int64_t ldq, const float* qkm1, const float* qk, float* r, int64_t n, int k,
                                 const LzNext& next, double* scal, double* c, double* partials, hipStream_t st);
// dst = f src
hipError_t lz_times(const float* src, double f, float* dst, int64_t n, hipStream_t st);
// Vectors so short that one block does the whole update of an iteration (see lanczos.hip): full orthogonalisation against an
// fp32 basis, and the three-term recurrence.  `host`: S_COUNT doubles of pinned host memory that also receive the scalars.
// chained: return at once after an iteration that could not advance; the three-term kernel takes beta_{k-1} from scal.
constexpr int LZ_AHEAD = 3;  // iterations of such a run the host may be ahead of
constexpr int64_t LZ_SMALL_N = 8192, LZ_SMALL_WORK = 256 * 1024;
bool lz_small(int64_t n, int64_t rows);
// What such an update works on.
struct LzSmall {
  int full;                        // orthogonalise against Q, else three terms
  const float* Q; int64_t ldq;     // full: the basis, its row stride,
  int nq;                          //   its rows (k + 1),
  float *row, *spill;              //   and where q_{k+1} goes (either may be NULL)
  const float* q; float* qp;       // three terms: q_k, and q_{k-1}, which q_{k+1} replaces
  int use_prev; float bprev;       //   with beta_{k-1}
  float* r;                        // the residual; three terms: a copy of H q_k (may be NULL)
  bf16* vb;                        // bf16 copy of q_{k+1} (may be NULL)
  int n;
  double tol;
  double *scal, *host;
  int chained;
  int64_t lds() const { return (full ? (int64_t)(nq + 1) * 8 : 0) + (int64_t)n * 4; }  // bytes; below 64 KB: n <= 8192, nq <= 2000
};
// hq: H q_k (may be u.r), flags: error bits and valid labels of the product that made it, or NULL.
hipError_t lz_small_update(const LzSmall& u, const float* hq, const int* flags, hipStream_t st);
hipError_t lz_widen(const void* src, int is_bf16, float* dst, int64_t n, hipStream_t st);

}  // namespace hf
