// Hessian-column statistics of the section "Banded Hessians" (counts of entries
// below thresholds, equal-width histogram of the absolute values): two
// HBM-bound streaming passes.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "hf_internal.h"

namespace hf {

static inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ---- column statistics --------------------------------------------------------
// stats (uint64): [0, 17) bucket counts (bucket b: entries that reach exactly b of the sorted
// thresholds), [17] NaN entries; [24] bit pattern of the largest |h_i| (non-negative floats order
// like their bit patterns); [32, 32 + n_bins) histogram.  Every counter exists CS_COPIES times, word w's at
// w * CS_COPIES, and block b uses copy b % CS_COPIES: adds from all blocks to one address take turns of 50 ns (14 us for the
// 256 blocks of the first pass).  [25], first copy: blocks of the second pass that are done; the last of them adds the copies up
// into `result` (pinned host memory, where the caller has some: no copy follows then).

// Both passes are bound by HBM: one block of 16 waves per CU walks the vector with four 16-byte loads in flight per
// thread, and what is done per entry has to fit in the 36 clocks a CU has for 64 of them at 7 TB/s.
// Few blocks also matter for the ends of the passes, which meet in global counters (2048 blocks x 50 bins: 25 us).
// Measured at n = 1.24e8 (kernels, us): first pass 136 -> 84, second 110 -> 79; the call 267 -> 186.
constexpr int CS_THREADS = 1024, CS_BLOCKS = 256;

// Calls f(x) for every entry of h, 4-byte aligned; REV: from the far end of the vector, where the first pass stopped and
// what it read last may still be in the memory-side cache.
template <bool REV, typename F>
__device__ __forceinline__ void cs_for_each(const float* __restrict__ h, int64_t n, F f) {
  const int64_t stride = (int64_t)gridDim.x * CS_THREADS;
  const int64_t gid = (int64_t)blockIdx.x * CS_THREADS + threadIdx.x;
  // scalar head up to the first 16-byte boundary, vector body, scalar tail
  const int64_t head = std::min<int64_t>(n, (int64_t)((16 - ((uintptr_t)h & 15)) & 15) / 4);
  const int64_t n4 = (n - head) >> 2;
  if (gid < head) f(h[gid]);
  const f32x4_t* h4 = (const f32x4_t*)(h + head);
  auto at = [&](int64_t i) { return __builtin_nontemporal_load(h4 + (REV ? n4 - 1 - i : i)); };
  auto take = [&](const f32x4_t& x) { f(x.x); f(x.y); f(x.z); f(x.w); };
  int64_t i = gid;
  if (i + 3 * stride < n4) {  // the next four groups are on their way while four are counted
    f32x4_t a = at(i), b = at(i + stride), c = at(i + 2 * stride), d = at(i + 3 * stride);
    i += 4 * stride;
    for (; i + 3 * stride < n4; i += 4 * stride) {
      const f32x4_t a1 = at(i), b1 = at(i + stride), c1 = at(i + 2 * stride), d1 = at(i + 3 * stride);
      take(a); take(b); take(c); take(d);
      a = a1; b = b1; c = c1; d = d1;
    }
    take(a); take(b); take(c); take(d);
  }
  for (; i < n4; i += stride) {
    take(at(i));
  }
  for (int64_t e = head + (n4 << 2) + gid; e < n; e += stride) f(h[e]);
}

// Thresholds arrive sorted ascending (the host sorts them and undoes the permutation), so an entry's contribution is one
// bucket index b = #{k : |h_i| >= t_k}; each thread counts buckets in its own LDS column with adds that return nothing (no
// conflicts: counter [bucket][thread]), and the per-threshold counts are the prefix sums of the bucket counts, formed on the
// host.  NaN entries land in bucket 17.
// TABLE: the top 11 bits of |h_i| (exponent and 3 bits of mantissa) name a cell of a table with the bucket of the cell's
// lowest value and the low 20 bits of the one threshold inside the cell, so a bucket takes one LDS read and one comparison of
// integers, NaNs included.  Needs cells with at most one
// threshold above their lowest value (thresholds closer than an eighth of an octave: the search instead).
// Otherwise: a branch-free binary search over the (padded to 16, +inf) thresholds, five dependent LDS reads.
constexpr int CS_CELLS = 2048;
template <bool TABLE>
__global__ __launch_bounds__(CS_THREADS) void colstats_pass1_kernel(const float* __restrict__ h, int64_t n, ColThresholds thr,
                                                                    unsigned long long* stats) {
  extern __shared__ unsigned cs_lds[];
  unsigned* const cnt = cs_lds;                                 // [18][CS_THREADS]
  unsigned* const cell = cs_lds + 18 * CS_THREADS;              // bucket << 21 | low bits at which the next one starts
  __shared__ float redm[CS_THREADS / 64];
  __shared__ float lt[CS_MAX_THRESHOLDS];
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < 18; ++k) cnt[k * CS_THREADS + t] = 0;
  if (t < CS_MAX_THRESHOLDS) lt[t] = thr.t[t];
  if (TABLE) {
    for (int c = t; c < CS_CELLS; c += CS_THREADS) {
      const float lo = __uint_as_float((unsigned)c << 20), hi = __uint_as_float(((unsigned)c << 20) | 0xFFFFFu);
      unsigned b = 0, in = 0x100000u;  // no value of the cell reaches the next bucket
#pragma unroll
      for (int k = 0; k < CS_MAX_THRESHOLDS; ++k) {
        if (lo >= thr.t[k]) ++b;
        else if (hi >= thr.t[k]) in = __float_as_uint(thr.t[k]) & 0xFFFFFu;
      }
      if (c == 0x7F8) { b = 16; in = 1; }  // infinity, which reaches all (padded) thresholds, and NaNs
      if (c > 0x7F8) b = 17;
      cell[c] = b << 21 | in;
    }
  }
  __syncthreads();
  float mx = 0.f;
  cs_for_each<false>(h, n, [&](float x) {
    const float a = fabsf(x);
    mx = fmaxf(mx, a);  // (ignores a NaN)
    unsigned b;
    if (TABLE) {
      const unsigned u = __float_as_uint(a), e = cell[u >> 20];
      b = (e >> 21) + ((u & 0xFFFFFu) >= (e & 0x1FFFFFu) ? 1u : 0u);
    } else {
      b = a >= lt[7] ? 8 : 0;
      b += a >= lt[b + 3] ? 4 : 0;
      b += a >= lt[b + 1] ? 2 : 0;
      b += a >= lt[b] ? 1 : 0;
      b += (b == 15 && a >= lt[15]) ? 1 : 0;
      b = a == a ? b : 17;
    }
    __hip_atomic_fetch_add(cnt + b * CS_THREADS + t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  });

  const int lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_down(mx, o, 64));
  if (lane == 0) redm[wave] = mx;
  __syncthreads();
  for (int k = wave; k < 18; k += CS_THREADS / 64) {  // bucket totals of the block
    unsigned s = 0;
    for (int i = lane; i < CS_THREADS; i += 64) s += cnt[k * CS_THREADS + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (lane == 0 && s) atomicAdd(stats + k * CS_COPIES + blockIdx.x % CS_COPIES, (unsigned long long)s);
  }
  if (t == 0) {
    float m = redm[0];
    for (int w = 1; w < CS_THREADS / 64; ++w) m = fmaxf(m, redm[w]);
    atomicMax((unsigned*)(stats + 24 * CS_COPIES + blockIdx.x % CS_COPIES), __float_as_uint(m));
  }
}

// Bin of |h_i|: floor(|h_i| * scale), scale = n_bins / max as one correctly rounded float32
// quotient; the maximum itself (and a product that is not a number, which needs an infinite
// maximum) lands in the last bin.  The maximum is the first pass's result, read from the counters,
// so no host round trip separates the passes; a column without a
// positive maximum (all zeros, or empty) leaves the bins untouched for the host to fill in.
// A bin's counter is kept 16 times, one for every 16th lane: a column that is nearly all zeros (the case the paper reports),
// or one value, sends a wave's lanes to one bin, and so to at most four lanes per counter and to different banks.
__global__ __launch_bounds__(CS_THREADS) void colstats_hist_kernel(const float* __restrict__ h, int64_t n,
                                                                   unsigned long long* stats, int nb, unsigned long long* result) {
  __shared__ unsigned lh[CS_MAX_BINS * 16];
  __shared__ int last_block;
  float mx = 0.f;
#pragma unroll
  for (int c = 0; c < CS_COPIES; ++c) mx = fmaxf(mx, __uint_as_float((unsigned)stats[24 * CS_COPIES + c]));
  const float scale = __fdiv_rn((float)nb, mx), last = (float)(nb - 1);
  for (int i = threadIdx.x; i < nb * 16; i += CS_THREADS) lh[i] = 0;
  __syncthreads();
  unsigned* const mine = lh + (threadIdx.x & 15);
  if (mx > 0.f) cs_for_each<true>(h, n, [&](float x) {
    const float a = fabsf(x), s = __fmul_rn(a, scale);
    if (a == a) {
      const int b = s == s ? (int)fminf(floorf(s), last) : nb - 1;
      __hip_atomic_fetch_add(mine + b * 16, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  });
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += CS_THREADS) {
    unsigned s = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) s += lh[i * 16 + ((r + i) & 15)];
    if (s) atomicAdd(stats + (32 + i) * CS_COPIES + blockIdx.x % CS_COPIES, (unsigned long long)s);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the adds are made at the memory side: acknowledged is done
  __syncthreads();
  if (threadIdx.x == 0)
    last_block = __hip_atomic_fetch_add(stats + 25 * CS_COPIES, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!last_block) return;
  for (int w = threadIdx.x; w < 32 + nb; w += CS_THREADS) {
    unsigned long long s = 0;
#pragma unroll
    for (int c = 0; c < CS_COPIES; ++c) {
      const unsigned long long x = __hip_atomic_load(stats + w * CS_COPIES + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s = w == 24 ? (x > s ? x : s) : s + x;
    }
    result[w] = s;
  }
}

// Each block sees at most n / CS_BLOCKS + 4096 entries, so its 32-bit counters cannot overflow for n <= 2^40 - 2^20 (fourteen
// times what 288 GB hold).
static inline int colstats_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(cdiv64(n, 4 * CS_THREADS), CS_BLOCKS)); }

hipError_t launch_colstats_pass1(const float* h, int64_t n, const ColThresholds& thr, unsigned long long* stats, hipStream_t st) {
  // at most one threshold in a cell of the table, those on its lowest value apart
  bool table = true;
  for (int k = 0; k + 1 < CS_MAX_THRESHOLDS && table; ++k) {
    unsigned a, b;
    memcpy(&a, &thr.t[k], 4);
    memcpy(&b, &thr.t[k + 1], 4);
    if (thr.t[k] > 0.f && thr.t[k + 1] < INFINITY && a >> 20 == b >> 20 && (a & 0xFFFFF) != 0) table = false;
  }
  const int lds = 18 * CS_THREADS * 4 + CS_CELLS * 4;
  static OncePerDevice once_t, once_s;
  hipError_t e = table ? once_t.lds_limit((const void*)colstats_pass1_kernel<true>, lds) : once_s.lds_limit((const void*)colstats_pass1_kernel<false>, lds);
  if (e != hipSuccess) return e;
  if (table) hipLaunchKernelGGL(colstats_pass1_kernel<true>, dim3(colstats_blocks(n)), dim3(CS_THREADS), lds, st, h, n, thr, stats);
  else hipLaunchKernelGGL(colstats_pass1_kernel<false>, dim3(colstats_blocks(n)), dim3(CS_THREADS), lds, st, h, n, thr, stats);
  return hipGetLastError();
}
hipError_t launch_colstats_hist(const float* h, int64_t n, unsigned long long* stats, int nb, unsigned long long* result, hipStream_t st) {
  hipLaunchKernelGGL(colstats_hist_kernel, dim3(colstats_blocks(n)), dim3(CS_THREADS), 0, st, h, n, stats, nb, result);
  return hipGetLastError();
}

// ---- counters for callers that cannot allocate -------------------------------------
// A fixed array in the library's device image, one copy per GPU, held until the process ends.
// Host code must not hand the symbol itself to a kernel: its device address is looked up once per
// device (with that device current) and only that pointer is used afterwards.
static __device__ __align__(256) unsigned long long scratch[CS_ARRAY_WORDS];

hipError_t colstats_static_counters(unsigned long long** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static unsigned long long* ptr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr[dev] = (unsigned long long*)p;
  }
  *out = ptr[dev];
  return hipSuccess;
}

}  // namespace hf
