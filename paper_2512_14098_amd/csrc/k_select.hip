// k_select.hip -- cf_select_topk and cf_rate_grid.
//
// Top-K of the plans kept by phase 1, ordered by R_d descending and plan id
// ascending (Alg. 2 evaluates the most promising survivors first; the rate
// grid scales with the headroom alpha of Sec. 4.3).  The order key is the
// 96-bit value (bits of R_d, ~id): unique per plan, so the K largest keys
// are found by an MSD radix select over the range of the kept keys, compacted,
// and placed by rank (number of larger keys).
//
// cf_topk_merge keeps the top-K of a plan space screened window by window:
// the window's selection and the running list are both in key order, so
// each element's place in the merged list is its index in its own list plus
// the number of elements of the other list ahead of it (a binary search).
#include <cmath>

#include "cf_internal.h"

namespace cf {
namespace {

// The key of a kept plan is (off, rid): off = bits of R_d minus the smallest
// kept bits, rid = kIdMax - id; the k largest keys are taken.  What is decided
// of the threshold: off >> shift == prefix and, once shift is 0,
// rid >> idshift == idprefix.  Pass d histograms the next kDigit bits of the
// keys that match, and pass d + 1 begins with every block picking the digit
// from that histogram: 4,096 bins read from L2 by each block cost less than a
// launch of their own or than a last block, whose device-scope fence writes
// the L2 back (10^6 plans: 39 us a pass with it, 6 us without).  A bucket that
// is taken whole ends the search; the passes after it return at once.
// 10^6 plans, 1,000 taken, the whole selection: 353 us before (24 launches of
// 8-bit digits, a serial pick, a rank by one key per thread), about 110 us now.
constexpr int kDigit = 12, kBins = 1 << kDigit, kPasses = 8;  // 64 bits of R_d and 24 of the id
constexpr unsigned kIdMax = 0xFFFFFFu;                         // P <= 2^24
struct Threshold {
  unsigned long long prefix;
  unsigned int idprefix;
  int shift, idshift;
  unsigned int k_rem;  // keys still to take at or below the prefix
  unsigned int done;   // the threshold is decided
};
struct SelState {
  unsigned long long mn, mx;  // smallest and largest bits of a kept R_d
  unsigned int k, kept;       // keys to take; kept plans
  unsigned int count;         // compacted so far
  Threshold th[kPasses];      // as pass d found it
  unsigned int hist[kPasses][kBins];
};

// calls f(p, bits of R_d) for every kept plan of this thread's share
template <class F>
__device__ __forceinline__ void for_kept(const double *rd, const uint8_t *flags, int P, F f) {
  const long long t0 = (long long)blockIdx.x * blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
  const bool words = ((uintptr_t)flags & 3u) == 0;
  for (long long q = t0; q * 4 < P; q += step) {
    const int p0 = (int)(q * 4), n = P - p0 < 4 ? P - p0 : 4;
    uint32_t w = 0;
    if (words && n == 4) {
      w = *(const uint32_t *)(flags + p0);
    } else {
      for (int i = 0; i < n; i++) w |= (uint32_t)flags[p0 + i] << (8 * i);
    }
    w &= 0x01010101u * CF_FLAG_KEEP;
    for (; w; w &= w - 1) {
      const int p = p0 + ((__ffs(w) - 1) >> 3);
      f(p, (unsigned long long)__double_as_longlong(rd[p]));
    }
  }
}

__global__ void __launch_bounds__(256) k_sel_init(SelState *st, unsigned int k) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g == 0) {
    st->mn = ~0ull;
    st->mx = 0;
    st->k = k;
    st->kept = 0;
    st->count = 0;
  }
  if (g < kPasses * kBins) (&st->hist[0][0])[g] = 0;
}

// range of the kept plans' R_d bits and their number
__global__ void __launch_bounds__(256) k_sel_range(const double *rd, const uint8_t *flags, int P, SelState *st) {
  __shared__ unsigned long long mn_s, mx_s;
  __shared__ unsigned int n_s;
  if (threadIdx.x == 0) {
    mn_s = ~0ull;
    mx_s = 0;
    n_s = 0;
  }
  __syncthreads();
  unsigned long long mn = ~0ull, mx = 0;
  unsigned int n = 0;
  for_kept(rd, flags, P, [&](int, unsigned long long b) {
    mn = b < mn ? b : mn;
    mx = b > mx ? b : mx;
    n++;
  });
  if (n) {
    atomicMin(&mn_s, mn);
    atomicMax(&mx_s, mx);
    atomicAdd(&n_s, n);
  }
  __syncthreads();
  if (threadIdx.x == 0 && n_s) {
    atomicMin(&st->mn, mn_s);
    atomicMax(&st->mx, mx_s);
    atomicAdd(&st->kept, n_s);
  }
}

// The threshold as far as passes 0 .. d-1 decide it (all 256 threads; the
// same in every block).
__device__ __forceinline__ Threshold threshold_at(const SelState *st, int d) {
  __shared__ unsigned int part[256];
  __shared__ Threshold out;
  const int tid = threadIdx.x;
  if (d == 0) {
    Threshold t = {0, 0, 0, 24, st->k, 0};
    if (st->kept <= st->k) t.done = 1;  // every kept plan
    else if (st->mx > st->mn) t.shift = 64 - __clzll((long long)(st->mx - st->mn));
    return t;
  }
  const Threshold t = st->th[d - 1];
  if (t.done) return t;
  // thread i holds bins [16 i, 16 i + 16); keys are taken from the top bin down
  constexpr int per = kBins / 256;
  unsigned int v[per], sum = 0;
#pragma unroll
  for (int i = 0; i < per; i++) {
    v[i] = st->hist[d - 1][tid * per + i];
    sum += v[i];
  }
  part[tid] = sum;
  __syncthreads();
  for (int w = 1; w < 256; w <<= 1) {  // inclusive sums from the top
    const unsigned int add = tid + w < 256 ? part[tid + w] : 0u;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  unsigned int cum = part[tid] - sum;  // keys in higher bins
#pragma unroll
  for (int i = per - 1; i >= 0; i--) {
    if (cum < t.k_rem && cum + v[i] >= t.k_rem) {
      Threshold n = t;
      const unsigned int digit = (unsigned int)(tid * per + i);
      if (t.shift == 0) {
        n.idshift = t.idshift > kDigit ? t.idshift - kDigit : 0;
        n.idprefix = (t.idprefix << (t.idshift - n.idshift)) | digit;
      } else {
        n.shift = t.shift > kDigit ? t.shift - kDigit : 0;
        n.prefix = (t.prefix << (t.shift - n.shift)) | digit;
      }
      n.k_rem = t.k_rem - cum;
      n.done = cum + v[i] == t.k_rem ? 1u : 0u;  // the whole bucket
      out = n;
    }
    cum += v[i];
  }
  __syncthreads();
  return out;
}

__global__ void __launch_bounds__(256) k_sel_pass(const double *rd, const uint8_t *flags, int P, SelState *st, int d) {
  __shared__ unsigned int h[kBins];
  const int tid = threadIdx.x;
  const Threshold t = threshold_at(st, d);
  if (blockIdx.x == 0 && tid == 0) st->th[d] = t;
  if (t.done) return;
  const unsigned long long mn = st->mn;
  for (int b = tid; b < kBins; b += 256) h[b] = 0;
  __syncthreads();
  const bool ids = t.shift == 0;  // R_d is decided (or the same everywhere)
  // the next digit: bits [s2, top) of off, or of rid
  const int top = ids ? t.idshift : t.shift, s2 = top > kDigit ? top - kDigit : 0;
  const unsigned int mask = (1u << (top - s2)) - 1u;
  for_kept(rd, flags, P, [&](int p, unsigned long long b) {
    const unsigned long long off = b - mn;
    if (ids) {
      const unsigned int rid = kIdMax - (unsigned int)p;
      if (off == t.prefix && (rid >> t.idshift) == t.idprefix) atomicAdd(&h[(rid >> s2) & mask], 1u);
    } else if (t.shift == 64 || (off >> t.shift) == t.prefix) {
      atomicAdd(&h[(unsigned int)(off >> s2) & mask], 1u);
    }
  });
  __syncthreads();
  for (int b = tid; b < kBins; b += 256)
    if (h[b]) atomicAdd(&st->hist[d][b], h[b]);
}

__global__ void __launch_bounds__(256) k_sel_compact(const double *rd, const uint8_t *flags, int P, SelState *st,
                                                    unsigned long long *khi, unsigned int *klo, int cap) {
  const Threshold t = threshold_at(st, kPasses);
  const unsigned long long mn = st->mn;
  for_kept(rd, flags, P, [&](int p, unsigned long long b) {
    const unsigned long long a = t.shift == 64 ? 0 : (b - mn) >> t.shift;
    const unsigned int rid = kIdMax - (unsigned int)p;
    if (a > t.prefix || (a == t.prefix && (rid >> t.idshift) >= t.idprefix)) {
      // one atomic per wavefront for the lanes that are here together
      const unsigned long long here = __ballot(1);
      const int lane = threadIdx.x & 63, lead = __ffsll((long long)here) - 1;
      unsigned int base = 0;
      if (lane == lead) base = atomicAdd(&st->count, (unsigned int)__popcll(here));
      base = (unsigned int)__shfl((int)base, lead, 64);
      const unsigned int i = base + (unsigned int)__popcll(here & ((1ull << lane) - 1ull));
      if ((int)i < cap) {
        khi[i] = b;
        klo[i] = 0xFFFFFFFFu - (unsigned int)p;
      }
    }
  });
}

// Place of every selected plan: the number of larger keys.  A wavefront ranks
// kRankPer keys at once, its lanes striding over the list.
constexpr int kRankPer = 4;
__global__ void __launch_bounds__(256) k_sel_rank(const unsigned long long *khi, const unsigned int *klo,
                                                 const SelState *st, int cap, int32_t *ids) {
  const int n = (int)(st->count < (unsigned)cap ? st->count : (unsigned)cap);
  const int lane = threadIdx.x & 63, i0 = (int)((blockIdx.x * 4 + (threadIdx.x >> 6)) * kRankPer);
  if (i0 >= n) return;
  unsigned long long hi[kRankPer];
  unsigned int lo[kRankPer];
  int rank[kRankPer];
#pragma unroll
  for (int q = 0; q < kRankPer; q++) {
    const int i = i0 + q < n ? i0 + q : n - 1;
    hi[q] = khi[i];
    lo[q] = klo[i];
    rank[q] = 0;
  }
  for (int j = lane; j < n; j += 64) {
    const unsigned long long h = khi[j];
    const unsigned int l = klo[j];
#pragma unroll
    for (int q = 0; q < kRankPer; q++) rank[q] += (h > hi[q] || (h == hi[q] && l > lo[q])) ? 1 : 0;
  }
#pragma unroll
  for (int q = 0; q < kRankPer; q++) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) rank[q] += __shfl_xor(rank[q], d, 64);
    if (lane == 0 && i0 + q < n) ids[rank[q]] = (int32_t)(0xFFFFFFFFu - lo[q]);
  }
}

// (R_d bits, plan number) of a precedes b: larger R_d, or equal R_d and a
// smaller plan number (the order of cf_select_topk, with 64-bit numbers)
__device__ __forceinline__ bool key_ahead(unsigned long long ra, uint64_t ga, unsigned long long rb, uint64_t gb) {
  return ra > rb || (ra == rb && ga < gb);
}

__global__ void k_topk_merge(const double *rd_run, const uint64_t *gid_run, int n_run, const double *rd_win,
                             const int32_t *ids_win, int n_win, uint64_t first, int k, double *rd_out,
                             uint64_t *gid_out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_run + n_win) return;
  const bool in_run = i < n_run;
  const int own = in_run ? i : i - n_run;
  double r;
  uint64_t g;
  if (in_run) {
    r = rd_run[own];
    g = gid_run[own];
  } else {
    const int32_t id = ids_win[own];
    r = rd_win[id];
    g = first + (uint64_t)id;
  }
  const unsigned long long rb = (unsigned long long)__double_as_longlong(r);
  // elements of the other list ahead of this one: a prefix of that list
  int lo = 0, hi = in_run ? n_win : n_run;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    unsigned long long ro;
    uint64_t go;
    if (in_run) {
      const int32_t id = ids_win[mid];
      ro = (unsigned long long)__double_as_longlong(rd_win[id]);
      go = first + (uint64_t)id;
    } else {
      ro = (unsigned long long)__double_as_longlong(rd_run[mid]);
      go = gid_run[mid];
    }
    if (key_ahead(ro, go, rb, g)) lo = mid + 1;
    else hi = mid;
  }
  const int pos = own + lo;
  if (pos < k) {
    rd_out[pos] = r;
    gid_out[pos] = g;
  }
}

__global__ void k_rate_grid(const double *rd, const int32_t *ids, int n, int K, double alpha, double *rates) {
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= (long long)n * K) return;
  const int i = (int)(j / K), k = (int)(j % K);
  const double A = rd[ids[i]] * alpha;
  rates[j] = (A * (double)(k + 1)) / (double)K;
}

}  // namespace
}  // namespace cf

extern "C" cf_status cf_select_topk(const double *rd_dev, const uint8_t *flags_dev, int32_t P, int32_t k,
                                    int32_t *ids_dev, int32_t *n_selected_host, void *stream) {
  using namespace cf;
  if (!rd_dev || !flags_dev || !ids_dev || !n_selected_host) return set_error(CF_EINVAL, "NULL argument");
  if (P < 0 || P > (1 << 24)) return set_error(CF_ECAPACITY, "P out of 0..2^24");
  if (k < 1 || k > 65536) return set_error(CF_ECAPACITY, "k out of 1..65536");
  hipStream_t s = as_stream(stream);
  cf_status st = CF_OK;
  const size_t bytes = 256 + sizeof(SelState) + (size_t)k * (sizeof(unsigned long long) + sizeof(unsigned int));
  char *scr = (char *)scratch_get(SCR_SELECT, bytes, &st);
  if (!scr) return st;
  SelState *ss = (SelState *)scr;
  unsigned long long *khi = (unsigned long long *)(scr + ((sizeof(SelState) + 255) & ~(size_t)255));
  unsigned int *klo = (unsigned int *)(khi + k);
  hipLaunchKernelGGL(k_sel_init, dim3(kPasses * kBins / 256), dim3(256), 0, s, ss, (unsigned)k);
  // four plans per thread, at most two blocks per CU (every block flushes a histogram)
  const unsigned grid = (unsigned)((P + 1023) / 1024 < 512 ? (P + 1023) / 1024 : 512);
  if (P > 0) {
    hipLaunchKernelGGL(k_sel_range, dim3(grid), dim3(256), 0, s, rd_dev, flags_dev, P, ss);
    for (int d = 0; d < kPasses; d++)
      hipLaunchKernelGGL(k_sel_pass, dim3(grid), dim3(256), 0, s, rd_dev, flags_dev, P, ss, d);
    hipLaunchKernelGGL(k_sel_compact, dim3(grid), dim3(256), 0, s, rd_dev, flags_dev, P, ss, khi, klo, k);
    hipLaunchKernelGGL(k_sel_rank, dim3((unsigned)((k + 4 * kRankPer - 1) / (4 * kRankPer))), dim3(256), 0, s, khi, klo,
                       ss, k, ids_dev);
  }
  st = hip_check(hipGetLastError(), "cf_select_topk launch");
  if (st != CF_OK) return st;
  unsigned int cnt = 0;
  st = hip_check(hipMemcpyAsync(&cnt, &ss->count, sizeof cnt, hipMemcpyDeviceToHost, s), "copy count");
  if (st != CF_OK) return st;
  st = hip_check(hipStreamSynchronize(s), "cf_select_topk sync");
  if (st != CF_OK) return st;
  *n_selected_host = (int32_t)(cnt < (unsigned)k ? cnt : (unsigned)k);
  return CF_OK;
}

extern "C" cf_status cf_rate_grid(const double *rd_dev, const int32_t *ids_dev, int32_t n, int32_t K,
                                  double alpha_max, double *rates_dev, void *stream) {
  using namespace cf;
  if (!rd_dev || !ids_dev || !rates_dev) return set_error(CF_EINVAL, "NULL argument");
  if (n < 0 || K < 1) return set_error(CF_EINVAL, "n >= 0 and K >= 1 required");
  if (!(alpha_max > 0.0) || !std::isfinite(alpha_max)) return set_error(CF_EINVAL, "alpha_max must be > 0");
  if (n == 0) return CF_OK;
  const long long tot = (long long)n * K;
  hipLaunchKernelGGL(k_rate_grid, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, as_stream(stream), rd_dev,
                     ids_dev, n, K, alpha_max, rates_dev);
  return hip_check(hipGetLastError(), "cf_rate_grid launch");
}

extern "C" cf_status cf_topk_merge(const double *rd_run_dev, const uint64_t *gid_run_dev, int32_t n_run,
                                   const double *rd_win_dev, const int32_t *ids_win_dev, int32_t n_win,
                                   uint64_t win_first, int32_t k, double *rd_out_dev, uint64_t *gid_out_dev,
                                   void *stream) {
  using namespace cf;
  if (k < 1 || k > 65536) return set_error(CF_ECAPACITY, "k out of 1..65536");
  if (n_run < 0 || n_run > 65536 || n_win < 0 || n_win > 65536)
    return set_error(CF_EINVAL, "n_run and n_win must be in 0..65536");
  if (!rd_out_dev || !gid_out_dev) return set_error(CF_EINVAL, "NULL output");
  if (n_run > 0 && (!rd_run_dev || !gid_run_dev)) return set_error(CF_EINVAL, "NULL running list");
  if (n_win > 0 && (!rd_win_dev || !ids_win_dev)) return set_error(CF_EINVAL, "NULL window");
  if ((const void *)rd_out_dev == (const void *)rd_run_dev || (const void *)gid_out_dev == (const void *)gid_run_dev)
    return set_error(CF_EINVAL, "outputs alias the running list");
  const int n = n_run + n_win;
  if (n == 0) return CF_OK;
  hipLaunchKernelGGL(k_topk_merge, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream), rd_run_dev,
                     gid_run_dev, n_run, rd_win_dev, ids_win_dev, n_win, win_first, k, rd_out_dev, gid_out_dev);
  return hip_check(hipGetLastError(), "cf_topk_merge launch");
}
