// k_trace.hip -- cf_trace_gen: synthetic Any-to-Any request traces.
//
// The workload of Sec. 3.1 (request types with fractions pi_t) with Poisson
// arrivals.  One thread per (seed, request) draws Philox4x64-10 blocks keyed
// by (seed, 0) with counter (request, field, attempt, 0); the gap ticks are
// then turned into arrival ticks by an exact u64 inclusive scan per seed.
// Per-type moments are u64 sums (order-free integer atomics).
#include "cf_internal.h"

namespace cf {
namespace {

constexpr int kSeedsPerLaunch = 64;
struct SeedChunk { uint64_t v[kSeedsPerLaunch]; };

enum { F_ARRIVAL = 0, F_PROMPT = 1, F_OUT = 2, F_PATCH = 3, F_AUDIN = 4, F_AUDOUT = 5, F_ROUTE = 6 };

__device__ __forceinline__ int64_t uni_int(uint64_t x, int64_t lo, int64_t hi) {
  return lo + (int64_t)(((x >> 32) * (uint64_t)(hi - lo + 1)) >> 32);
}

__device__ __forceinline__ int64_t clamp_round(double v, int64_t lo, int64_t hi) {
  double r = rint(v);
  if (r <= (double)lo) return lo;
  if (r >= (double)hi) return hi;
  return (int64_t)r;
}

__global__ void k_zero_u64(uint64_t *p, long long n) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// inclusive sum over the wavefront's lanes
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint64_t o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// One block of kDraw consecutive requests of a seed.  What bounds it are the
// Philox rounds (quarter-rate 32 x 32 multiplies) and the fp64 logarithm,
// root and exponential of a length.  A thread per request would run every
// field's draws for the whole wavefront where some lane needs them (audio
// lengths of a third of the requests, second attempts of the polar method,
// 4.6 % of the draws but nearly every wavefront): eleven Philox blocks per
// request where five are needed.  So each request first draws its arrival and
// route blocks, then the block's draws (request, field) are listed in LDS and
// taken densely, one per thread, attempt by attempt; a rejected draw is listed
// again for the next attempt.  The order of the list does not matter: a draw
// depends on (seed, request, field, attempt) only.
// 64 seeds x 10^5 requests of the omni workload: 748 us before, 462 us now under the profiler's
// kernel trace; the whole call without it 710 -> 437 us.
constexpr int kDraw = 256;
constexpr int kFields = 5;  // prompt, out, patches, audio in, audio out
struct DrawLds {
  unsigned long long mom[CF_MAX_TYPES * 8];
  cf_dist len[CF_MAX_TYPES][4];
  uint64_t wsum[kDraw / 64];
  uint32_t val[kFields][kDraw];
  uint16_t list[2][kDraw * kFields];  // request (bits 0..7) and field (8..10) of a draw
  uint8_t type[kDraw], nimg[kDraw];
  int n_list[2];
};

__global__ void __launch_bounds__(kDraw) k_trace_draw(KModel m, SeedChunk seeds, int s0, int n, cf_trace tr,
                                                      uint64_t *moments, uint64_t *tot, int nb) {
  __shared__ DrawLds sh;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < CF_MAX_TYPES * 8) sh.mom[tid] = 0;
  if (tid < CF_MAX_TYPES * 4) (&sh.len[0][0])[tid] = (&m.len[0][0])[tid];
  if (tid < 2) sh.n_list[tid] = 0;
  const int sl = blockIdx.y;
  const int s = s0 + sl;
  const uint64_t seed = seeds.v[sl];
  const long long i0 = (long long)blockIdx.x * kDraw, i = i0 + tid;
  const size_t o = (size_t)s * (size_t)n + (size_t)i;
  const bool in = i < n;
  __syncthreads();
  int t = 0, nimg = 0;
  uint64_t gap = 0;
#pragma unroll
  for (int f = 0; f < kFields; f++) sh.val[f][tid] = 0;
  if (in) {
    uint64_t x[4], y[4];
    philox4x64_10((uint64_t)i, F_ARRIVAL, 0, 0, seed, 0, x);
    philox4x64_10((uint64_t)i, F_ROUTE, 0, 0, seed, 0, y);
    gap = (uint64_t)rint(-dev_log(u01(x[0])) * 0x1p32);
    const uint64_t v = ((x[1] >> 32) * m.wsum) >> 32;
    uint64_t cum = m.weight[0];
    while (cum <= v && t + 1 < m.nt) { t++; cum += m.weight[t]; }
    if (m.img_kind[t] == CF_IMG_CONST) nimg = m.img_lo[t];
    else if (m.img_kind[t] == CF_IMG_UNIFORM) nimg = (int)uni_int(x[2], m.img_lo[t], m.img_hi[t]);
    tr.rkey0_dev[o] = y[0];
    tr.rkey1_dev[o] = y[1];
    tr.akey_dev[o] = (uint32_t)(y[2] >> 32);
  }
  sh.type[tid] = (uint8_t)t;
  sh.nimg[tid] = (uint8_t)nimg;
  // the draws of this request: patches (field 2), and each length that is not constant
#pragma unroll
  for (int f = 0; f < kFields; f++) {
    bool draw = false;
    if (in) {
      if (f == 2) {
        draw = nimg > 0;
      } else {
        const cf_dist &d = sh.len[t][f < 2 ? f : f - 1];
        if (d.kind == CF_DIST_CONST) sh.val[f][tid] = (uint32_t)(int64_t)d.p0;
        draw = d.kind == CF_DIST_LOGNORMAL || d.kind == CF_DIST_EXP;
      }
    }
    const unsigned long long bal = __ballot(draw);
    int base = 0;
    if (lane == 0 && bal) base = atomicAdd(&sh.n_list[0], __popcll(bal));
    base = __shfl(base, 0, 64);
    if (draw) sh.list[0][base + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(tid | (f << 8));
  }
  // the gaps' inclusive sums inside the block
  uint64_t incl = wave_incl_scan(gap, lane);
  if (lane == 63) sh.wsum[tid >> 6] = incl;
  __syncthreads();
  for (int k = 0; k < (tid >> 6); k++) incl += sh.wsum[k];
  if (in) tr.arr_ticks_dev[o] = incl;  // the scan adds the blocks before this one
  if (tid == kDraw - 1) tot[(size_t)s * nb + blockIdx.x] = incl;
  for (int k = 0;; k++) {  // attempt k of the listed draws
    const int cur = k & 1, cnt = sh.n_list[cur];
    if (cnt == 0) break;
    for (int q = tid; q < cnt; q += kDraw) {
      const int e = sh.list[cur][q], r = e & 255, f = e >> 8;
      const uint64_t field = f == 0 ? F_PROMPT : f == 1 ? F_OUT : f == 2 ? F_PATCH : f == 3 ? F_AUDIN : F_AUDOUT;
      uint64_t x[4];
      philox4x64_10((uint64_t)(i0 + r), field, (uint64_t)k, 0, seed, 0, x);
      if (f == 2) {
        uint32_t patches = 0;
        const int ni = sh.nimg[r];
#pragma unroll
        for (int a = 0; a < 4; a++)
          if (a < ni) patches += (uint32_t)uni_int(x[a], m.patch_lo, m.patch_hi);
        sh.val[f][r] = patches;
        continue;
      }
      const cf_dist &d = sh.len[sh.type[r]][f < 2 ? f : f - 1];
      if (d.kind == CF_DIST_EXP) {
        sh.val[f][r] = (uint32_t)clamp_round(d.p0 * (-dev_log(u01(x[0]))), d.lo, d.hi);
        continue;
      }
      // Marsaglia polar method: pairs (x0, x1), then (x2, x3), of blocks k = 0 .. 31
      double v1 = 2.0 * u01(x[0]) - 1.0, v2 = 2.0 * u01(x[1]) - 1.0;
      double w = v1 * v1 + v2 * v2;
      if (!(w > 0.0 && w < 1.0)) {
        v1 = 2.0 * u01(x[2]) - 1.0;
        v2 = 2.0 * u01(x[3]) - 1.0;
        w = v1 * v1 + v2 * v2;
      }
      double z = 0.0;
      if (w > 0.0 && w < 1.0) {
        z = v1 * sqrt((-2.0 * dev_log(w)) / w);
      } else if (k < 31) {
        sh.list[cur ^ 1][atomicAdd(&sh.n_list[cur ^ 1], 1)] = (uint16_t)e;
        continue;
      }
      sh.val[f][r] = (uint32_t)clamp_round(d.scale * dev_exp(d.p0 + d.p1 * z), d.lo, d.hi);
    }
    __syncthreads();
    if (tid == 0) sh.n_list[cur] = 0;
    __syncthreads();
  }
  if (in) {
    const uint32_t prompt = sh.val[0][tid], out = sh.val[1][tid], patches = sh.val[2][tid], ain = sh.val[3][tid],
                   aout = sh.val[4][tid];
    tr.type_dev[o] = (uint8_t)t;
    tr.n_img_dev[o] = (uint8_t)nimg;
    tr.patches_dev[o] = (uint16_t)patches;
    tr.prompt_dev[o] = (uint16_t)prompt;
    tr.out_dev[o] = (uint16_t)out;
    tr.aud_in_ms_dev[o] = ain;
    tr.aud_out_ms_dev[o] = aout;
    unsigned long long *mt = sh.mom + t * 8;
    atomicAdd(mt + 0, 1ull);
    atomicAdd(mt + 1, (unsigned long long)prompt);
    atomicAdd(mt + 2, (unsigned long long)out);
    if (patches) atomicAdd(mt + 3, (unsigned long long)patches);
    if (ain) {
      atomicAdd(mt + 4, (unsigned long long)ain);
      atomicAdd(mt + 6, (unsigned long long)((ain + 79u) / 80u));
    }
    if (aout) {
      atomicAdd(mt + 5, (unsigned long long)aout);
      atomicAdd(mt + 7, (unsigned long long)((aout + 79u) / 80u));
    }
  }
  __syncthreads();
  if (tid < m.nt * 8 && sh.mom[tid] != 0)
    atomicAdd((unsigned long long *)(moments + (size_t)s * m.nt * 8 + tid), sh.mom[tid]);
}

// ---- exact u64 inclusive scan of each seed's gaps: the draw leaves the sums
// inside its blocks and the blocks' totals; those are scanned per seed and
// added back.
// One block per seed; a round scans kTotBlock * kTotPer totals, and the rounds
// depend on each other, so a block takes as many totals at once as it can hold:
// with one wavefront and 64 totals a round, generating one trace of 2^26
// requests (262,144 totals) took 9.53 ms, now 7.32; 2^20 requests 181 -> 153 us.
constexpr int kTotBlock = 1024, kTotPer = 4;
__global__ void __launch_bounds__(kTotBlock) k_scan_totals(uint64_t *tot, int nb) {
  __shared__ uint64_t wsum[kTotBlock / 64];
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t carry = 0;
  uint64_t *t = tot + (size_t)s * nb;
  for (int b0 = 0; b0 < nb; b0 += kTotBlock * kTotPer) {
    const int i0 = b0 + tid * kTotPer;
    uint64_t v[kTotPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kTotPer; j++) {
      v[j] = i0 + j < nb ? t[i0 + j] : 0;
      sum += v[j];
    }
    const uint64_t incl = wave_incl_scan(sum, lane);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint64_t e = carry + incl - sum;  // exclusive
#pragma unroll
    for (int k = 0; k < kTotBlock / 64; k++) {
      const uint64_t x = wsum[k];
      if (k < wave) e += x;
      carry += x;
    }
#pragma unroll
    for (int j = 0; j < kTotPer; j++) {
      if (i0 + j < nb) t[i0 + j] = e;
      e += v[j];
    }
    __syncthreads();  // the wavefronts' sums are read before the next round writes them
  }
}

constexpr int kAddPer = 4;  // blocks of the draw per block
__global__ void __launch_bounds__(kDraw) k_scan_add(uint64_t *a, int n, const uint64_t *tot, int nb) {
  const int s = blockIdx.y;
  uint64_t *base = a + (size_t)s * n;
#pragma unroll
  for (int q = 0; q < kAddPer; q++) {
    const int b = blockIdx.x * kAddPer + q;
    const long long i = (long long)b * kDraw + threadIdx.x;
    if (i < n && b > 0) base[i] += tot[(size_t)s * nb + b];
  }
}

}  // namespace
}  // namespace cf

extern "C" cf_status cf_trace_gen(const cf_model_desc *model, const uint64_t *seeds_host,
                                  int32_t n_seeds, int32_t n_req, const cf_trace *out,
                                  uint64_t *moments_dev, void *stream) {
  using namespace cf;
  KModel m;
  cf_status st = lower_model(model, &m);
  if (st != CF_OK) return st;
  if (!seeds_host || !out || !moments_dev) return set_error(CF_EINVAL, "NULL argument");
  if (n_seeds < 1 || n_req < 0) return set_error(CF_EINVAL, "n_seeds >= 1 and n_req >= 0 required");
  if (out->n_seeds != n_seeds || out->n_req != n_req)
    return set_error(CF_EINVAL, "trace descriptor sizes differ from the call's");
  if (n_req > (1 << 26)) return set_error(CF_ECAPACITY, "n_req above 2^26");
  if (n_req > 0 && (!out->arr_ticks_dev || !out->type_dev || !out->n_img_dev || !out->patches_dev ||
                    !out->prompt_dev || !out->out_dev || !out->aud_in_ms_dev || !out->aud_out_ms_dev ||
                    !out->rkey0_dev || !out->rkey1_dev || !out->akey_dev))
    return set_error(CF_EINVAL, "NULL trace array");
  hipStream_t s = as_stream(stream);
  const long long nmom = (long long)n_seeds * m.nt * 8;
  hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)((nmom + 255) / 256)), dim3(256), 0, s, moments_dev, nmom);
  if (n_req == 0) return hip_check(hipGetLastError(), "cf_trace_gen launch");
  const int nb = (n_req + kDraw - 1) / kDraw;
  uint64_t *tot = (uint64_t *)scratch_get(SCR_TRACE, sizeof(uint64_t) * (size_t)nb * n_seeds, &st);
  if (!tot) return st;
  for (int s0 = 0; s0 < n_seeds; s0 += kSeedsPerLaunch) {
    SeedChunk sc;
    const int ns = n_seeds - s0 < kSeedsPerLaunch ? n_seeds - s0 : kSeedsPerLaunch;
    for (int j = 0; j < kSeedsPerLaunch; j++) sc.v[j] = j < ns ? seeds_host[s0 + j] : 0;
    hipLaunchKernelGGL(k_trace_draw, dim3((unsigned)nb, (unsigned)ns), dim3(kDraw), 0, s, m, sc, s0, n_req, *out,
                       moments_dev, tot, nb);
  }
  if (nb > 1) {  // one block's sums need nothing added
    hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)n_seeds), dim3(kTotBlock), 0, s, tot, nb);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((nb + kAddPer - 1) / kAddPer), (unsigned)n_seeds), dim3(kDraw), 0, s,
                       out->arr_ticks_dev, n_req, tot, nb);
  }
  return hip_check(hipGetLastError(), "cf_trace_gen launch");
}
