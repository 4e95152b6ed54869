// cf_fine.h -- what the request-level simulator's kernels share: the launch's
// arguments, the layout of a wavefront's memory, and wavefront primitives.
#pragma once
#include "cf_internal.h"

namespace cf {
namespace fine {

constexpr int kMaxSI = CF_MAX_EXEC * CF_MAX_COMP;  // stage instances
static_assert(kMaxSI <= 512, "an LLM stage instance index fits the 9 bits of a gate word");
constexpr int kChunk = 64;                          // queue chunk entries

constexpr uint32_t kNone = 0xFFFFFFFFu;

enum { IT_BATCH = 0, IT_PREFILL = 1, IT_DECODE = 2, IT_FINISH = 3 };
enum { DL_DELIVER = 0, DL_TICK = 1 };

// a delay-line entry: due time and what is delivered (one 16-byte block)
struct __attribute__((aligned(16))) DlEnt {
  double t;
  uint32_t v, pad;
};

struct Layout {
  size_t req;
  size_t run, hist, mem, dl, pool, pool_next, pool_free;
  size_t bytes;
  int run_cap, hist_slots, n_chunks;
  uint32_t dl_mask;
};

struct FineArgs {
  KModel m;
  int P;
  const uint8_t *n_nodes, *node_comp, *node_rep, *node_gpus, *n_alt, *alt_w, *alt_node;
  const uint16_t *node_batch;
  const uint8_t *node_rep2, *node_gpus2, *node_w;  // a node's second configuration (NULL: none)
  const uint16_t *node_batch2;
  const int32_t *plan_ids;
  int n_plans;
  const double *rates;
  int K;
  const uint64_t *ticks, *rkey0, *rkey1;
  const uint8_t *type;
  const uint16_t *patches, *prompt, *out;
  const uint32_t *aud_in, *aud_out, *akey;
  int S, n;
  uint32_t *met, *cnt, *status;
  uint64_t *events;
  double *lat;
  const int32_t *lat_triples;
  int n_lat;
  uint32_t *hist;      // optional [n_plans][K][S][T][nb + 1] latency histograms
  const double *tg;    // their target table [T][nb][4]
  int nb;
  char *slab;
  Layout L;
  unsigned int *ticket;
  unsigned int total;
  int nsi_cap;  // stage instances provided in LDS
  int nl_cap, nt_cap;  // k_fine<true>: LLM stage instances and thinker ring slots provided in LDS
  uint64_t lim_instants;  // instants a simulation may take (a test limit; ~0 = none)
  // order in which a seed's (plan, rate) pairs are taken: entry j is i * K + k
  // (null: rate index first, then plan)
  const uint32_t *order;
};

// a queue end, chunk c (-1: none) and position p <= kChunk in it, as one word
// (chunk indices stay below 2^25: at most 2^26 requests on 8 components)
__device__ __forceinline__ uint32_t qend(int c, int p) { return ((uint32_t)(c + 1) << 7) | (uint32_t)p; }
__device__ __forceinline__ int qend_chunk(uint32_t w) { return (int)(w >> 7) - 1; }
__device__ __forceinline__ int qend_pos(uint32_t w) { return (int)(w & 127u); }

__device__ __forceinline__ int lane_id() { return threadIdx.x; }
__device__ __forceinline__ uint32_t ru(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int ri(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t ru64(uint64_t v) {
  return ((uint64_t)ru((uint32_t)(v >> 32)) << 32) | ru((uint32_t)v);
}
__device__ __forceinline__ double rdb(double v) {
  return __longlong_as_double((long long)ru64((uint64_t)__double_as_longlong(v)));
}
// the value lane x holds (x wave-uniform)
__device__ __forceinline__ double lane_val(double v, int x) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), x);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t bal) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
}
// wavefront minimum of a u32 through DPP row shifts and row broadcasts
// (identity ~0 for lanes whose source is out of range); result in lane 63
__device__ __forceinline__ uint32_t dpp_min_u32(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x113, 0xf, 0xf, false));  // row_shr:3
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x114, 0xf, 0xe, false));  // row_shr:4
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x118, 0xf, 0xc, false));  // row_shr:8
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast:15
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)~0u, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// minimum of non-negative doubles (or +inf) over the wavefront: the bit
// patterns of such doubles order like the values, so the high words are
// reduced first and the low words among the lanes holding that high word
__device__ __forceinline__ double wave_min_time(double t) {
  const uint64_t b = (uint64_t)__double_as_longlong(t);
  const uint32_t hi = dpp_min_u32((uint32_t)(b >> 32));
  const uint32_t lo = dpp_min_u32((uint32_t)(b >> 32) == hi ? (uint32_t)b : ~0u);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// inclusive prefix sum over the lanes through DPP: row_shr 1, 2, 4, 8 scan
// each row of 16 lanes (identity 0 where the source is out of range), then
// row_bcast 15 and row_bcast 31 carry the row totals into the later rows.
// Needs every lane active.
__device__ __forceinline__ uint32_t dpp_scan_add(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}
// wavefront sum (uniform result)
__device__ __forceinline__ uint32_t dpp_sum_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)dpp_scan_add(v), 63);
}
// exclusive prefix sum of v over the lanes, and the total
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t &total) {
  const uint32_t x = dpp_scan_add(v);
  total = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  return x - v;
}

// Device memory (global address space) addressed by a 32-bit byte offset
// from a base held in scalar registers: loads and stores take the
// scalar-base + vector-offset form, with no 64-bit address arithmetic per
// lane.  What is indexed this way is at most 4 GiB: parts of a wavefront's memory
// and one seed's part of a trace array.
#define CF_GLOBAL __attribute__((address_space(1)))
template <typename T>
struct GPtr {
  CF_GLOBAL T *p;
  __device__ __forceinline__ CF_GLOBAL T &operator[](uint32_t i) const {
    return *(CF_GLOBAL T *)((CF_GLOBAL char *)p + i * (uint32_t)sizeof(T));
  }
  __device__ __forceinline__ GPtr operator+(uint32_t i) const { return GPtr{&(*this)[i]}; }
};
template <typename T>
__device__ __forceinline__ GPtr<T> gptr_at(char *base, size_t off) {
  return GPtr<T>{(CF_GLOBAL T *)(base + off)};
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// element o of a trace array, which may hold any number of seeds.  An arrival in
// k_fine and the 64 of k_fine_gate's blocks form their nine addresses per lane from
// one element number: with a base per array in scalar registers (below) more
// registers spill there: 28 triples of 3,000 requests in k_fine_gate 516 -> 528 ms, in
// k_fine<true> 608 -> 614 ms; 24,576 triples of 1,000 in k_fine<false> 69.7 -> 70.3 ms.
template <typename T>
__device__ __forceinline__ T gload(const T *p, size_t o) {
  return *(const CF_GLOBAL T *)(p + o);
}

// k_fine_reg: element i of a trace array's part from element off on (wave-uniform: the
// seed's first request).  The part's address is formed in 64 bits, because the
// array may hold any number of seeds; i is a request of one seed, at most 2^26
// elements of 8 bytes, so that its offset fits 32 bits.
template <typename T>
__device__ __forceinline__ T gload(const T *p, size_t off, uint32_t i) {
  const CF_GLOBAL char *part = (const CF_GLOBAL char *)(p + off);
  // kept in scalar registers: without this the compiler adds offsets per lane
  // (24 triples of 1,000 requests 7.95 ms, with it 7.77; 7.90 by element numbers)
  asm("" : "+s"(part));
  return *(const CF_GLOBAL T *)(part + i * (uint32_t)sizeof(T));
}

// k_fine_reg.hip: the simulator with its whole control state in registers, for
// launches of models without a gated stage whose plans have at most
// kRegStages stage instances.  args: the launch's FineArgs in device memory.
constexpr int kRegStages = 64;
void launch_fine_reg(const FineArgs *args, unsigned waves, hipStream_t s);

// k_fine_gate.hip: the same for models whose only LLM components are one gate
// source and the one component gated by it.
bool fine_gate_takes(const KModel &m);
void launch_fine_gate(const FineArgs *args, int n_comp, unsigned waves, hipStream_t s);

}  // namespace fine
}  // namespace cf
