// k_enum.hip -- cf_enum_logical, cf_enum_count, cf_enum_plans: plan
// enumeration (Sec. 4.2, Alg. 1) and the executor partitions of Eq. (1).
//
// Logical plans are few (hundreds to thousands) and are built on the host.
// Physical plans are many (a logical plan of five nodes on 64 GPUs has
// billions), so they are numbered and produced on the device by unranking:
//   - per logical plan, cnt[v][b] = number of executor assignments of nodes
//     v.. within b GPUs (one block per logical plan, the budgets across
//     threads, the nodes from the last to the first), kept as its running
//     sums over b (cum_row), or itself where nodes hold two configurations;
//   - offsets = exclusive prefix sum of cnt[0][N] * 9^(types with two
//     alternatives);
//   - four consecutive plan indices per thread: for each, the logical plan by
//     counting the offsets once per block, the routing weights as base-9
//     digits of the index within it, the executor assignment by walking the
//     table (at node v with budget b, the candidates (k, n) in order each own
//     cnt[v+1][b - gpus_k n] consecutive numbers); the plan-table columns
//     are written slot-major, four plans per 32-bit store, so a wavefront
//     fills 256 consecutive bytes of a slot row per store instruction.
#include "cf_internal.h"
#include "cf_phase1.h"

#include <algorithm>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace cf {
namespace {

constexpr int kEnumMaxN = 64;                       // GPU budget limit (executors per plan)
constexpr int kTabStride = kEnumMaxN + 1;           // budgets 0..N
constexpr int kTabSize = (CF_MAX_NODES + 1) * kTabStride;  // u64 entries per logical plan

cf_status check_opts(const cf_model_desc *d, const cf_enum_opts *o) {
  if (!d || !o) return set_error(CF_EINVAL, "NULL argument");
  if (d->n_comp < 1 || d->n_comp > CF_MAX_COMP || d->n_types < 1 || d->n_types > CF_MAX_TYPES)
    return set_error(CF_EINVAL, "model sizes");
  if (o->n_gpus < 1 || o->n_gpus > kEnumMaxN) return set_error(CF_EINVAL, "n_gpus must be in 1..%d", kEnumMaxN);
  if (o->k_s < 1 || o->k_s > 2) return set_error(CF_EINVAL, "k_s must be 1 or 2");
  if (o->het != 0 && o->het != 1) return set_error(CF_EINVAL, "het must be 0 or 1");
  for (int c = 0; c < d->n_comp; c++) {
    if (o->n_batch[c] < 1 || o->n_batch[c] > 8) return set_error(CF_EINVAL, "n_batch[%d]", c);
    for (int k = 0; k < o->n_batch[c]; k++)
      if (o->batch[c][k] < 1 || o->batch[c][k] > CF_MAX_BATCH) return set_error(CF_EINVAL, "batch[%d][%d]", c, k);
    if (o->n_gpu_opt[c] < 1 || o->n_gpu_opt[c] > 4) return set_error(CF_EINVAL, "n_gpu_opt[%d]", c);
    for (int k = 0; k < o->n_gpu_opt[c]; k++)
      if (o->gpu_opt[c][k] < 1 || o->gpu_opt[c][k] > o->n_gpus) return set_error(CF_EINVAL, "gpu_opt[%d][%d]", c, k);
  }
  return CF_OK;
}

// ------------------------------------------------------------------ host: logical plans
struct Subplan {
  uint32_t cs, cov;
  std::vector<uint8_t> nodes;  // ascending masks
  int node_of(int c) const {
    for (size_t k = 0; k < nodes.size(); k++)
      if ((nodes[k] >> c) & 1u) return (int)k;
    return -1;
  }
};

int uf_find(int *par, int x) {
  while (par[x] != x) {
    par[x] = par[par[x]];
    x = par[x];
  }
  return x;
}

std::string plan_key(const cf_logical &L, int T) {
  std::string k;
  k.push_back((char)L.n_nodes);
  for (int v = 0; v < L.n_nodes; v++) k.push_back((char)L.node_comp[v]);
  for (int t = 0; t < T; t++) {
    k.push_back((char)L.n_alt[t]);
    for (int a = 0; a < L.n_alt[t]; a++)
      for (int c = 0; c < CF_MAX_COMP; c++) k.push_back((char)L.alt_node[t][a][c]);
  }
  return k;
}

void route_type(cf_logical &L, int t, int a, uint32_t path, const Subplan &s, const int *node_map) {
  for (int c = 0; c < CF_MAX_COMP; c++)
    if ((path >> c) & 1u) L.alt_node[t][a][c] = (uint8_t)node_map[s.node_of(c)];
}

// ------------------------------------------------------------------ device
struct EnumView {
  int N;
  const cf_logical *logical;
  int n_logical;
  int ng;             // most GPU options of a component
  uint64_t *tab;      // [n_logical][tab_size]: cum_row rows, or cnt[v][b] with second configurations (NULL: not kept)
  uint64_t *totals;   // [n_logical]
};

// u64 entries of one logical plan's table: 8.8 KB with second configurations, else 8.3 KB per GPU
// option (33 KB for four)
__host__ __device__ __forceinline__ size_t tab_size(bool het, int ng) {
  return het ? (size_t)kTabSize : (size_t)CF_MAX_NODES * ng * kTabStride;
}

// Node v, GPU option gi of plan l's table: row[b] = the assignments of nodes v.. within b GPUs
// whose node v takes option gi and one given batch size, the sum of cnt[v+1][b - g n] over
// n >= 1.  row[b] - row[b - g n] of them have at most n executors at v, so a rank's batch size
// follows from whole rows and its n from a binary search, instead of one table read per
// (batch size, n) passed over.
__device__ __forceinline__ const uint64_t *cum_row(const EnumView &V, int l, int v, int gi) {
  return V.tab + (size_t)l * tab_size(false, V.ng) + (size_t)((v * V.ng + gi) * kTabStride);
}

__device__ __forceinline__ uint64_t sat_add(uint64_t a, uint64_t b) { return a > ~0ull - b ? ~0ull : a + b; }
__device__ __forceinline__ uint64_t sat_mul(uint64_t a, uint64_t b) { return (b && a > ~0ull / b) ? ~0ull : a * b; }

// The option tables a node indexes by its lowest component, staged in LDS.
struct OptsLds {
  uint8_t n_batch[CF_MAX_COMP], n_gpu[CF_MAX_COMP];
  uint8_t gpu[CF_MAX_COMP][4];
  uint16_t batch[CF_MAX_COMP][8];
};

__device__ void stage_opts(OptsLds &s, const cf_enum_opts &o, int tid, int nthreads) {
  for (int i = tid; i < CF_MAX_COMP; i += nthreads) {
    s.n_batch[i] = (uint8_t)o.n_batch[i];
    s.n_gpu[i] = (uint8_t)o.n_gpu_opt[i];
    for (int k = 0; k < 4; k++) s.gpu[i][k] = o.gpu_opt[i][k];
    for (int k = 0; k < 8; k++) s.batch[i][k] = o.batch[i][k];
  }
}

// One block per logical plan: cnt[v][b], then the plan's total.  Counting a space
// needs the totals only and keeps no table: the rows of four GPU options are 3.8
// times the bytes of cnt, and writing them took cf_enum_count of 745 logical plans
// on 24 GPUs 68 us instead of 64.
__global__ void __launch_bounds__(128) k_enum_table(cf_enum_opts o, EnumView V) {
  __shared__ OptsLds so;
  __shared__ uint64_t cnt[CF_MAX_NODES + 1][kTabStride];
  const int l = blockIdx.x, b = threadIdx.x;
  stage_opts(so, o, threadIdx.x, blockDim.x);
  const cf_logical &L = V.logical[l];
  const int nv = L.n_nodes <= CF_MAX_NODES ? L.n_nodes : CF_MAX_NODES;
  uint64_t *out = V.tab ? V.tab + (size_t)l * tab_size(o.het, V.ng) : nullptr;
  if (b <= V.N) cnt[nv][b] = 1;
  __syncthreads();
  for (int v = nv - 1; v >= 0; v--) {
    if (b <= V.N) {
      const int c0 = L.node_comp[v] ? __ffs(L.node_comp[v]) - 1 : 0;
      uint64_t tot = 0;
      for (int gi = 0; gi < so.n_gpu[c0]; gi++) {
        const int g = so.gpu[c0][gi];
        uint64_t per_cfg = 0;
        for (int n = 1; g * n <= b; n++) per_cfg = sat_add(per_cfg, cnt[v + 1][b - g * n]);
        if (!o.het && out) out[(v * V.ng + gi) * kTabStride + b] = per_cfg;
        for (int bi = 0; bi < so.n_batch[c0]; bi++) tot = sat_add(tot, per_cfg);
      }
      if (o.het) {
        // two configurations k1 < k2 (GPU option major, batch minor), n1, n2 >= 1, 9 weights
        const int nb = so.n_batch[c0], K = so.n_gpu[c0] * nb;
        for (int k1 = 0; k1 < K; k1++)
          for (int k2 = k1 + 1; k2 < K; k2++) {
            const int g1 = so.gpu[c0][k1 / nb], g2 = so.gpu[c0][k2 / nb];
            for (int n1 = 1; g1 * n1 + g2 <= b; n1++)
              for (int n2 = 1; g1 * n1 + g2 * n2 <= b; n2++)
                tot = sat_add(tot, sat_mul(9, cnt[v + 1][b - g1 * n1 - g2 * n2]));
          }
      }
      cnt[v][b] = tot;
    }
    __syncthreads();
  }
  if (o.het && out)
    for (int i = threadIdx.x; i < (nv + 1) * kTabStride; i += blockDim.x) out[i] = (&cnt[0][0])[i];
  if (threadIdx.x == 0) {
    uint64_t tot = cnt[0][V.N];
    for (int t = 0; t < CF_MAX_TYPES; t++)
      if (L.n_alt[t] == 2) tot = sat_mul(tot, 9);
    V.totals[l] = tot;
  }
}

// offsets[0] = 0, offsets[l+1] = offsets[l] + totals[l] (saturating); one block.
__global__ void __launch_bounds__(1024) k_enum_offsets(const uint64_t *totals, int n, uint64_t *offsets) {
  __shared__ uint64_t part[1024];
  __shared__ uint64_t carry_s;
  const int tid = threadIdx.x;
  if (tid == 0) {
    carry_s = 0;
    offsets[0] = 0;
  }
  __syncthreads();
  for (int base = 0; base < n; base += 1024) {
    const uint64_t x = base + tid < n ? totals[base + tid] : 0;
    part[tid] = x;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
      const uint64_t add = tid >= d ? part[tid - d] : 0;
      __syncthreads();
      part[tid] = sat_add(part[tid], add);
      __syncthreads();
    }
    if (base + tid < n) offsets[base + tid + 1] = sat_add(carry_s, part[tid]);
    __syncthreads();
    if (tid == 1023) carry_s = sat_add(carry_s, part[1023]);
    __syncthreads();
  }
}

struct PlanOut {
  int P;
  uint8_t *n_nodes, *node_comp, *node_rep, *node_gpus, *n_alt, *alt_w, *alt_node;
  uint16_t *node_batch;
  uint8_t *node_rep2, *node_gpus2, *node_w;  // second configurations (NULL: not written)
  uint16_t *node_batch2;
};

// The position of plan idx: its logical plan, routing digits and the cursor
// of the executor-assignment walk.
struct Cursor {
  int l, nv;
  bool ok;
  uint64_t q;   // rank among the executor assignments still to place
  int b;        // GPUs left
  uint32_t w;   // routing weights, 4 bits per type with two alternatives, in type order
};

// What the consecutive plans of a block share.  Spaces hold many plans per logical plan, so a
// block nearly always lies within one: its rank is divided by the routing digits once, a
// thread's plan follows by 32-bit arithmetic, and the plan's record is read from LDS.
struct BlockPos {
  int lo, hi;        // logical plans of the block's first and last plan
  uint32_t R, r0;    // 9^(types with two alternatives) of lo, and the first plan's routing rank
  uint64_t q0;       // the first plan's executor-assignment rank
  int na2;
  alignas(8) uint8_t route[CF_MAX_TYPES][2][CF_MAX_COMP];  // lo's record
  uint8_t comp[CF_MAX_NODES], n_alt[CF_MAX_TYPES];
  uint8_t nv;
};

// Fills bp for the plans first..last (last < offsets[n_logical]); all threads of the block, ends
// with a barrier.  offsets[l] never decreases: the plan's logical plan is the number of
// offsets up to its index, less one, counted by all threads at once.
__device__ __forceinline__ void block_pos(BlockPos &bp, const EnumView &V, const uint64_t *offsets, uint64_t first,
                                          uint64_t last) {
  const int tid = threadIdx.x;
  if (tid == 0) bp.lo = bp.hi = -1;
  __syncthreads();
  int nlo = 0, nhi = 0;
  for (int base = 0; base < V.n_logical; base += blockDim.x) {
    const uint64_t x = base + tid < V.n_logical ? offsets[base + tid] : ~0ull;
    nlo += __popcll(__ballot(base + tid < V.n_logical && x <= first));
    nhi += __popcll(__ballot(base + tid < V.n_logical && x <= last));
  }
  if ((tid & 63) == 0) {
    atomicAdd(&bp.lo, nlo);
    atomicAdd(&bp.hi, nhi);
  }
  __syncthreads();
  if (tid == 0) {
    if (bp.lo < 0) bp.lo = 0;
    if (bp.hi < bp.lo) bp.hi = bp.lo;
  }
  __syncthreads();
  const cf_logical &L = V.logical[bp.lo];
  for (int i = tid; i < CF_MAX_TYPES * 2 * CF_MAX_COMP; i += blockDim.x)
    (&bp.route[0][0][0])[i] = (&L.alt_node[0][0][0])[i];
  if (tid < CF_MAX_NODES) bp.comp[tid] = L.node_comp[tid];
  if (tid < CF_MAX_TYPES) bp.n_alt[tid] = L.n_alt[tid];
  if (tid == 0) {
    bp.nv = L.n_nodes;
    int na2 = 0;
    for (int t = 0; t < CF_MAX_TYPES; t++) na2 += L.n_alt[t] == 2;
    uint32_t R = 1;
    for (int i = 0; i < na2; i++) R *= 9;
    const uint64_t local = first - offsets[bp.lo];
    bp.na2 = na2;
    bp.R = R;
    bp.q0 = local / R;
    bp.r0 = (uint32_t)(local - bp.q0 * R);
  }
  __syncthreads();
}

__device__ __forceinline__ void set_digits(Cursor &c, uint32_t r, int na2) {
  c.w = 0;
  for (int i = na2 - 1; i >= 0; i--) {  // lowest type is the most significant digit
    c.w |= (r % 9 + 1) << (4 * i);
    r /= 9;
  }
}

// The cursor of the block's plan number d (index idx = first + d).
__device__ Cursor locate(const EnumView &V, const uint64_t *offsets, const BlockPos &bp, uint64_t idx, uint32_t d,
                         bool valid) {
  Cursor c;
  c.b = V.N;
  c.ok = valid && idx < offsets[V.n_logical];
  c.l = bp.lo;
  if (bp.lo == bp.hi) {  // one logical plan in the block
    const uint32_t x = bp.r0 + d, dq = x / bp.R;  // below 9^8 + the block's plans
    c.nv = c.ok ? bp.nv : 0;
    c.q = bp.q0 + dq;
    set_digits(c, x - dq * bp.R, bp.na2);
    return c;
  }
  int lo = bp.lo, hi = bp.hi + 1;  // offsets[lo] <= idx < offsets[hi]
  if (c.ok) {
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (offsets[mid] <= idx) lo = mid; else hi = mid;
    }
  }
  c.l = lo;
  const cf_logical &L = V.logical[lo];
  c.nv = c.ok ? L.n_nodes : 0;
  const uint64_t local = c.ok ? idx - offsets[lo] : 0;
  int na2 = 0;
  for (int t = 0; t < CF_MAX_TYPES; t++) na2 += L.n_alt[t] == 2;
  uint32_t R = 1;
  for (int i = 0; i < na2; i++) R *= 9;
  c.q = local / R;
  set_digits(c, (uint32_t)(local - c.q * R), na2);
  return c;
}

struct NodeCfg {
  uint8_t comp, rep, gpus;
  uint16_t batch;
  uint8_t rep2, gpus2, w;  // a second configuration (rep2 = 0: none, w = 10)
  uint16_t batch2;
};

// Node v (component set comp) of the plan at cursor c in a space of one configuration per node:
// the candidates (GPU option gi, batch size bi, n) in order own cnt[v+1][b - gpus_gi n]
// consecutive ranks each.  False: no candidate holds the rank.  step: the largest power of two
// up to the GPU budget.
__device__ __forceinline__ bool place_one(const EnumView &V, const OptsLds &so, Cursor &c, int v, int comp, int step,
                                          int &c0, int &gi, int &bi, int &n) {
  c0 = comp ? __ffs(comp) - 1 : 0;
  const int nb = so.n_batch[c0];
  for (gi = 0; gi < so.n_gpu[c0]; gi++) {
    const uint64_t *row = cum_row(V, c.l, v, gi);
    const uint64_t S = row[c.b];
    bi = 0;
    while (bi < nb && c.q >= S) {
      c.q -= S;
      bi++;
    }
    if (bi == nb) continue;
    // most executors passed over: row[b - g t] >= S - q holds up to it and for no larger t
    const int g = so.gpu[c0][gi];
    const uint64_t left = S - c.q;
    int t = 0;
    uint64_t at = S;
    for (int d = step; d; d >>= 1) {
      const int bb = c.b - g * (t + d);
      const uint64_t x = bb >= 0 ? row[bb] : 0ull;
      if (x >= left) {
        t += d;
        at = x;
      }
    }
    c.q -= S - at;
    n = t + 1;
    c.b -= g * n;
    return true;
  }
  return false;
}

// Node v of the plan at cursor c; with het (a table of cnt) the candidates (k, n), then the
// candidates (k1, k2, n1, n2, w), which own cnt[v+1][b - gpus_k1 n1 - gpus_k2 n2] each.
__device__ NodeCfg place(const EnumView &V, const OptsLds &so, const BlockPos &bp, Cursor &c, int v, bool het,
                         int step) {
  NodeCfg r = {0, 0, 0, 0, 0, 0, 10, 0};
  if (v >= c.nv) return r;
  r.comp = bp.lo == bp.hi ? bp.comp[v] : V.logical[c.l].node_comp[v];
  if (!het) {
    int k0, gi, bi, n;
    if (place_one(V, so, c, v, r.comp, step, k0, gi, bi, n)) {
      r.rep = (uint8_t)n;
      r.gpus = so.gpu[k0][gi];
      r.batch = so.batch[k0][bi];
    }
    return r;
  }
  const uint64_t *tab = V.tab + (size_t)c.l * kTabSize + (size_t)(v + 1) * kTabStride;
  const int c0 = r.comp ? __ffs(r.comp) - 1 : 0;
  const int nb = so.n_batch[c0];
  for (int gi = 0; gi < so.n_gpu[c0]; gi++) {
    const int g = so.gpu[c0][gi];
    for (int bi = 0; bi < nb; bi++) {
      for (int n = 1; g * n <= c.b; n++) {
        const uint64_t k = tab[c.b - g * n];
        if (c.q < k) {
          r.rep = (uint8_t)n;
          r.gpus = (uint8_t)g;
          r.batch = so.batch[c0][bi];
          c.b -= g * n;
          return r;
        }
        c.q -= k;
      }
    }
  }
  if (het) {
    const int K = so.n_gpu[c0] * nb;
    for (int k1 = 0; k1 < K; k1++)
      for (int k2 = k1 + 1; k2 < K; k2++) {
        const int g1 = so.gpu[c0][k1 / nb], g2 = so.gpu[c0][k2 / nb];
        for (int n1 = 1; g1 * n1 + g2 <= c.b; n1++)
          for (int n2 = 1; g1 * n1 + g2 * n2 <= c.b; n2++) {
            const uint64_t k = tab[c.b - g1 * n1 - g2 * n2];
            const uint64_t k9 = sat_mul(k, 9);  // the nine weights, k ranks each
            if (c.q < k9) {
              const uint64_t wi = c.q / k;
              c.q -= wi * k;
              r.rep = (uint8_t)n1;
              r.gpus = (uint8_t)g1;
              r.batch = so.batch[c0][k1 % nb];
              r.rep2 = (uint8_t)n2;
              r.gpus2 = (uint8_t)g2;
              r.batch2 = so.batch[c0][k2 % nb];
              r.w = (uint8_t)(wi + 1);
              c.b -= g1 * n1 + g2 * n2;
              return r;
            }
            c.q -= k9;
          }
      }
  }
  return r;
}

// Four consecutive plans per thread, each slot row written with one 32-bit
// store (64-bit for the batch row): a wavefront writes 256 bytes of a row
// per instruction.  Needs out.P % 4 == 0; the last thread writes bytes.
// HET: the space has nodes of two configurations (o.het); without them the
// walk over configuration pairs is not compiled in.
// Bound by the vector-memory issue rate: a byte load of the logical plan's
// record per plan and route slot (512 a thread) took longer than the 233 B
// written per plan.  With the block's record in LDS, the plan index divided
// once per block and the walk by binary search, 2,000,000 omni plans and
// their phase 1 take 389 us instead of 482 (16 GPUs, three batch sizes).
constexpr int kPlansPerThread = 4;
template <bool HET>
__global__ void __launch_bounds__(256) k_enum_unrank(cf_enum_opts o, EnumView V, const uint64_t *offsets,
                                                    uint64_t first, int count, PlanOut out) {
  __shared__ OptsLds so;
  __shared__ BlockPos bp;
  stage_opts(so, o, threadIdx.x, blockDim.x);
  const int pb = blockIdx.x * blockDim.x * kPlansPerThread;  // the block's first plan
  const int pe = min(count - pb, (int)blockDim.x * kPlansPerThread);
  block_pos(bp, V, offsets, first + (uint64_t)pb, first + (uint64_t)(pb + pe - 1));
  const int p0 = pb + threadIdx.x * kPlansPerThread;
  if (p0 >= count) return;
  const bool one = bp.lo == bp.hi;
  const int step = 1 << (31 - __clz(V.N));
  const size_t P = (size_t)out.P;
  const bool packed = p0 + kPlansPerThread <= count && (out.P % kPlansPerThread) == 0;
  // consecutive plans of one logical plan that differ only in their routing
  // weights share the executor assignment: it is walked once
  Cursor cur[kPlansPerThread];
  bool same[kPlansPerThread];
#pragma unroll
  for (int j = 0; j < kPlansPerThread; j++) {
    cur[j] = locate(V, offsets, bp, first + (uint64_t)(p0 + j), (uint32_t)(p0 + j - pb), p0 + j < count);
    same[j] = j > 0 && cur[j].ok && cur[j - 1].ok && cur[j].l == cur[j - 1].l && cur[j].q == cur[j - 1].q;
  }
  auto put8 = [&](uint8_t *row, const uint8_t *x) {
    if (packed) {
      *(uint32_t *)(row + p0) = (uint32_t)x[0] | ((uint32_t)x[1] << 8) | ((uint32_t)x[2] << 16) | ((uint32_t)x[3] << 24);
    } else {
      for (int j = 0; j < kPlansPerThread; j++)
        if (p0 + j < count) row[p0 + j] = x[j];
    }
  };
  uint8_t b8[kPlansPerThread];
#pragma unroll
  for (int j = 0; j < kPlansPerThread; j++) b8[j] = (uint8_t)cur[j].nv;
  put8(out.n_nodes, b8);
  for (int v = 0; v < CF_MAX_NODES; v++) {
    NodeCfg nc[kPlansPerThread];
#pragma unroll
    for (int j = 0; j < kPlansPerThread; j++) nc[j] = same[j] ? nc[j - 1] : place(V, so, bp, cur[j], v, HET, step);
#pragma unroll
    for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].comp;
    put8(out.node_comp + v * P, b8);
#pragma unroll
    for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].rep;
    put8(out.node_rep + v * P, b8);
#pragma unroll
    for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].gpus;
    put8(out.node_gpus + v * P, b8);
    uint16_t *brow = out.node_batch + v * P;
    if (packed) {
      *(uint64_t *)(brow + p0) = (uint64_t)nc[0].batch | ((uint64_t)nc[1].batch << 16) |
                                 ((uint64_t)nc[2].batch << 32) | ((uint64_t)nc[3].batch << 48);
    } else {
      for (int j = 0; j < kPlansPerThread; j++)
        if (p0 + j < count) brow[p0 + j] = nc[j].batch;
    }
    if (out.node_rep2) {
#pragma unroll
      for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].rep2;
      put8(out.node_rep2 + v * P, b8);
#pragma unroll
      for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].gpus2;
      put8(out.node_gpus2 + v * P, b8);
#pragma unroll
      for (int j = 0; j < kPlansPerThread; j++) b8[j] = nc[j].w;
      put8(out.node_w + v * P, b8);
      uint16_t *b2row = out.node_batch2 + v * P;
      for (int j = 0; j < kPlansPerThread; j++)
        if (p0 + j < count) b2row[p0 + j] = nc[j].batch2;
    }
  }
  int i2[kPlansPerThread] = {0, 0, 0, 0};
  for (int t = 0; t < CF_MAX_TYPES; t++) {
    uint8_t na[kPlansPerThread], w0[kPlansPerThread], w1[kPlansPerThread];
#pragma unroll
    for (int j = 0; j < kPlansPerThread; j++) {
      na[j] = cur[j].ok ? (one ? bp.n_alt[t] : V.logical[cur[j].l].n_alt[t]) : 0;
      w0[j] = na[j] == 1 ? 10 : 0;
      w1[j] = 0;
      if (na[j] == 2) {
        w0[j] = (uint8_t)((cur[j].w >> (4 * i2[j])) & 15u);
        w1[j] = (uint8_t)(10 - w0[j]);
        i2[j]++;
      }
    }
    put8(out.n_alt + t * P, na);
    put8(out.alt_w + (2 * t) * P, w0);
    put8(out.alt_w + (2 * t + 1) * P, w1);
    for (int a = 0; a < 2; a++) {
      if (one) {  // eight routes in one LDS read, each written for the four plans at once
        const uint64_t r8 = *(const uint64_t *)bp.route[t][a];
#pragma unroll
        for (int c = 0; c < CF_MAX_COMP; c++) {
#pragma unroll
          for (int j = 0; j < kPlansPerThread; j++) b8[j] = cur[j].ok ? (uint8_t)(r8 >> (8 * c)) : (uint8_t)255;
          put8(out.alt_node + ((2 * t + a) * CF_MAX_COMP + c) * P, b8);
        }
        continue;
      }
      for (int c = 0; c < CF_MAX_COMP; c++) {
#pragma unroll
        for (int j = 0; j < kPlansPerThread; j++)
          b8[j] = cur[j].ok ? V.logical[cur[j].l].alt_node[t][a][c] : (uint8_t)255;
        put8(out.alt_node + ((2 * t + a) * CF_MAX_COMP + c) * P, b8);
      }
    }
  }
}

// Enumeration fused with phase 1: a thread numbers its plan, builds the
// plan's nodes and routes in registers and LDS exactly as k_enum_unrank
// would write them, and screens it as k_coarse would read them, writing only
// R_d, the bottleneck and the flags (13 B per plan instead of the 233 B
// table written and read back).
//
// A plan's batch size and GPUs per executor are options of the space, so the work per request
// of every (type, component, option) is computed once per block into LDS (work_s, two
// divisions each), and the routing shares (pq_s) likewise.  TAB: off where the options are so
// many that the table would take more than kWorkBytes; the work is then computed per plan.
// Issue-bound: linear walks over (batch size, n), 64-bit divisions by the routing digits and two
// fp64 divisions per term were most of it.  10^7 omni plans in three windows, selections
// included: 1,978 -> 1,188 us.
constexpr int kScrBlock = 256;
constexpr int kWorkBytes = 16384;
struct ScreenPrep {
  double ex[CF_MAX_TYPES][CF_MAX_COMP], en[CF_MAX_TYPES][CF_MAX_COMP];
  uint16_t opt_b[CF_MAX_COMP * 32];  // an option's batch size and multiplier index
  uint8_t opt_g[CF_MAX_COMP * 32];
};
template <bool TAB>
__global__ void __launch_bounds__(kScrBlock) k_enum_screen(cf_enum_opts o, EnumView V, const uint64_t *offsets,
                                                          uint64_t first, int count, KModel m, const uint64_t *moments,
                                                          int n_gpus, int n_opt, double *rd, int32_t *bott,
                                                          uint8_t *flags) {
  __shared__ OptsLds so;
  __shared__ BlockPos bp;
  __shared__ double pq_s[CF_MAX_TYPES][10];  // pi_t q: [w] for w of ten tenths, [0] for one alternative
  __shared__ double u_s[CF_MAX_NODES][kScrBlock];
  __shared__ uint8_t k_s[CF_MAX_NODES][kScrBlock];  // a node's option, opt_base[c0] + gi nb + bi
  __shared__ uint16_t opt_base[CF_MAX_COMP];
  extern __shared__ double work_s[];            // TAB: [t][c][option]
  // with the table these are read before u_s is written and take its place: 38 KB and the
  // table (2.4 KB for the omni model with three batch sizes and one GPU option, four blocks per
  // CU; at most 16 KB, two blocks)
  ScreenPrep *pr;
  if constexpr (TAB) {
    pr = (ScreenPrep *)&u_s[0][0];
  } else {
    __shared__ ScreenPrep own;
    pr = &own;
  }
  const int tid = threadIdx.x;
  stage_opts(so, o, tid, blockDim.x);
  phase1_means(m, moments, tid, pr->ex, pr->en);
  if (tid < m.nt * 10) {
    const int t = tid / 10, w = tid % 10;
    const double pi = (double)m.weight[t] / (double)m.wsum;
    pq_s[t][w] = pi * (w ? (double)w / 10.0 : 1.0);
  }
  if (tid < m.nc) {  // the options of components before this one come first
    int base = 0;
    for (int c = 0; c < tid; c++) base += o.n_batch[c] * o.n_gpu_opt[c];
    opt_base[tid] = (uint16_t)base;
    for (int gi = 0; gi < o.n_gpu_opt[tid]; gi++)
      for (int bi = 0; bi < o.n_batch[tid]; bi++) {
        const int g = o.gpu_opt[tid][gi];
        pr->opt_b[base + gi * o.n_batch[tid] + bi] = o.batch[tid][bi];
        pr->opt_g[base + gi * o.n_batch[tid] + bi] = (uint8_t)(g > 8 ? 7 : g - 1);
      }
  }
  const int pb = blockIdx.x * kScrBlock;
  const int pe = min(count - pb, kScrBlock);
  block_pos(bp, V, offsets, first + (uint64_t)pb, first + (uint64_t)(pb + pe - 1));
  if constexpr (TAB) {
    for (int i = tid; i < m.nt * m.nc * n_opt; i += kScrBlock) {
      const int k = i % n_opt, c = (i / n_opt) % m.nc, t = i / (n_opt * m.nc);
      work_s[i] = phase1_work(m, c, pr->opt_b[k], pr->ex[t][c], pr->en[t][c], m.tps[c][pr->opt_g[k]]);
    }
    __syncthreads();
  }
  const int p = pb + tid;
  if (p >= count) return;
  Cursor cur = locate(V, offsets, bp, first + (uint64_t)p, (uint32_t)tid, true);
  const int nv = cur.nv;
  const bool one = bp.lo == bp.hi;
  const int step = 1 << (31 - __clz(V.N));
  uint32_t rep[CF_MAX_NODES], gp[CF_MAX_NODES];
#pragma unroll
  for (int v = 0; v < CF_MAX_NODES; v++) {
    rep[v] = gp[v] = 0;
    if (v < nv) {
      const int comp = one ? bp.comp[v] : V.logical[cur.l].node_comp[v];
      int c0, gi, bi, n;
      k_s[v][tid] = 0;
      if (place_one(V, so, cur, v, comp, step, c0, gi, bi, n)) {
        rep[v] = (uint8_t)n;
        gp[v] = so.gpu[c0][gi];
        k_s[v][tid] = (uint8_t)(opt_base[c0] + gi * so.n_batch[c0] + bi);
      }
      u_s[v][tid] = 0.0;
    }
  }
  if (!cur.ok || nv < 1) {
    rd[p] = 0.0;
    bott[p] = -1;
    flags[p] = CF_FLAG_INVALID;
    return;
  }
  const cf_logical &L = V.logical[cur.l];
  int i2 = 0;
  for (int t = 0; t < m.nt; t++) {
    const uint32_t path = m.path[t];
    const uint32_t na = one ? bp.n_alt[t] : L.n_alt[t];
    uint32_t wl[2] = {0u, 0u};  // tenths; 0 is the whole of one alternative
    if (na == 2) {
      wl[0] = (cur.w >> (4 * i2)) & 15u;
      wl[1] = 10u - wl[0];
      i2++;
    }
#pragma unroll
    for (int a = 0; a < 2; a++) {
      if (a < (int)na) {
        const double pq = pq_s[t][wl[a]];
        const uint64_t r8 = one ? *(const uint64_t *)bp.route[t][a] : 0ull;
#pragma unroll
        for (int c = 0; c < CF_MAX_COMP; c++) {
          if (!((path >> c) & 1u)) continue;
          const int v = one ? (int)((r8 >> (8 * c)) & 255u) : L.alt_node[t][a][c];
          const int k = k_s[v][tid];
          double w;
          if constexpr (TAB) w = work_s[(t * m.nc + c) * n_opt + k];
          else w = phase1_work(m, c, pr->opt_b[k], pr->ex[t][c], pr->en[t][c], m.tps[c][pr->opt_g[k]]);
          u_s[v][tid] = u_s[v][tid] + pq * w;
        }
      }
    }
  }
  phase1_result(nv, rep, gp, [&](int v) { return u_s[v][tid]; }, n_gpus, &rd[p], &bott[p], &flags[p]);
}

int most_gpu_options(const cf_enum_opts *o) {
  int ng = 1;
  for (int c = 0; c < CF_MAX_COMP; c++) ng = std::max(ng, std::min<int>(o->n_gpu_opt[c], 4));
  return ng;
}

// tab_out NULL: only the totals.  The scratch is sized for the table all the
// same, so that an enumeration after a count allocates nothing.
cf_status run_tables(const cf_enum_opts *opts, const cf_logical *logical_dev, int n_logical, uint64_t **tab_out,
                     uint64_t **totals_out, hipStream_t s) {
  cf_status st = CF_OK;
  const size_t per = tab_size(opts->het, most_gpu_options(opts));
  const size_t bytes = sizeof(uint64_t) * ((size_t)n_logical * per + (size_t)n_logical);
  uint64_t *scr = (uint64_t *)scratch_get(SCR_ENUM, bytes, &st);
  if (!scr) return st;
  EnumView V;
  V.N = opts->n_gpus;
  V.logical = logical_dev;
  V.n_logical = n_logical;
  V.tab = tab_out ? scr : nullptr;
  V.ng = most_gpu_options(opts);
  V.totals = scr + (size_t)n_logical * per;
  hipLaunchKernelGGL(k_enum_table, dim3((unsigned)n_logical), dim3(128), 0, s, *opts, V);
  st = hip_check(hipGetLastError(), "cf_enum table launch");
  if (tab_out) *tab_out = V.tab;
  *totals_out = V.totals;
  return st;
}

}  // namespace
}  // namespace cf

extern "C" cf_status cf_enum_logical(const cf_model_desc *model, const cf_enum_opts *opts, cf_logical *out_host,
                                     int32_t cap, int32_t *n_out) {
  using namespace cf;
  cf_status st = check_opts(model, opts);
  if (st != CF_OK) return st;
  if (!out_host || !n_out || cap < 0) return set_error(CF_EINVAL, "NULL output or cap < 0");
  *n_out = 0;
  const int T = model->n_types, C = model->n_comp;
  const uint32_t all_types = (1u << T) - 1u;
  // subgraphs: distinct unions of type paths, ascending
  std::set<uint32_t> subgraphs;
  for (uint32_t u = 1; u <= all_types; u++) {
    uint32_t cs = 0;
    for (int t = 0; t < T; t++)
      if ((u >> t) & 1u) cs |= model->path_mask[t];
    subgraphs.insert(cs);
  }
  // simple subplans
  std::vector<Subplan> S;
  for (uint32_t cs : subgraphs) {
    uint32_t cov = 0;
    for (int t = 0; t < T; t++)
      if (!(model->path_mask[t] & ~cs)) cov |= 1u << t;
    std::vector<std::pair<int, int>> edges;
    for (int p = 0; p < C; p++)
      for (int c = 0; c < C; c++) {
        if (!((opts->colocatable[p] >> c) & 1u)) continue;
        bool on = false;
        for (int t = 0; t < T && !on; t++) on = ((cov >> t) & 1u) && ((model->parents[t][c] >> p) & 1u);
        if (on) edges.emplace_back(p, c);
      }
    if (edges.size() > 16) return set_error(CF_ECAPACITY, "more than 16 colocatable edges in a subgraph");
    std::set<std::vector<uint8_t>> seen;
    for (uint32_t m = 0; m < (1u << edges.size()); m++) {
      int par[CF_MAX_COMP];
      for (int c = 0; c < CF_MAX_COMP; c++) par[c] = c;
      for (size_t i = 0; i < edges.size(); i++)
        if ((m >> i) & 1u) {
          const int ra = uf_find(par, edges[i].first), rb = uf_find(par, edges[i].second);
          if (ra != rb) par[std::max(ra, rb)] = std::min(ra, rb);
        }
      std::map<int, uint8_t> groups;
      for (int c = 0; c < CF_MAX_COMP; c++)
        if ((cs >> c) & 1u) groups[uf_find(par, c)] |= (uint8_t)(1u << c);
      std::vector<uint8_t> nodes;
      for (auto &g : groups) nodes.push_back(g.second);
      std::sort(nodes.begin(), nodes.end());
      if (!seen.insert(nodes).second) continue;
      S.push_back(Subplan{cs, cov, nodes});
    }
  }
  // logical plans
  std::set<std::string> emitted;
  int n = 0;
  auto emit = [&](const cf_logical &L) -> cf_status {
    if (!emitted.insert(plan_key(L, T)).second) return CF_OK;
    if (n >= cap) return set_error(CF_ECAPACITY, "more than %d logical plans", cap);
    out_host[n++] = L;
    return CF_OK;
  };
  auto blank = []() {
    cf_logical L;
    memset(&L, 0, sizeof L);
    memset(L.alt_node, 255, sizeof L.alt_node);
    return L;
  };
  for (const Subplan &s : S) {
    if (s.cov != all_types) continue;
    cf_logical L = blank();
    L.n_nodes = (uint8_t)s.nodes.size();
    int ident[CF_MAX_COMP];
    for (size_t v = 0; v < s.nodes.size(); v++) {
      L.node_comp[v] = s.nodes[v];
      ident[v] = (int)v;
    }
    for (int t = 0; t < T; t++) {
      L.n_alt[t] = 1;
      route_type(L, t, 0, model->path_mask[t], s, ident);
    }
    if ((st = emit(L)) != CF_OK) return st;
  }
  if (opts->k_s == 2) {
    for (size_t i = 0; i < S.size(); i++)
      for (size_t j = i; j < S.size(); j++) {
        const Subplan &A = S[i], &B = S[j];
        if ((A.cov | B.cov) != all_types) continue;
        std::vector<std::pair<int, int>> matchable;  // (node of B, equal node of A), in B's order
        for (size_t v = 0; v < B.nodes.size(); v++)
          for (size_t w = 0; w < A.nodes.size(); w++)
            if (B.nodes[v] == A.nodes[w]) matchable.emplace_back((int)v, (int)w);
        const uint32_t n_sets = opts->share ? (1u << matchable.size()) : 1u;
        for (uint32_t sh = 0; sh < n_sets; sh++) {
          if (opts->share && matchable.size() == B.nodes.size() && sh == n_sets - 1) continue;
          int amap[CF_MAX_COMP], bmap[CF_MAX_COMP];
          int nv = (int)A.nodes.size();
          for (int v = 0; v < nv; v++) amap[v] = v;
          for (size_t v = 0; v < B.nodes.size(); v++) bmap[v] = -1;
          for (size_t k = 0; k < matchable.size(); k++)
            if ((sh >> k) & 1u) bmap[matchable[k].first] = matchable[k].second;
          for (size_t v = 0; v < B.nodes.size(); v++)
            if (bmap[v] < 0) bmap[v] = nv++;
          if (nv > CF_MAX_NODES) continue;
          cf_logical L = blank();
          L.n_nodes = (uint8_t)nv;
          for (size_t v = 0; v < A.nodes.size(); v++) L.node_comp[v] = A.nodes[v];
          for (size_t v = 0; v < B.nodes.size(); v++) L.node_comp[bmap[v]] = B.nodes[v];
          for (int t = 0; t < T; t++) {
            const bool inA = (A.cov >> t) & 1u, inB = (B.cov >> t) & 1u;
            int na = 0;
            if (inA) route_type(L, t, na++, model->path_mask[t], A, amap);
            if (inB) {
              route_type(L, t, na, model->path_mask[t], B, bmap);
              if (na == 1 && !memcmp(L.alt_node[t][0], L.alt_node[t][1], CF_MAX_COMP))
                memset(L.alt_node[t][1], 255, CF_MAX_COMP);
              else
                na++;
            }
            L.n_alt[t] = (uint8_t)na;
          }
          if ((st = emit(L)) != CF_OK) return st;
        }
      }
  }
  *n_out = n;
  return CF_OK;
}

extern "C" cf_status cf_enum_count(const cf_model_desc *model, const cf_enum_opts *opts, const cf_logical *logical_dev,
                                   int32_t n_logical, uint64_t *offsets_dev, uint64_t *total_host, void *stream) {
  using namespace cf;
  cf_status st = check_opts(model, opts);
  if (st != CF_OK) return st;
  if (n_logical < 0 || !offsets_dev || !total_host || (n_logical > 0 && !logical_dev))
    return set_error(CF_EINVAL, "NULL array or n_logical < 0");
  hipStream_t s = as_stream(stream);
  *total_host = 0;
  if (n_logical == 0) {
    const uint64_t zero = 0;
    st = hip_check(hipMemcpyAsync(offsets_dev, &zero, sizeof zero, hipMemcpyHostToDevice, s), "cf_enum_count copy");
    if (st != CF_OK) return st;
    return hip_check(hipStreamSynchronize(s), "cf_enum_count sync");
  }
  uint64_t *totals = nullptr;
  if ((st = run_tables(opts, logical_dev, n_logical, nullptr, &totals, s)) != CF_OK) return st;
  hipLaunchKernelGGL(k_enum_offsets, dim3(1), dim3(1024), 0, s, totals, n_logical, offsets_dev);
  if ((st = hip_check(hipGetLastError(), "cf_enum offsets launch")) != CF_OK) return st;
  st = hip_check(hipMemcpyAsync(total_host, offsets_dev + n_logical, sizeof(uint64_t), hipMemcpyDeviceToHost, s),
                 "cf_enum_count copy");
  if (st != CF_OK) return st;
  if ((st = hip_check(hipStreamSynchronize(s), "cf_enum_count sync")) != CF_OK) return st;
  if (*total_host == ~0ull) return set_error(CF_ECAPACITY, "the number of physical plans does not fit 64 bits");
  return CF_OK;
}

extern "C" cf_status cf_enum_plans(const cf_model_desc *model, const cf_enum_opts *opts, const cf_logical *logical_dev,
                                   int32_t n_logical, const uint64_t *offsets_dev, uint64_t total, uint64_t first,
                                   int32_t count, const cf_plan_table *out, void *stream) {
  using namespace cf;
  cf_status st = check_opts(model, opts);
  if (st != CF_OK) return st;
  if (!out || count < 0 || out->P < count) return set_error(CF_EINVAL, "output table smaller than count");
  if (count == 0) return CF_OK;
  if (n_logical < 1 || !logical_dev || !offsets_dev) return set_error(CF_EINVAL, "no logical plans");
  if (first > total || (uint64_t)count > total - first) return set_error(CF_EINVAL, "first + count > total");
  if (!out->n_nodes_dev || !out->node_comp_dev || !out->node_rep_dev || !out->node_batch_dev ||
      !out->node_gpus_dev || !out->n_alt_dev || !out->alt_w_dev || !out->alt_node_dev)
    return set_error(CF_EINVAL, "NULL plan-table array");
  const int ng = (out->node_rep2_dev != nullptr) + (out->node_batch2_dev != nullptr) +
                 (out->node_gpus2_dev != nullptr) + (out->node_w_dev != nullptr);
  if (ng != 0 && ng != 4) return set_error(CF_EINVAL, "second-configuration arrays: all four or none");
  if (opts->het && ng == 0) return set_error(CF_EINVAL, "het plans need the second-configuration arrays");
  hipStream_t s = as_stream(stream);
  uint64_t *tab = nullptr, *totals = nullptr;
  if ((st = run_tables(opts, logical_dev, n_logical, &tab, &totals, s)) != CF_OK) return st;
  EnumView V;
  V.N = opts->n_gpus;
  V.logical = logical_dev;
  V.n_logical = n_logical;
  V.ng = most_gpu_options(opts);
  V.tab = tab;
  V.totals = totals;
  PlanOut o;
  o.P = out->P;
  o.n_nodes = const_cast<uint8_t *>(out->n_nodes_dev);
  o.node_comp = const_cast<uint8_t *>(out->node_comp_dev);
  o.node_rep = const_cast<uint8_t *>(out->node_rep_dev);
  o.node_batch = const_cast<uint16_t *>(out->node_batch_dev);
  o.node_gpus = const_cast<uint8_t *>(out->node_gpus_dev);
  o.n_alt = const_cast<uint8_t *>(out->n_alt_dev);
  o.alt_w = const_cast<uint8_t *>(out->alt_w_dev);
  o.alt_node = const_cast<uint8_t *>(out->alt_node_dev);
  o.node_rep2 = const_cast<uint8_t *>(out->node_rep2_dev);
  o.node_batch2 = const_cast<uint16_t *>(out->node_batch2_dev);
  o.node_gpus2 = const_cast<uint8_t *>(out->node_gpus2_dev);
  o.node_w = const_cast<uint8_t *>(out->node_w_dev);
  const unsigned threads = (unsigned)((count + kPlansPerThread - 1) / kPlansPerThread);
  if (opts->het)
    hipLaunchKernelGGL(k_enum_unrank<true>, dim3((threads + 255) / 256), dim3(256), 0, s, *opts, V, offsets_dev, first,
                       count, o);
  else
    hipLaunchKernelGGL(k_enum_unrank<false>, dim3((threads + 255) / 256), dim3(256), 0, s, *opts, V, offsets_dev,
                       first, count, o);
  return hip_check(hipGetLastError(), "cf_enum_plans launch");
}

extern "C" cf_status cf_enum_screen(const cf_model_desc *model, const cf_enum_opts *opts, const cf_logical *logical_dev,
                                    int32_t n_logical, const uint64_t *offsets_dev, uint64_t total, uint64_t first,
                                    int32_t count, const uint64_t *moments_dev, int32_t n_gpus, double *rd_dev,
                                    int32_t *bottleneck_dev, uint8_t *flags_dev, void *stream) {
  using namespace cf;
  cf_status st = check_opts(model, opts);
  if (st != CF_OK) return st;
  if (opts->het) return set_error(CF_EUNSUPPORTED, "cf_enum_screen takes one configuration per node");
  KModel m;
  if ((st = lower_model(model, &m)) != CF_OK) return st;
  if (count < 0) return set_error(CF_EINVAL, "count < 0");
  if (count == 0) return CF_OK;
  if (n_logical < 1 || !logical_dev || !offsets_dev || !moments_dev || !rd_dev || !bottleneck_dev || !flags_dev)
    return set_error(CF_EINVAL, "NULL argument");
  if (first > total || (uint64_t)count > total - first) return set_error(CF_EINVAL, "first + count > total");
  hipStream_t s = as_stream(stream);
  uint64_t *tab = nullptr, *totals = nullptr;
  if ((st = run_tables(opts, logical_dev, n_logical, &tab, &totals, s)) != CF_OK) return st;
  EnumView V;
  V.N = opts->n_gpus;
  V.logical = logical_dev;
  V.n_logical = n_logical;
  V.ng = most_gpu_options(opts);
  V.tab = tab;
  V.totals = totals;
  int n_opt = 0;
  for (int c = 0; c < model->n_comp; c++) n_opt += opts->n_batch[c] * opts->n_gpu_opt[c];
  const size_t work = sizeof(double) * (size_t)m.nt * m.nc * n_opt;
  const dim3 grid((unsigned)((count + kScrBlock - 1) / kScrBlock));
  if (work <= (size_t)kWorkBytes)
    hipLaunchKernelGGL(k_enum_screen<true>, grid, dim3(kScrBlock), work, s, *opts, V, offsets_dev, first, count, m,
                       moments_dev, n_gpus, n_opt, rd_dev, bottleneck_dev, flags_dev);
  else
    hipLaunchKernelGGL(k_enum_screen<false>, grid, dim3(kScrBlock), 0, s, *opts, V, offsets_dev, first, count, m,
                       moments_dev, n_gpus, n_opt, rd_dev, bottleneck_dev, flags_dev);
  return hip_check(hipGetLastError(), "cf_enum_screen launch");
}
