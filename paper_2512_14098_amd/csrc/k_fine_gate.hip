// k_fine_gate.hip -- the request-level simulator (Sec. 4.3, Alg. 2 phase 3)
// for models with one gated stage (thinker -> talker), with its control state
// in registers: the rules, results and status words of k_fine<true>.
//
// As in k_fine_reg.hip the aim is fewer instructions and no waits for LDS on
// the way from one instant to the next: k_fine<true> holds up to 320 stage
// instances of a 64-GPU plan in LDS, so each field costs an LDS latency and
// comes back in a vector register, and its 9.6 KB per wavefront hold it at 16
// wavefronts per CU.  Here lane x holds executor x: its iteration, its runs,
// its wake time and the running sets of its thinker and its talker, one
// register per field, so that only the queues are left in LDS.  That fits the
// models whose only LLM components are one gate source and the one component
// gated by it; others take k_fine<true>.
// The gated part is k_fine<true>'s: a talker's running slot carries its gate
// word and join step, a thinker's ring (one per executor, in memory) holds the
// ends of its last and of its running steps, executors with blocked talker
// requests keep a wake time and register with the thinkers they wait for, and
// a thinker and a talker that only wait for each other run jointly.  A lane of
// a gated scan reads another executor's step counter by a lane permutation,
// so the scans run with every lane active.  The ends of a run's steps that
// stay in one binade are integers of its spacing, one multiplication per lane
// (run_walk and one addition per step otherwise).
// Measured against k_fine<true>: 32,000 triples of 2,000 requests, plans on 64
// GPUs, 687 -> 495 ms; 6,432 triples of 4,000 requests, plans on 16 GPUs,
// which end on their longest triple, 570 -> 504 ms.  With the queues in
// registers too the indexed accesses cost more than LDS; scalar reads of
// k_fine<true>'s LDS fields alone slow it by 6 %.
#include "cf_fine_reg.h"
#include "cf_run.h"

namespace cf {
namespace fine {
namespace {

constexpr int kRing = 256;                 // thinker step-time ring
constexpr int kKeep = 64;                  // completed steps kept in the ring
constexpr uint32_t kThRun = kRing - kKeep; // longest thinker decode run
constexpr uint64_t kMant = (1ull << 52) - 1;  // a double's significand field
constexpr uint32_t MISC_TH_DONE = 16u;     // thinker finished
// A talker's running slot: request; tokens so far (bits 0..15), its own token
// count (16..30) and MARK (in the current decode step); gate word: gated for
// its type (bit 31), thinker's executor (16..21), thinker's token count
// (0..15); join step in the thinker's stage.  A thinker's: request, step at
// which it finishes.
constexpr uint32_t MARK = 0x80000000u, RG_GATED = 0x80000000u;
__device__ __forceinline__ uint32_t rk_own(uint32_t k) { return (k >> 16) & 0x7FFFu; }
constexpr uint32_t IN_TH = 1u << 13;       // info word: c is the type's gate source
constexpr uint32_t IN_TA = 1u << 14;       // c is gated for the type
// iteration kinds of e_st (bits 0..2); members<> also takes K_FINISH (thinker
// slots that finish at a step), K_STEP (a talker step over the marked slots)
// and K_JOINT (the talker slots of a joint run)
enum { K_BATCH = 0, K_PREFILL = 1, K_DECODE = 2, K_JOINT = 3, K_FINISH = 4, K_STEP = 5 };
// component word (lane c): attributes summed into X (bits 0..6), output-length
// attribute (8..10), kind (12..13), output of some type (14), children over
// all types (16..23), batch cap - 1 (24..31)
// executor word e_geo: component set (bits 8..15), GPUs index (16..18), batch (20..28)
// executor state e_st: kind (bits 0..2), component run last (4..7, 15: none), members (12..20)

struct GateLds {
  uint32_t info[CF_MAX_COMP][CF_MAX_TYPES];
  uint32_t npar[CF_MAX_TYPES];  // parents on the path, 4 bits per component
  double slo[CF_MAX_TYPES][4];
  double tps[CF_MAX_COMP][8];
  double lat[CF_MAX_COMP][5];   // k0, k1, k2, d0, d1
  unsigned long long watch[CF_MAX_EXEC];  // per thinker executor: executors to notify when its steps are (re)scheduled
  uint32_t met[CF_MAX_TYPES], cnt[CF_MAX_TYPES];
  uint8_t route[CF_MAX_TYPES][2][CF_MAX_COMP];
  uint8_t nalt[CF_MAX_TYPES], aw[CF_MAX_TYPES][2], path[CF_MAX_TYPES], nout[CF_MAX_TYPES], src[CF_MAX_TYPES];
  uint8_t vbase[CF_MAX_NODES], vrep[CF_MAX_NODES], vminc[CF_MAX_NODES], vcomp[CF_MAX_NODES];
  uint8_t vrep1[CF_MAX_NODES], vw[CF_MAX_NODES];
  uint16_t vbatch[CF_MAX_NODES], vbatch2[CF_MAX_NODES];
};

// queues by component and executor: length, head and tail (qend); after
// GateLds, for the model's components only
struct GateQ {
  uint32_t qn[CF_MAX_EXEC], qh[CF_MAX_EXEC], qt[CF_MAX_EXEC];
};
extern __shared__ GateQ gate_q[];

struct Gate {
  const FineArgs *A;
  GateLds *sh;
  CF_GLOBAL char *slab;
  uint32_t o_run, o_mem, o_dl, o_pool, o_next, o_free, o_ring;
  GPtr<const uint64_t> ticks;
  uint32_t seed;
  double lam, now, dl_head_t, comm;
  uint64_t events, dirty, busy, runm, done_now, rewake, ta_mask;  // ta_mask: executors hosting a talker
  uint32_t status, dl_head, dl_tail, dl_mask, nc;
  int pool_top, pool_fresh, pool_hot, n_chunks, n_done, nx, lat_slot, cth, cta;
  bool tp_any;
  uint32_t *hrow;
  // executor x in lane x: end of its iteration, wake time; a run's first step
  // end, step time and (joint run) talker step time
  double e_end, e_wake, e_t1, e_dur, e_dur2;
  uint32_t e_itgt, e_st, e_geo;
  uint32_t th_rn, th_roff, th_iter, th_minfin, th_sched;  // thinker
  uint32_t ta_rn, ta_roff;                          // talker
  uint32_t c_word;                                  // component c in lane c
  double a_t;                                       // request i of the block of arrivals in lane i
  uint64_t a_ex;
  uint32_t a_type;
};

__device__ __forceinline__ CArgs &args(const Gate &S) { return args(S.A); }
// a T at byte offset off of the wavefront's memory
template <typename T>
__device__ __forceinline__ CF_GLOBAL T &at(const Gate &S, uint32_t off) {
  return *(CF_GLOBAL T *)(S.slab + off);
}
// a T at byte off of request r's block
template <typename T>
__device__ __forceinline__ CF_GLOBAL T &req_at(const Gate &S, uint32_t r, uint32_t off) {
  return at<T>(S, r * (uint32_t)sizeof(RReq) + off);
}

// ------------------------------------------------------------------ queues
// The free chunks are a stack whose top stays in a register: a queue that
// empties and fills again takes its chunk back without a memory access.
__device__ __forceinline__ int chunk_alloc(Gate &S) {
  int c = S.pool_hot;
  if (c >= 0) {
    S.pool_hot = -1;
    return c;
  }
  if (S.pool_top > 0) return ri(at<int>(S, S.o_free + 4u * (uint32_t)--S.pool_top));
  if (S.pool_fresh < S.n_chunks) return S.pool_fresh++;
  S.status |= CF_ST_OVERFLOW;
  return -1;
}
__device__ __forceinline__ void chunk_free(Gate &S, int c) {
  if (c < 0 || c >= S.n_chunks || S.pool_top >= S.n_chunks) {
    S.status |= CF_ST_OVERFLOW;
    return;
  }
  if (S.pool_hot >= 0) at<int>(S, S.o_free + 4u * (uint32_t)S.pool_top++) = S.pool_hot;  // every lane, the same word
  S.pool_hot = c;
}

// appends, in lane order, the requests r of the lanes `on` (mask bal) to component c's queue at executor x
__device__ __forceinline__ void q_push(Gate &S, int x, int c, uint64_t bal, bool on, uint32_t r) {
  const int cnt = __popcll(bal);
  const uint32_t qn = ru(gate_q[c].qn[x]);
  uint32_t qt = ru(gate_q[c].qt[x]);
  if (qn == 0) {
    const int ch = chunk_alloc(S);
    if (ch < 0) return;
    qt = qend(ch, 0);
    gate_q[c].qh[x] = qt;
  }
  const int tc = qend_chunk(qt), tp = qend_pos(qt);
  // the entries fill the tail chunk, then at most one fresh chunk (cnt <= 64)
  const int room = kChunk - tp;
  int c1 = tc;
  if (cnt > room) {
    c1 = chunk_alloc(S);
    if (c1 < 0) return;
    at<int>(S, S.o_next + 4u * (uint32_t)tc) = c1;
  }
  if (on) {
    const int k = (int)lanes_below(bal);
    at<uint32_t>(S, S.o_pool + 4u * (uint32_t)((k < room ? tc * kChunk + tp : c1 * kChunk - room) + k)) = r;
  }
  gate_q[c].qt[x] = cnt <= room ? qt + (uint32_t)cnt : qend(c1, cnt - room);
  gate_q[c].qn[x] = qn + (uint32_t)cnt;
}

// appends one request (wave-uniform r)
__device__ __forceinline__ void q_push1(Gate &S, int x, int c, uint32_t r) {
  const uint32_t qn = ru(gate_q[c].qn[x]);
  uint32_t qt = ru(gate_q[c].qt[x]);
  if (qn == 0) {
    const int ch = chunk_alloc(S);
    if (ch < 0) return;
    qt = qend(ch, 0);
    gate_q[c].qh[x] = qt;
  } else if (qend_pos(qt) == kChunk) {
    const int ch = chunk_alloc(S);
    if (ch < 0) return;
    at<int>(S, S.o_next + 4u * (uint32_t)qend_chunk(qt)) = ch;
    qt = qend(ch, 0);
  }
  at<uint32_t>(S, S.o_pool + 4u * (uint32_t)(qend_chunk(qt) * kChunk + qend_pos(qt))) = r;
  gate_q[c].qt[x] = qt + 1u;
  gate_q[c].qn[x] = qn + 1u;
}

// Takes the first k entries of component c's queue at executor x to offset dst, 64 at a time (a
// block spans at most two chunks), and sums their attributes sel.
__device__ __forceinline__ uint32_t q_take(Gate &S, int x, int c, int k, uint32_t dst, uint32_t sel) {
  const uint32_t qh = ru(gate_q[c].qh[x]);
  int hc = qend_chunk(qh), hp = qend_pos(qh);
  const int qn = (int)ru(gate_q[c].qn[x]);
  uint32_t xs = 0;
  for (int b = 0; b < k; b += 64) {
    const int cnt = k - b < 64 ? k - b : 64;
    const int room = kChunk - hp;  // entries left in the head chunk
    // the block reaches into the next chunk, or entries remain after this chunk's last
    const bool more = cnt > room || (cnt == room && b + cnt < qn);
    int nx = hc;
    if (more) {
      nx = ri(at<int>(S, S.o_next + 4u * (uint32_t)hc));
      if (nx < 0 || nx >= S.n_chunks) {
        S.status |= CF_ST_OVERFLOW;
        return 0;
      }
    }
    if (lane_id() < cnt) {
      const uint32_t r = at<uint32_t>(
          S, S.o_pool + 4u * (uint32_t)((lane_id() < room ? hc * kChunk + hp : nx * kChunk - room) + lane_id()));
      const u32x4 aw = req_at<u32x4>(S, r, kOffAttr);
      xs += x_in(aw, sel);
      at<uint32_t>(S, dst + 4u * (uint32_t)(b + lane_id())) = r;
    }
    hp += cnt;
    if (more) {
      chunk_free(S, hc);
      hc = nx;
      hp -= kChunk;
    }
  }
  gate_q[c].qn[x] = (uint32_t)(qn - k);
  if (qn == k) chunk_free(S, hc);
  else gate_q[c].qh[x] = qend(hc, hp);
  return dpp_sum_u32(xs);
}

// ------------------------------------------------------------------ arrivals
// Prepares the 64 requests from base on: arrival times, routes and blocks.
__device__ __forceinline__ void load_arrivals(Gate &S, uint32_t base) {
  CArgs &A = args(S);
  CModel &m = A.m;
  const GateLds &sh = *S.sh;
  const uint32_t r = base + (uint32_t)lane_id();
  S.a_t = __builtin_inf();
  S.a_ex = ~0ull;
  S.a_type = CF_MAX_TYPES;
  if (r < (uint32_t)A.n) {
    const size_t o = (size_t)S.seed * (size_t)A.n + r;
    const uint64_t tk = S.ticks[r];
    const uint32_t t = gload(A.type, o), ak = gload(A.akey, o);
    const uint64_t k0 = gload(A.rkey0, o), k1 = gload(A.rkey1, o);
    u32x4 w;
    w.x = (uint32_t)gload(A.prompt, o) | ((uint32_t)gload(A.out, o) << 16);
    w.y = gload(A.patches, o);
    w.z = gload(A.aud_in, o);
    w.w = gload(A.aud_out, o);
    S.a_t = ((double)tk * 0x1p-32) / S.lam;
    if (t < (uint32_t)m.nt) {
      int alt = 0;
      if (sh.nalt[t] == 2) {
        const uint64_t w0 = sh.aw[t][0], w1 = sh.aw[t][1];
        alt = (((uint64_t)ak * (w0 + w1)) >> 32) < w0 ? 0 : 1;
      }
      uint64_t ex = ~0ull;
      const uint32_t path = sh.path[t];
      for (int c = 0; c < m.nc; c++) {
        if (!((path >> c) & 1u)) continue;
        const int v = sh.route[t][alt][c];
        const int mc = sh.vminc[v];
        const uint32_t key = (uint32_t)((mc < 4 ? k0 : k1) >> (16 * (mc & 3))) & 0xFFFFu;
        const uint64_t x = (uint64_t)(sh.vbase[v] + node_exec(key, sh.vrep1[v], (uint32_t)(sh.vrep[v] - sh.vrep1[v]),
                                                              sh.vw[v]));
        ex ^= (0xFFull ^ x) << (8 * c);
      }
      S.a_ex = ex;
      S.a_type = t | ((uint32_t)sh.src[t] << 8);
      req_at<u32x4>(S, r, 0) = u32x4{(uint32_t)ex, (uint32_t)(ex >> 32), 0u, (uint32_t)sh.nout[t] | (t << 8)};
      req_at<u32x4>(S, r, kOffAttr) = w;
    }
  }
}

__device__ __forceinline__ void arrive(Gate &S, uint32_t r) {
  const int i = (int)(r & 63u);
  S.events++;
  const uint32_t ts = rl(S.a_type, i);  // type and source components
  if (ts == CF_MAX_TYPES) {
    S.status |= CF_ST_INVALID;
    return;
  }
  const uint64_t ex = rl64(S.a_ex, i);
  for (uint32_t src = ts >> 8; src; src &= src - 1) {
    const int c = __builtin_ctz(src);
    const int x = (int)((ex >> (8 * c)) & 63u);
    S.events++;
    q_push1(S, x, c, r);
    S.dirty |= 1ull << x;
  }
}

// ------------------------------------------------------------------ deliveries
// step 2: the delayed deliveries due now, in production order, up to 64 at a time
__device__ __forceinline__ void deliver_due(Gate &S) {
  while (S.dl_head != S.dl_tail && S.dl_head_t == S.now) {
    const uint32_t n = S.dl_tail - S.dl_head;
    u32x4 e = {0, 0x7FF00000u, 0, 0};
    if ((uint32_t)lane_id() < n) e = at<u32x4>(S, S.o_dl + ((S.dl_head + (uint32_t)lane_id()) & S.dl_mask) * 16u);
    const double et = words_double(e.x, e.y);
    const uint64_t late = ballot(et != S.now);
    const int k = late ? ff1(late) : 64;  // entries due
    if (k == 0) {  // the head's time is kept in dl_head_t: cannot happen
      S.status |= CF_ST_OVERFLOW;
      return;
    }
    const bool on = lane_id() < k;
    const uint32_t r = on ? e.z >> 4 : 0u;
    const uint32_t c2 = e.z & 7u;
    const u32x4 q = req_at<u32x4>(S, r, 0);
    const uint32_t x = (uint32_t)((((uint64_t)q.y << 32) | q.x) >> (8 * c2)) & 63u;
    const uint32_t np = (S.sh->npar[(q.w >> 8) & 7u] >> (4 * c2)) & 15u;
    uint64_t ready = ballot(on && np <= 1u);
    // components with several parents: count this delivery and the earlier
    // ones of the same request in this block
    for (uint64_t m = ballot(on && np > 1u); m; m &= m - 1) {
      const int i = ff1(m);
      const uint32_t rr = rl(r, i), ci = rl(c2, i);
      uint32_t join = rl(q.z, i) + (1u << (4 * ci));
      for (uint64_t d = ballot(on && r == rr && np > 1u) & ((1ull << i) - 1ull); d; d &= d - 1)
        join += 1u << (4 * rl(c2, ff1(d)));
      req_at<uint32_t>(S, rr, 8) = join;
      if (((join >> (4 * ci)) & 15u) == rl(np, i)) ready |= 1ull << i;
    }
    const uint32_t stage = x * 8u + c2;
    const bool rdy = (ready >> lane_id()) & 1ull;
    for (uint64_t left = ready; left;) {
      const int f = ff1(left);
      const uint32_t st = rl(stage, f);
      const bool mine = rdy && stage == st;
      const uint64_t bal = ballot(mine);
      S.events += (uint64_t)__popcll(bal);
      q_push(S, (int)(st >> 3), (int)(st & 7u), bal, mine, r);
      S.dirty |= 1ull << (st >> 3);
      left &= ~bal;
    }
    S.dl_head += (uint32_t)k;
    if (S.dl_head == S.dl_tail) S.dl_head_t = __builtin_inf();
    else if (k < 64) S.dl_head_t = words_double(rl(e.x, k), rl(e.y, k));
    else S.dl_head_t = rdb(at<double>(S, S.o_dl + (S.dl_head & S.dl_mask) * 16u));
  }
}

// ------------------------------------------------------------------ gating
// value of lane `lane` (per lane; every lane active)
__device__ __forceinline__ uint32_t lane_of(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(lane << 2), (int)v);
}
__device__ __forceinline__ CF_GLOBAL double &ring_at(const Gate &S, uint32_t x, uint32_t step) {
  return at<double>(S, S.o_ring + (x * (uint32_t)kRing + (step & (kRing - 1))) * 8u);
}

// What the talker slot w (lanes with `in`) at executor y waits for: the time
// the thinker token is visible at y (-inf: not gated for its type; +inf: its
// step is not scheduled).  pend: that time may still change; remote: the
// thinker runs on another executor.  Every lane active.
struct Vis {
  double t;
  uint32_t xth;
  bool pend, remote;
};
__device__ __forceinline__ Vis slot_vis(const Gate &S, const u32x4 &w, bool in, int y, bool &undecided) {
  const bool gated = in && (w.z & RG_GATED) != 0;
  const uint32_t xth = gated ? (w.z >> 16) & 63u : (uint32_t)y;
  const uint32_t nth = w.z & 0xFFFFu, tok1 = (w.y & 0xFFFFu) + 1u;
  const uint32_t k = tok1 < nth ? tok1 : nth;
  const uint32_t it = lane_of(S.th_iter, xth), sched = lane_of(S.th_sched, xth);
  const uint32_t q = w.w + k - 1u, r = gated ? w.x : 0u;
  const double delta = xth == (uint32_t)y ? 0.0 : S.comm;
  const bool first = k <= 1u;
  Vis v;
  v.xth = xth;
  v.remote = xth != (uint32_t)y;
  const bool wait = q > sched;                 // the step is not scheduled yet
  v.pend = gated && !first && (wait || q > it);  // or only predicted
  double e = ring_at(S, xth, q);               // every kept or scheduled step's entry
  if (gated && first) e = req_at<double>(S, r, kOffTim);
  if (gated && !first && !v.pend && it - q >= (uint32_t)kKeep) {
    if (k == nth && (req_at<uint32_t>(S, r, 12) & MISC_TH_DONE)) {
      e = req_at<double>(S, r, kOffLast);
    } else {
      e = ring_at(S, xth, it - (kKeep - 1));  // oldest kept step: token k is no later
      if (!(e + delta <= S.now)) {
        undecided = true;
        e = __builtin_inf();
      }
    }
  }
  v.t = !gated ? -__builtin_inf() : (!first && wait) ? __builtin_inf() : e + delta;
  return v;
}
__device__ __forceinline__ uint32_t ta_slots(const Gate &S, int x) { return S.o_run + rl(S.ta_roff, x) * 16u; }

// marks the eligible slots of executor x's talker; returns their number
__device__ __forceinline__ uint32_t gate_scan(Gate &S, int x) {
  const int rn = (int)rl(S.ta_rn, x);
  const uint32_t slots = ta_slots(S, x);
  bool undecided = false;
  uint32_t cnt = 0;
  for (int b = 0; b < rn; b += 64) {
    const int j = b + lane_id();
    const bool in = j < rn;
    const u32x4 w = at<u32x4>(S, slots + (uint32_t)j * 16u);
    const Vis v = slot_vis(S, w, in, x, undecided);
    const bool el = in && v.t <= S.now;
    // only a changed mark is written
    if (in && el != ((w.y & MARK) != 0)) at<uint32_t>(S, slots + (uint32_t)j * 16u + 4u) = w.y ^ MARK;
    cnt += (uint32_t)__popcll(ballot(el));
  }
  if (ballot(undecided)) S.status |= CF_ST_OVERFLOW;
  return cnt;
}

// the decode steps of the thinker on executor x were (re)scheduled: the
// registered executors recompute their wake time
__device__ __forceinline__ void notify(Gate &S, int x) {
  const uint64_t w = ru64(S.sh->watch[x]);
  if (w) {
    S.rewake |= w;
    S.sh->watch[x] = 0;
  }
}

// Recomputes the wake time of executor y, which hosts a talker: the earliest
// visibility time, after now, of the token that a blocked request waits for
// from a thinker on another executor.  Only kept while y is idle or in a run;
// y registers with the thinkers whose steps are not final.  Returns whether
// some such request is eligible already.
__device__ __forceinline__ bool gate_wake(Gate &S, int y) {
  const uint64_t ybit = 1ull << y;
  double w = __builtin_inf();
  bool now_el = false;
  if (!(S.busy & ybit) || (S.runm & ybit)) {
    const int rn = (int)rl(S.ta_rn, y);
    const uint32_t slots = ta_slots(S, y);
    bool undecided = false;
    for (int b = 0; b < rn; b += 64) {
      const int j = b + lane_id();
      const bool in = j < rn;
      const u32x4 sw = at<u32x4>(S, slots + (uint32_t)j * 16u);
      const Vis v = slot_vis(S, sw, in, y, undecided);
      if (in && v.remote) {
        if (v.pend) atomicOr(&S.sh->watch[v.xth], ybit);
        if (v.t <= S.now) now_el = true;
        else w = v.t < w ? v.t : w;
      }
    }
    if (ballot(undecided)) S.status |= CF_ST_OVERFLOW;
    if (rn > 0) w = wave_min_time(w);
    now_el = ballot(now_el) != 0;
  }
  wld(S.e_wake, y, w);
  return now_el;
}

// ------------------------------------------------------------------ completions
// The n members of an iteration of component c on executor x that ended now,
// in member order, 64 per pass.  KIND:
//   K_BATCH    ENC/GEN members finish their component;
//   K_PREFILL  members get their first token (a thinker's is delivered to the
//              talker) and finish or join the running set;
//   K_FINISH   the thinker slots that finish at step `it` finish;
//   K_STEP     every marked talker slot gains a token;
//   K_JOINT    every talker slot gains `it` tokens, the last of them now if `ends`.
// Finished slots' places are closed (a kept slot only moves down, and a page
// is read before it is written).  Lanes without a member read request 0's
// block and are masked afterwards.
template <int KIND>
__device__ __forceinline__ void members(Gate &S, int x, int c, int n, uint32_t it, bool ends) {
  GateLds &sh = *S.sh;
  constexpr bool SLOTS = KIND == K_FINISH || KIND == K_STEP || KIND == K_JOINT;
  const uint32_t cw = rl(S.c_word, c);
  const uint32_t chany = (cw >> 16) & 0xFFu;
  const bool outc = (cw >> 14) & 1u, genc = KIND == K_BATCH && ((cw >> 12) & 3u) == CF_GEN;
  const bool talker = KIND == K_STEP || KIND == K_JOINT || (KIND == K_PREFILL && c == S.cta);
  const uint32_t slots = KIND == K_BATCH ? 0u : S.o_run + rl(talker ? S.ta_roff : S.th_roff, x) * 16u;
  const double now = S.now;
  uint32_t w = 0, mn = kNone;
  for (int b = 0; b < n; b += 64) {
    const int j = b + lane_id();
    bool valid = j < n;
    uint32_t r;
    if constexpr (SLOTS) {
      const uint32_t so = slots + (uint32_t)j * 16u;
      bool fin, keep, moved;
      if constexpr (KIND == K_FINISH) {
        const uint64_t sv = at<uint64_t>(S, so);
        const uint32_t key = (uint32_t)(sv >> 32);
        fin = valid && key == it;
        keep = valid && key != it;
        const uint64_t kb = ballot(keep);
        const uint32_t d = w + lanes_below(kb);
        if (keep && d != (uint32_t)j) at<uint64_t>(S, slots + d * 16u) = sv;
        mn = keep && key < mn ? key : mn;
        w += (uint32_t)__popcll(kb);
        r = (uint32_t)sv;
      } else {
        u32x4 sv = at<u32x4>(S, so);
        const uint32_t k0 = sv.y;
        const bool step = valid && (KIND == K_JOINT || (k0 & MARK));
        const uint32_t tok = (k0 & 0xFFFFu) + (KIND == K_JOINT ? it : 1u);
        sv.y = step ? (k0 & (0x7FFFu << 16)) | tok : k0;
        fin = step && (KIND == K_STEP || ends) && tok == rk_own(k0);
        keep = valid && !fin;
        const uint64_t kb = ballot(keep);
        const uint32_t d = w + lanes_below(kb);
        moved = d != (uint32_t)j;
        if (keep && moved) at<u32x4>(S, slots + d * 16u) = sv;
        if (keep && !moved && sv.y != k0) at<uint32_t>(S, so + 4u) = sv.y;
        w += (uint32_t)__popcll(kb);
        r = sv.x;
      }
      valid = fin;
      if (!ballot(valid)) continue;
    } else {
      r = at<uint32_t>(S, S.o_mem + (uint32_t)(x * CF_MAX_BATCH + j) * 4u);
    }
    r = valid ? r : 0u;
    const u32x4 q = req_at<u32x4>(S, r, 0);
    u32x4 aw, tw;
    uint64_t tkv;
    if constexpr (KIND == K_PREFILL) aw = req_at<u32x4>(S, r, kOffAttr);
    if (KIND != K_PREFILL ? outc : c == S.cta) tw = req_at<u32x4>(S, r, kOffTim);
    if (outc) tkv = S.ticks[r];
    const uint32_t t = (q.w >> 8) & 7u;
    const uint32_t info = sh.info[c][t];
    bool fin = valid, stream = false;
    if constexpr (KIND == K_PREFILL) {
      uint32_t no = attr_in(aw, (cw >> 8) & 7u);
      no = (info & IN_PFO) || no < 1u ? 1u : no;
      fin = valid && no == 1u;
      const bool append = valid && no != 1u;
      const uint64_t ab = ballot(append);
      if (!talker) {
        const uint32_t iter = rl(S.th_iter, x), key = iter + no - 1u;
        if (valid && (info & IN_TTFT)) {
          const uint64_t nb = (uint64_t)__double_as_longlong(now);
          tw = u32x4{(uint32_t)nb, (uint32_t)(nb >> 32), no, iter};
          req_at<u32x4>(S, r, kOffTim) = tw;
        }
        stream = valid && (info & IN_TH);
        if (ab) {
          const uint32_t rn = rl(S.th_rn, x);
          if (append) at<uint64_t>(S, slots + (rn + lanes_below(ab)) * 16u) = ((uint64_t)key << 32) | r;
          wl(S.th_rn, x, rn + (uint32_t)__popcll(ab));
          const uint32_t km = dpp_min_u32(append ? key : kNone), om = rl(S.th_minfin, x);
          wl(S.th_minfin, x, km < om ? km : om);
        }
      } else {
        if (valid && (info & IN_TTFT)) {  // a type whose first LLM is the talker component
          const uint64_t nb = (uint64_t)__double_as_longlong(now);
          tw = u32x4{(uint32_t)nb, (uint32_t)(nb >> 32), no, 0u};
          req_at<u32x4>(S, r, kOffTim) = tw;
        }
        if (ab) {
          const uint32_t rn = rl(S.ta_rn, x);
          uint32_t gw = 0, gq = 0;
          if (info & IN_TA) {
            const uint32_t thi = sh.info[S.cth][t];
            uint32_t nth = attr_in(aw, (rl(S.c_word, S.cth) >> 8) & 7u);
            nth = (thi & IN_PFO) || nth < 1u ? 1u : nth;
            gw = RG_GATED | ((((S.cth < 4 ? q.x : q.y) >> (8 * (S.cth & 3))) & 63u) << 16) | nth;
            gq = tw.w;
          }
          if (append) at<u32x4>(S, slots + (rn + lanes_below(ab)) * 16u) = u32x4{r, 1u | (no << 16), gw, gq};
          wl(S.ta_rn, x, rn + (uint32_t)__popcll(ab));
        }
      }
      if (!ballot(fin || stream)) continue;
    }
    uint32_t join = q.z, misc = q.w;
    bool put = false;
    // deliveries: a thinker's streaming one to the talker first, then the
    // children; remote ones join the delay line, local ones enqueue when the
    // last input is there
    {
      const uint32_t ch = fin ? info & 0xFFu : 0u;
      const uint32_t sbit = 1u << S.cta;
      const uint32_t all = KIND == K_PREFILL && !talker ? chany | sbit : chany;
      uint32_t rc = 0, ready = 0;
      bool srem = false;
      for (uint32_t cc = all; cc; cc &= cc - 1) {
        const int c2 = __builtin_ctz(cc);
        const uint32_t own = 1u << c2;
        const bool str = KIND == K_PREFILL && stream && c2 == S.cta;
        const uint32_t bit = str ? own : ch & own;
        const uint32_t xe = ((c2 < 4 ? q.x : q.y) >> (8 * (c2 & 3))) & 0xFFu;
        const bool local = xe == (uint32_t)x;
        if (str) srem = !local;
        else rc |= local ? 0u : bit;
        if (local && bit) {
          const uint32_t np = (sh.npar[t] >> (4 * c2)) & 15u;
          if (np > 1u) {
            join += 1u << (4 * c2);
            put = true;
            if (((join >> (4 * c2)) & 15u) == np) ready |= bit;
          } else {
            ready |= bit;
          }
        }
      }
      const uint32_t ndl = (uint32_t)__popc(rc) + (srem ? 1u : 0u);
      const uint64_t db = ballot(ndl != 0);
      if (db) {
        uint32_t off, total;
        if (ballot(ndl > 1) == 0) {
          off = lanes_below(db);
          total = (uint32_t)__popcll(db);
        } else {
          off = wave_excl_scan(ndl, total);
        }
        if (S.dl_tail - S.dl_head + total > S.dl_mask + 1u) {
          S.status |= CF_ST_OVERFLOW;
          return;
        }
        const double due = now + S.comm;
        const uint64_t du = (uint64_t)__double_as_longlong(due);
        uint32_t pos = S.dl_tail + off;
        if (KIND == K_PREFILL && srem) {
          at<u32x4>(S, S.o_dl + (pos & S.dl_mask) * 16u) =
              u32x4{(uint32_t)du, (uint32_t)(du >> 32), (r << 4) | (DL_DELIVER << 3) | (uint32_t)S.cta, 0u};
          pos++;
        }
        for (uint32_t cc = chany; cc; cc &= cc - 1) {
          const int c2 = __builtin_ctz(cc);
          if ((rc >> c2) & 1u) {
            at<u32x4>(S, S.o_dl + (pos & S.dl_mask) * 16u) =
                u32x4{(uint32_t)du, (uint32_t)(du >> 32), (r << 4) | (DL_DELIVER << 3) | (uint32_t)c2, 0u};
            pos++;
          }
        }
        if (S.dl_head == S.dl_tail) S.dl_head_t = rdb(due);
        S.dl_tail += total;
      }
      if (ballot(ready != 0)) {
        for (uint32_t cc = all; cc; cc &= cc - 1) {
          const int c2 = __builtin_ctz(cc);
          const bool on = (ready >> c2) & 1u;
          const uint64_t bal = ballot(on);
          if (!bal) continue;
          S.events += (uint64_t)__popcll(bal);
          q_push(S, x, c2, bal, on, r);
        }
      }
    }
    if (fin && (info & IN_TH)) {
      misc |= MISC_TH_DONE;
      put = true;
    }
    // outputs, completed requests: latencies, SLO check, per-type counts
    bool done = false;
    if (outc) {
      const bool out = fin && (info & IN_OUT);
      if (out) {
        misc -= 1u;
        put = true;
        done = (misc & 15u) == 0;
      }
      if (genc && out && !done) req_at<double>(S, r, kOffLast + 8) = now;
      const uint64_t dbal = ballot(done);
      if (dbal) {
        if (done) {
          const bool here = (info & IN_TTFT) != 0, llm = (info & IN_LLM) != 0, gen = (info & IN_GENO) != 0;
          if (KIND == K_PREFILL && !here) tw = req_at<u32x4>(S, r, kOffTim);
          // last token and media time: this stage's, or from the block
          double tl = now, tm = now;
          if ((llm && !here) || (gen && !genc)) {
            const u32x4 lw = req_at<u32x4>(S, r, kOffLast);
            tl = here ? now : words_double(lw.x, lw.y);
            tm = genc ? now : words_double(lw.z, lw.w);
          }
          const double a = ((double)tkv * 0x1p-32) / S.lam;
          double ttft = 0.0, tpot = 0.0, media = 0.0;
          if (llm) {
            const double tf = words_double(tw.x, tw.y);
            ttft = tf - a;
            if (tw.z > 1u) tpot = (tl - tf) / (double)(tw.z - 1u);
          }
          const double e2e = now - a;
          if (gen) media = tm - a;
          const double *slo = sh.slo[t];
          const bool ok = ttft <= slo[0] && tpot <= slo[1] && e2e <= slo[2] && media <= slo[3];
          atomicAdd(&sh.cnt[t], 1u);
          if (ok) atomicAdd(&sh.met[t], 1u);
          if (S.hrow) {
            CArgs &A = args(S);
            atomicAdd(S.hrow + t * (uint32_t)(A.nb + 1) + target_bin(A.tg, A.nb, (int)t, ttft, tpot, e2e, media), 1u);
          }
          if (S.lat_slot >= 0) {
            CArgs &A = args(S);
            double *Lp = A.lat + ((size_t)S.lat_slot * A.n + r) * 4;
            Lp[0] = ttft;
            Lp[1] = tpot;
            Lp[2] = e2e;
            Lp[3] = media;
          }
        }
        S.events += (uint64_t)__popcll(dbal);
        S.n_done += __popcll(dbal);
      }
    }
    // the last token's time (a finished thinker's gates its talker, so it is
    // kept even when the request is complete)
    if (SLOTS && valid && (info & IN_TTFT)) req_at<double>(S, r, kOffLast) = now;
    if (put) req_at<uint64_t>(S, r, 8) = ((uint64_t)misc << 32) | join;
  }
  if constexpr (KIND == K_FINISH) {
    wl(S.th_rn, x, w);
    wl(S.th_minfin, x, dpp_min_u32(mn));
  } else if constexpr (SLOTS) {
    wl(S.ta_rn, x, w);
  }
}

// the iteration of executor x ended now
__device__ __forceinline__ void complete(Gate &S, int x) {
  const uint32_t st = rl(S.e_st, x);
  const uint64_t xbit = 1ull << x;
  S.busy &= ~xbit;
  S.runm &= ~xbit;
  S.dirty |= xbit;
  S.done_now |= xbit;
  wld(S.e_end, x, __builtin_inf());
  const uint32_t kind = st & 7u;
  const int c = (int)((st >> 4) & 15u), n = (int)((st >> 12) & 511u);
  if (kind == K_BATCH) {
    S.events += (uint64_t)n;
    members<K_BATCH>(S, x, c, n, 0u, false);
  } else if (kind == K_PREFILL) {
    S.events += (uint64_t)n;
    members<K_PREFILL>(S, x, c, n, 0u, false);
  } else if (kind == K_DECODE && c == S.cta) {
    S.events += (uint64_t)n;
    members<K_STEP>(S, x, c, (int)rl(S.ta_rn, x), 0u, false);
  } else {
    // thinker steps; a joint run of m steps (thinker first) also gave every
    // talker slot m / 2 tokens, and its last step's stage resumes the round robin
    const uint32_t it0 = rl(S.th_iter, x), rn = rl(S.th_rn, x);
    uint32_t it = rl(S.e_itgt, x);
    bool fin = true;
    if (kind == K_JOINT) {
      const uint32_t m = it, nta = m >> 1, rng = rl(S.ta_rn, x);
      it = it0 + ((m + 1u) >> 1);
      S.events += (uint64_t)rng * (uint64_t)nta;
      fin = m & 1u;
      wl(S.e_st, x, (uint32_t)(fin ? S.cth : S.cta) << 4);
      wl(S.th_iter, x, it);
      S.events += (uint64_t)rn * (uint64_t)(it - it0);
      if (nta) members<K_JOINT>(S, x, S.cta, (int)rng, nta, !fin);
    } else {
      wl(S.th_iter, x, it);  // the ring already holds the ends of these steps
      S.events += (uint64_t)rn * (uint64_t)(it - it0);
    }
    if (fin && it == rl(S.th_minfin, x)) members<K_FINISH>(S, x, S.cth, (int)rn, it, false);
  }
}

// ------------------------------------------------------------------ starts
// What executor x's talker waits for, seen from its thinker, when none of its
// requests is eligible: qmin, the first thinker step whose token one of them
// waits for; joint: all of them (there are some) wait for the thinker's next
// step; kta: talker steps before the first of them finishes.
struct GateView {
  uint32_t qmin, kta;
  bool joint;
};
__device__ __forceinline__ GateView gate_view(const Gate &S, int x) {
  const uint32_t next = rl(S.th_iter, x) + 1u;
  const int rn = (int)rl(S.ta_rn, x);
  const uint32_t slots = ta_slots(S, x);
  uint32_t qmin = kNone, kta = kNone;
  bool other = false;  // a running request that does not wait for the thinker's next step
  for (int b = 0; b < rn; b += 64) {
    const int j = b + lane_id();
    if (j < rn) {
      const u32x4 w = at<u32x4>(S, slots + (uint32_t)j * 16u);
      const uint32_t tok = w.y & 0xFFFFu;
      bool waits_next = false;
      if ((w.z & RG_GATED) && (int)((w.z >> 16) & 63u) == x) {
        const uint32_t nth = w.z & 0xFFFFu, k = tok + 1u < nth ? tok + 1u : nth, q = w.w + k - 1u;
        // a thinker on this executor has finished once its last step is completed
        if (k > 1u && !(k == nth && q < next)) {
          qmin = q < qmin ? q : qmin;
          waits_next = q == next;
        }
      }
      other |= !waits_next;
      const uint32_t left = rk_own(w.y) - tok;
      kta = left < kta ? left : kta;
    }
  }
  GateView v;
  v.qmin = dpp_min_u32(qmin);
  v.kta = dpp_min_u32(kta);
  v.joint = rn > 0 && ballot(other) == 0;
  return v;
}

// Joint run: with every talker request waiting for the thinker's next token
// and nothing else to run, the executor alternates a thinker and a talker step
// over all its running requests up to the first step with a finishing request.
// False (nothing started) for steps of zero duration.
__device__ __forceinline__ bool start_joint(Gate &S, int x, double tps_th, double tps_ta, uint32_t kta) {
  const GateLds &sh = *S.sh;
  double d1 = sh.lat[S.cth][3] + sh.lat[S.cth][4] * (double)rl(S.th_rn, x);
  double d2 = sh.lat[S.cta][3] + sh.lat[S.cta][4] * (double)rl(S.ta_rn, x);
  if (S.tp_any) {
    d1 = tps_th * d1;
    d2 = tps_ta * d2;
  }
  if (!(d1 > 0.0) || !(d2 > 0.0)) return false;
  const uint32_t it0 = rl(S.th_iter, x);
  const uint32_t kth = rl(S.th_minfin, x) - it0;  // thinker steps up to its first finisher
  uint32_t n = 2u * (kth < kThRun ? kth : kThRun) - 1u;
  if (2u * kta < n) n = 2u * kta;
  const uint32_t nth = (n + 1u) >> 1;
  double t = S.now;
  const uint64_t b0 = ru64((uint64_t)__double_as_longlong(t));
  const uint64_t D1 = step_units(rdb(d1), (int)(b0 >> 52)), D2 = step_units(rdb(d2), (int)(b0 >> 52));
  if (D1 && D2 && (b0 & kMant) + (uint64_t)nth * (D1 + D2) <= kMant) {
    // the run stays in its start's binade and neither duration ties there:
    // every thinker step adds D1 units of the spacing, every talker step D2
    for (uint32_t s = (uint32_t)lane_id() + 1u; s <= nth; s += 64u)
      ring_at(S, (uint32_t)x, it0 + s) =
          __longlong_as_double((long long)(b0 + (uint64_t)s * D1 + (uint64_t)(s - 1u) * D2));
    t = __longlong_as_double((long long)(b0 + (uint64_t)nth * D1 + (uint64_t)(n - nth) * D2));
  } else {
    // lane j keeps the end of the j-th thinker step of the current block of
    // 64, written to the ring when the block is complete
    double tl = 0.0;
    for (uint32_t s = 1; s <= nth; s++) {
      t = t + d1;
      const uint32_t j = (s - 1u) & 63u;
      tl = (uint32_t)lane_id() == j ? t : tl;
      if (j == 63u || s == nth) {
        if ((uint32_t)lane_id() <= j) ring_at(S, (uint32_t)x, it0 + s - j + (uint32_t)lane_id()) = tl;
      }
      if (2u * s <= n) t = t + d2;
    }
  }
  wl(S.th_sched, x, it0 + nth);
  wld(S.e_t1, x, S.now + d1);
  wld(S.e_dur, x, d1);
  wld(S.e_dur2, x, d2);
  wl(S.e_itgt, x, n);  // steps of the run, thinker first
  wld(S.e_end, x, t);
  S.busy |= 1ull << x;
  S.runm |= 1ull << x;
  wl(S.e_st, x, K_JOINT | ((uint32_t)S.cth << 4));
  return true;
}

// Starts the next iteration of idle executor x.  work: components with a batch
// or prefill or a thinker decode step to run (bits 0..7), of them prefills
// (8..15), and the talker if only its gate can tell (16..23).
__device__ __forceinline__ void try_start(Gate &S, int x, uint32_t work) {
  const uint32_t sure = work & 0xFFu, maybe = (work >> 16) & 0xFFu;
  if (!(sure | maybe)) return;
  const uint64_t xbit = 1ull << x;
  const uint32_t geo = rl(S.e_geo, x), c0 = (rl(S.e_st, x) >> 4) & 15u;
  // round robin: the first component with work after the one run last
  const uint32_t late = c0 == 15u ? 0xFFu : ~((2u << c0) - 1u);
  auto first_of = [&](uint32_t m) { return __builtin_ctz((m & late) ? m & late : m); };
  int c = first_of(sure | maybe);
  bool ta_ok = false, scanned = false;
  uint32_t nel = 0;
  if (maybe && (c == S.cta)) {
    nel = gate_scan(S, x);
    scanned = true;
    ta_ok = nel > 0;
    if (!ta_ok) {
      if (!sure) return;
      c = first_of(sure);
    }
  }
  const double *lat = S.sh->lat[c];
  const uint32_t tpi = (geo >> 16) & 7u;
  const double tps = S.tp_any ? S.sh->tps[c][tpi] : 1.0;
  const uint32_t cbit = 1u << c;
  double end;
  uint32_t kind, n;
  if (ta_ok) {
    // a talker step over the eligible requests
    kind = K_DECODE;
    n = nel;
    double dur = lat[3] + lat[4] * (double)n;
    if (S.tp_any) dur = tps * dur;
    end = S.now + dur;
  } else if (c != S.cth || (work & (cbit << 8))) {
    const uint32_t cw = rl(S.c_word, c), batch = (geo >> 20) & 511u, cap = (cw >> 24) + 1u;
    const uint32_t beff = batch < cap ? batch : cap, qn = ru(gate_q[c].qn[x]);
    kind = (work & (cbit << 8)) ? K_PREFILL : K_BATCH;
    const uint32_t room = kind == K_BATCH ? beff : beff - rl(c == S.cth ? S.th_rn : S.ta_rn, x);
    n = qn < room ? qn : room;
    const double k0 = lat[0], k1 = lat[1], k2 = lat[2];
    const uint32_t xs = q_take(S, x, c, (int)n, S.o_mem + (uint32_t)(x * CF_MAX_BATCH * 4), cw & 0x7Fu);
    double dur = (k0 + k1 * (double)xs) + k2 * (double)n;
    if (S.tp_any) dur = tps * dur;
    // an encoder started on an executor that was idle before this instant
    if (((cw >> 12) & 3u) == CF_ENC && !(S.done_now & xbit)) dur = dur + args(S).m.cpu_pre;
    end = S.now + dur;
  } else {
    // a thinker decode step; alone, a run up to its first finishing step, its
    // ring's reach, or the first step a local talker request waits for
    kind = K_DECODE;
    const uint32_t it1 = rl(S.th_iter, x) + 1u;
    n = rl(S.th_rn, x);
    bool lazy = (sure & (sure - 1u)) == 0;
    if (lazy && maybe && !scanned) lazy = gate_scan(S, x) == 0;
    uint32_t bound = it1;
    if (lazy) {
      bound = it1 - 1u + kThRun;
      if ((S.ta_mask >> x) & 1ull) {
        const GateView gv = gate_view(S, x);
        if (gv.joint && start_joint(S, x, tps, S.tp_any ? S.sh->tps[S.cta][tpi] : 1.0, gv.kta)) {
          notify(S, x);
          return;
        }
        bound = gv.qmin < bound ? gv.qmin : bound;
      }
    }
    double dur = lat[3] + lat[4] * (double)n;
    if (S.tp_any) dur = tps * dur;
    uint32_t itgt = it1;
    const double t1 = S.now + dur;
    end = t1;
    uint32_t fin = rl(S.th_minfin, x);
    fin = fin < bound ? fin : bound;
    if (lazy && dur > 0.0 && fin > it1) {
      uint32_t taken = 0;
      end = run_walk(t1, dur, fin - it1, __builtin_inf(), &taken);
      itgt += taken;
      if (taken) {
        S.runm |= xbit;
        wld(S.e_t1, x, t1);
        wld(S.e_dur, x, dur);
      }
    }
    // the predicted end of every step, one step per lane
    const uint32_t last = itgt - it1;
    const uint64_t b1 = ru64((uint64_t)__double_as_longlong(t1));
    const uint64_t D = last ? step_units(rdb(dur), (int)(b1 >> 52)) : 0;
    if (last == 0 || (D && (b1 & kMant) + (uint64_t)last * D <= kMant)) {
      // inside one binade step i ends i D units after the first
      for (uint32_t i = (uint32_t)lane_id(); i <= last; i += 64u)
        ring_at(S, (uint32_t)x, it1 + i) = __longlong_as_double((long long)(b1 + (uint64_t)i * D));
    } else {
      for (uint32_t i = (uint32_t)lane_id(); i <= last; i += 64u) {
        uint32_t taken = 0;
        ring_at(S, (uint32_t)x, it1 + i) = run_walk(t1, dur, i, __builtin_inf(), &taken);
      }
    }
    wl(S.th_sched, x, itgt);
    wl(S.e_itgt, x, itgt);
    notify(S, x);
  }
  wld(S.e_end, x, end);
  S.busy |= xbit;
  wl(S.e_st, x, kind | ((uint32_t)c << 4) | (n << 12));
}

// An input reached executor x, in a run: it stops at the first step that ends
// at or after now (the steps before it are unchanged).
__device__ __forceinline__ void cut_run(Gate &S, int x) {
  if (!(lane_val(S.e_end, x) > S.now)) return;
  const uint32_t it0 = rl(S.th_iter, x), itgt = rl(S.e_itgt, x);
  const double t1 = lane_val(S.e_t1, x), d1 = lane_val(S.e_dur, x);
  if ((rl(S.e_st, x) & 7u) == K_JOINT) {
    const double d2 = lane_val(S.e_dur2, x);
    double t = t1;
    uint32_t j = 1;
    while (t < S.now && j < itgt) {
      j++;
      t = t + ((j & 1u) ? d1 : d2);
    }
    wld(S.e_end, x, t);
    wl(S.e_itgt, x, j);
    if (j < itgt) {
      wl(S.th_sched, x, it0 + ((j + 1u) >> 1));
      notify(S, x);
    }
    return;
  }
  uint32_t taken = 0;
  const double t = run_walk(t1, d1, itgt - (it0 + 1u), S.now, &taken);
  const uint32_t j = it0 + 1u + taken;
  wld(S.e_end, x, t);
  wl(S.e_itgt, x, j);
  if (taken == 0) S.runm &= ~(1ull << x);
  if (j < itgt) {
    wl(S.th_sched, x, j);
    notify(S, x);
  }
}

// ------------------------------------------------------------------ setup
// Plan p into LDS and registers; false: the plan is malformed.
__device__ __forceinline__ bool setup_plan(Gate &S, int p) {
  CArgs &A = args(S);
  CModel &m = A.m;
  GateLds &sh = *S.sh;
  const size_t P = (size_t)A.P;
  const int lane = lane_id();
  const int nv = ri(A.n_nodes[p]);
  if (nv < 1 || nv > CF_MAX_NODES) return false;
  bool bad = false;
  if (lane < CF_MAX_NODES) {
    const uint32_t rep = lane < nv ? A.node_rep[lane * P + p] : 0;
    const uint32_t rep2 = (lane < nv && A.node_rep2) ? A.node_rep2[lane * P + p] : 0;
    const uint32_t b2 = rep2 ? A.node_batch2[lane * P + p] : 0, w = rep2 ? A.node_w[lane * P + p] : 0;
    const uint32_t cm = lane < nv ? A.node_comp[lane * P + p] : 0, bn = lane < nv ? A.node_batch[lane * P + p] : 0;
    sh.vcomp[lane] = (uint8_t)cm;
    sh.vminc[lane] = (uint8_t)(cm ? __ffs(cm) - 1 : 0);
    sh.vrep[lane] = (uint8_t)(rep + rep2 < 255 ? rep + rep2 : 255);
    sh.vrep1[lane] = (uint8_t)rep;
    sh.vbatch[lane] = (uint16_t)bn;
    sh.vbatch2[lane] = (uint16_t)b2;
    sh.vw[lane] = (uint8_t)w;
    if (rep2 && (rep < 1 || w < 1 || w > 9 || b2 < 1 || b2 > CF_MAX_BATCH || A.node_gpus2[lane * P + p] < 1)) bad = true;
    if (lane < nv && (cm == 0 || (cm >> m.nc) || rep + rep2 < 1 || bn < 1 || bn > CF_MAX_BATCH)) bad = true;
  }
  if (ballot(bad)) return false;
  for (int j = lane; j < CF_MAX_TYPES * 2 * CF_MAX_COMP; j += 64) (&sh.route[0][0][0])[j] = A.alt_node[j * P + p];
  if (lane < CF_MAX_TYPES) sh.nalt[lane] = lane < m.nt ? A.n_alt[lane * P + p] : 0;
  if (lane < 2 * CF_MAX_TYPES) (&sh.aw[0][0])[lane] = A.alt_w[lane * P + p];
  __syncthreads();
  int base = 0, run_need = 0;
  for (int v = 0; v < nv; v++) {
    const uint32_t cm = ru(sh.vcomp[v]);
    const int rep = ri(sh.vrep[v]), rep1 = ri(sh.vrep1[v]), b1 = ri(sh.vbatch[v]), b2 = ri(sh.vbatch2[v]);
    sh.vbase[v] = (uint8_t)(base < 255 ? base : 255);
    base += rep;
    for (uint32_t cc = cm; cc; cc &= cc - 1) {
      const int c = __builtin_ctz(cc);
      if (m.kind[c] == CF_LLM)
        run_need += rep1 * (b1 < m.cap[c] ? b1 : m.cap[c]) + (rep - rep1) * (b2 < m.cap[c] ? b2 : m.cap[c]);
    }
  }
  if (base > CF_MAX_EXEC) return false;
  // routes: lane t * 16 + a * 8 + c, in two rounds of 64
  bool ok = true;
  for (int j = lane; j < m.nt * 16; j += 64) {
    const int t = j >> 4, a = (j >> 3) & 1, c = j & 7, na = sh.nalt[t];
    if (na < 1 || na > 2) ok = false;
    if (a < na) {
      if (na > 1 && sh.aw[t][a] < 1) ok = false;
      if ((m.path[t] >> c) & 1u) {
        const int v = sh.route[t][a][c];
        if (v >= nv || !((sh.vcomp[v] >> c) & 1u)) ok = false;
      }
    }
  }
  if (ballot(!ok)) return false;
  if (run_need > A.L.run_cap) {
    S.status |= CF_ST_OVERFLOW;
    return true;
  }
  S.nx = base;
  // executors, one lane each; a running set takes the batch its component
  // may have there
  uint32_t th_b = 0, ta_b = 0;
  bool ta = false;
  if (lane < base) {
    int v = 0;
    while (v + 1 < nv && sh.vbase[v + 1] <= lane) v++;
    const uint32_t cm = sh.vcomp[v];
    const bool second = lane - sh.vbase[v] >= sh.vrep1[v];
    const uint32_t batch = second ? sh.vbatch2[v] : sh.vbatch[v];
    uint32_t tp = 0;
    if (m.tp_any) {
      const uint32_t g = second ? A.node_gpus2[v * P + p] : A.node_gpus[v * P + p];
      tp = g < 1 ? 0 : (g > 8 ? 7 : g - 1);
    }
    S.e_geo = (cm << 8) | (tp << 16) | (batch << 20);
    const uint32_t hc = (uint32_t)m.cap[S.cth], ac = (uint32_t)m.cap[S.cta];
    if ((cm >> S.cth) & 1u) th_b = batch < hc ? batch : hc;
    ta = (cm >> S.cta) & 1u;
    if (ta) ta_b = batch < ac ? batch : ac;
  }
  sh.watch[lane] = 0;
  S.ta_mask = ballot(ta);
  uint32_t th_n, ta_n;
  S.th_roff = wave_excl_scan(th_b, th_n);
  S.ta_roff = th_n + wave_excl_scan(ta_b, ta_n);
  __syncthreads();
  return true;
}

__device__ __forceinline__ void setup_model(Gate &S) {
  CModel &m = args(S).m;
  GateLds &sh = *S.sh;
  const int lane = lane_id();
  {
    const int c = lane >> 3, t = lane & 7;
    uint32_t w = 0;
    if (c < m.nc && t < m.nt) {
      w = m.child[t][c];
      if (m.ttft_c[t] == c) w |= IN_TTFT;
      if ((m.outm[t] >> c) & 1u) w |= IN_OUT;
      if ((m.pfo[t] >> c) & 1u) w |= IN_PFO;
      if (m.gen_out[t]) w |= IN_GENO;
      if (m.th_c[t] == c) w |= IN_TH;
      if (m.ta_c[t] == c) w |= IN_TA;
      if (m.ttft_c[t] >= 0) w |= IN_LLM;
    }
    sh.info[c][t] = w;
    sh.tps[c][t] = m.tps[c][t];
  }
  if (lane < CF_MAX_TYPES) {
    uint32_t np = 0;
    for (int c = 0; c < CF_MAX_COMP; c++) np |= (uint32_t)(m.npar[lane][c] & 15u) << (4 * c);
    sh.npar[lane] = np;
    sh.path[lane] = (uint8_t)m.path[lane];
    sh.nout[lane] = (uint8_t)__popc(m.outm[lane]);
    sh.src[lane] = (uint8_t)m.srcm[lane];
  }
  S.cth = __builtin_ctz(m.gate_src_mask);
  S.cta = __builtin_ctz(m.gated_mask);
  S.nc = (uint32_t)m.nc;
  if (lane < CF_MAX_TYPES * 4) (&sh.slo[0][0])[lane] = (&m.slo[0][0])[lane];
  S.c_word = 0;
  if (lane < m.nc) {
    sh.lat[lane][0] = m.k0[lane];
    sh.lat[lane][1] = m.k1[lane];
    sh.lat[lane][2] = m.k2[lane];
    sh.lat[lane][3] = m.d0[lane];
    sh.lat[lane][4] = m.d1[lane];
    uint32_t chany = 0, out = 0;
    for (int t = 0; t < m.nt; t++) {
      chany |= m.child[t][lane];
      out |= (m.outm[t] >> lane) & 1u;
    }
    S.c_word = (m.xsel[lane] & 0x7Fu) | (((uint32_t)m.nout_attr[lane] & 7u) << 8) | ((uint32_t)m.kind[lane] << 12) |
               (out << 14) | (chany << 16) | ((uint32_t)(m.cap[lane] - 1) << 24);
  }
}

// 96 VGPRs, 5 wavefronts per SIMD (16 VGPRs and 198 SGPRs spilled): 495 ms on the
// launch of 32,000 triples above; 4 (128 VGPRs) 563 ms, 6 (63 VGPRs spilled) 586 ms.
__global__ void __launch_bounds__(64, 5) k_fine_gate(const FineArgs *__restrict__ Ap) {
  __shared__ GateLds sh;
  const int lane = lane_id();
  Gate S;
  S.A = Ap;
  S.sh = &sh;
  setup_model(S);
  {
    CArgs &A = args(S);
    const __attribute__((address_space(4))) Layout &L = A.L;
    char *slab = A.slab + (size_t)blockIdx.x * L.bytes;
    S.slab = (CF_GLOBAL char *)(slab + L.req);
    S.o_run = (uint32_t)(L.run - L.req);
    S.o_mem = (uint32_t)(L.mem - L.req);
    S.o_dl = (uint32_t)(L.dl - L.req);
    S.o_pool = (uint32_t)(L.pool - L.req);
    S.o_next = (uint32_t)(L.pool_next - L.req);
    S.o_free = (uint32_t)(L.pool_free - L.req);
    S.o_ring = (uint32_t)(L.hist - L.req);
    S.dl_mask = L.dl_mask;
    S.n_chunks = L.n_chunks;
    S.comm = A.m.comm;
    S.tp_any = A.m.tp_any != 0;
  }
  __syncthreads();
  for (;;) {
    CArgs &A = args(S);
    const unsigned int per_seed = (unsigned int)A.n_plans * (unsigned int)A.K;
    unsigned int tk = 0;
    if (lane == 0) tk = atomicAdd(A.ticket, 1u);
    tk = ru(tk);
    if (tk >= A.total) break;
    // the same order of triples as k_fine
    const int s = (int)(tk / per_seed);
    const unsigned int rem = tk % per_seed;
    int k, i;
    if (A.order) {
      const uint32_t e = ru(A.order[rem]);
      i = (int)(e / (unsigned)A.K);
      k = (int)(e % (unsigned)A.K);
    } else {
      k = (int)(rem / (unsigned)A.n_plans);
      i = (int)(rem % (unsigned)A.n_plans);
    }
    const int p = ri(A.plan_ids[i]);
    const size_t oidx = ((size_t)i * A.K + k) * A.S + s;
    S.seed = (uint32_t)s;
    S.ticks = GPtr<const uint64_t>{(const CF_GLOBAL uint64_t *)(A.ticks + (size_t)s * A.n)};
    S.lam = rdb(A.rates[(size_t)i * A.K + k]);
    S.events = 0;
    S.status = 0;
    S.dirty = S.busy = S.runm = S.done_now = 0;
    S.dl_head = S.dl_tail = 0;
    S.dl_head_t = __builtin_inf();
    S.pool_top = 0;
    S.pool_fresh = 0;
    S.pool_hot = -1;
    S.n_done = 0;
    S.now = 0.0;
    S.lat_slot = -1;
    // nothing of the lanes' state lives across triples
    S.e_end = per_lane(__builtin_inf());
    S.e_wake = per_lane(__builtin_inf());
    S.e_t1 = per_lane(0.0);
    S.e_dur = per_lane(0.0);
    S.e_dur2 = per_lane(0.0);
    S.e_itgt = per_lane(0u);
    S.e_st = per_lane(15u << 4);  // no component run yet
    for (uint32_t c = 0; c < S.nc; c++) gate_q[c].qn[lane] = 0;
    S.th_rn = per_lane(0u);
    S.th_iter = per_lane(0u);
    S.th_minfin = per_lane(kNone);
    S.th_sched = per_lane(0u);
    S.ta_rn = per_lane(0u);
    S.rewake = 0;
    S.a_t = __builtin_inf();
    S.a_ex = ~0ull;
    S.e_geo = S.a_type = S.th_roff = S.ta_roff = 0;
    S.hrow = A.hist ? A.hist + oidx * (size_t)A.m.nt * (size_t)(A.nb + 1) : nullptr;
    for (int j = 0; j < A.n_lat; j++)
      if (A.lat_triples[j] == (int32_t)oidx) S.lat_slot = j;
    if (lane < CF_MAX_TYPES) {
      sh.met[lane] = 0;
      sh.cnt[lane] = 0;
    }
    __syncthreads();
    const bool ok = (p >= 0 && p < A.P) && S.lam > 0.0 && S.lam < __builtin_inf() && setup_plan(S, p);
    if (!ok) S.status |= CF_ST_INVALID;
    if (ok && !(S.status & CF_ST_OVERFLOW) && A.n > 0) {
      const uint32_t n = (uint32_t)A.n;
      uint32_t next_arr = 0;
      load_arrivals(S, 0);
      double t_arr = lane_val(S.a_t, 0);
      // instants that may still be taken before the budget (2 events + 16 n +
      // 4096, at most lim_instants) is looked at again: it only grows
      uint64_t granted = 0;
      uint32_t left = 0;
      for (;;) {
        // --- next pending time: the earliest iteration end or wake time (none:
        // +inf; non-negative doubles order like their bits), the delay line's
        // head and the next arrival
        const uint64_t eb = (uint64_t)__double_as_longlong(S.e_end), wb = (uint64_t)__double_as_longlong(S.e_wake);
        const uint64_t mb = wb < eb ? wb : eb;
        const uint32_t hi = (uint32_t)(mb >> 32);
        const uint32_t hmin = dpp_min_u32(hi);
        const uint64_t at_min = ballot(hi == hmin);
        double te = __builtin_inf();
        if (hmin != 0x7FF00000u) {
          const uint32_t lmin = (at_min & (at_min - 1)) == 0 ? rl((uint32_t)mb, ff1(at_min))
                                                             : dpp_min_u32(hi == hmin ? (uint32_t)mb : ~0u);
          te = words_double(lmin, hmin);
        }
        double t = te < S.dl_head_t ? te : S.dl_head_t;
        t = rdb(t_arr < t ? t_arr : t);
        if (t == __builtin_inf()) break;
        if (left == 0) {
          const uint64_t lim = args(S).lim_instants;
          uint64_t bound = 2 * S.events + 16ull * n + 4096ull;
          bound = bound < lim ? bound : lim;
          if (granted >= bound) {
            S.status |= CF_ST_DEADLOCK;
            break;
          }
          left = bound - granted < (1u << 30) ? (uint32_t)(bound - granted) : 1u << 30;
          granted += left;
        }
        left--;
        if (t != S.now) S.done_now = 0;  // an instant may follow at the same time
        S.now = t;
        // --- step 1: iterations ending at t, ascending executor
        if (te == t) {
          uint64_t ends = ballot(S.e_end == t);
          // wake times due: the executor examines its components in step 3
          const bool wk = S.e_wake == t;
          if (wk) S.e_wake = __builtin_inf();
          S.dirty |= ballot(wk);
          while (ends) {
            const int x = ff1(ends);
            ends &= ends - 1;
            complete(S, x);
          }
          __syncthreads();
        }
        // --- step 2: delayed deliveries due at t, then arrivals at t
        deliver_due(S);
        while (t_arr == t) {
          arrive(S, next_arr);
          next_arr++;
          if ((next_arr & 63u) == 0 && next_arr < n) load_arrivals(S, next_arr);
          t_arr = next_arr < n ? lane_val(S.a_t, (int)(next_arr & 63u)) : __builtin_inf();
        }
        // --- step 3: executors whose state changed: cut runs, start iterations;
        // then the wake times of those examined or notified.  An executor found
        // with a request eligible now is examined once more (at most once).
        __syncthreads();
        uint64_t cand = S.dirty, extra = 0;
        S.dirty = 0;
        uint32_t work = 0;
        if (cand & ~S.busy) {
          // lane x: what executor x could run (try_start)
          const uint32_t cth = (uint32_t)S.cth, cta = (uint32_t)S.cta, batch = (S.e_geo >> 20) & 511u;
          uint32_t q = 0;
#pragma unroll
          for (int c = 0; c < CF_MAX_COMP; c++)
            if ((uint32_t)c < S.nc) q |= (gate_q[c].qn[lane] > 0 ? 1u : 0u) << c;
          const uint32_t hcap = (rl(S.c_word, S.cth) >> 24) + 1u, acap = (rl(S.c_word, S.cta) >> 24) + 1u;
          const uint32_t llm = (1u << cth) | (1u << cta);
          const bool hp = ((q >> cth) & 1u) && S.th_rn < (batch < hcap ? batch : hcap);
          const bool ap = ((q >> cta) & 1u) && S.ta_rn < (batch < acap ? batch : acap);
          const uint32_t pre = (hp ? 1u << cth : 0u) | (ap ? 1u << cta : 0u);
          work = (q & ~llm) | pre | (S.th_rn > 0 ? 1u << cth : 0u) | (pre << 8) |
                 (S.ta_rn > 0 && !ap ? 1u << (16u + cta) : 0u);
        }
        for (;;) {
          S.rewake |= cand & S.ta_mask;
          while (cand) {
            const int x = ff1(cand);
            cand &= cand - 1;
            if (!((S.busy >> x) & 1ull)) try_start(S, x, rl(work, x));
            else if ((S.runm >> x) & 1ull) cut_run(S, x);
          }
          while (S.rewake) {
            const int y = ff1(S.rewake);
            S.rewake &= S.rewake - 1;
            if (gate_wake(S, y) && !((extra >> y) & 1ull)) cand |= 1ull << y;
          }
          if (!cand || (S.status & CF_ST_OVERFLOW)) break;
          extra |= cand;
        }
        if (S.status & (CF_ST_OVERFLOW | CF_ST_INVALID)) break;
      }
      if (S.n_done < A.n && !(S.status & (CF_ST_OVERFLOW | CF_ST_INVALID))) S.status |= CF_ST_DEADLOCK;
    }
    __syncthreads();
    CArgs &Ao = args(S);
    if (lane < Ao.m.nt) {
      Ao.met[oidx * Ao.m.nt + lane] = sh.met[lane];
      Ao.cnt[oidx * Ao.m.nt + lane] = sh.cnt[lane];
    }
    if (lane == 0) {
      Ao.events[oidx] = S.events;
      Ao.status[oidx] = S.status;
    }
    __syncthreads();
  }
}

}  // namespace

bool fine_gate_takes(const KModel &m) {
  uint32_t llm = 0;
  for (int c = 0; c < m.nc; c++)
    if (m.kind[c] == CF_LLM) llm |= 1u << c;
  return __builtin_popcount(m.gate_src_mask) == 1 && __builtin_popcount(m.gated_mask) == 1 &&
         llm == (m.gate_src_mask | m.gated_mask) && m.gate_src_mask != m.gated_mask;
}
void launch_fine_gate(const FineArgs *args, int n_comp, unsigned waves, hipStream_t s) {
  hipLaunchKernelGGL(k_fine_gate, dim3(waves), dim3(64), sizeof(GateQ) * (size_t)n_comp, s, args);
}

}  // namespace fine
}  // namespace cf
