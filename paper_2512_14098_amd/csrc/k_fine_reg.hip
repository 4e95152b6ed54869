// k_fine_reg.hip -- the request-level simulator (Sec. 4.3, Alg. 2 phase 3)
// with its whole control state in registers: one wavefront per (plan, rate,
// seed) triple, as in k_fine.hip and with the same rules, results and status
// words, for models without a gated stage and launches whose plans have at
// most 64 stage instances.
//
// What bounds this simulator is instruction issue (counters of a whole launch:
// profiles/k_fine_c1.md).  Control state in LDS is what costs the
// instructions: every uniform field that is read comes back in a vector
// register, so that its arithmetic and its branches go through the vector
// pipe and the execution mask.  Here
//   - lane x holds executor x (end of its iteration, decode run, state word),
//     lane s stage instance s (queue ends and length, running set, step
//     counter) and lane c component c's latency model; a field is read by
//     v_readlane into a scalar register and written by v_writelane, so
//     control flow is scalar and no instant waits for LDS or for the scalar
//     cache;
//   - the stages with work are three ballots per instant for all executors,
//     and one executor's round robin is bit arithmetic on them;
//   - arrivals are prepared 64 at a time, lane i for request i of the block
//     (arrival time, routes, the request's memory block), so that an arrival
//     itself only enqueues;
//   - deliveries due together are taken up to 64 at a time;
//   - a completed iteration's members are one loop over pages of 64 lanes,
//     in which a finishing decode step also compacts its running slots;
//   - a stage's queue entries go to registers and their lengths are summed in
//     one pass (one load for the entries, one for the lengths).
// 64 stage instances is one per lane; the plans of up to 32 GPUs of a
// two-component model always fit.
// Measured against k_fine<false> on the same launches: 15,360 triples of 10^4
// requests of the two-component model on 8 GPUs 535 -> 347 ms; 6,400 triples
// of 5,000 text-to-image requests 90 -> 56 ms; 24 triples of 1,000 requests
// (one wavefront per CU, latency only) 14.3 -> 7.9 ms.
#include "cf_fine_reg.h"
#include "cf_run.h"

namespace cf {
namespace fine {
namespace {

// component word (lane c): attributes summed into X (bits 0..6), output-length
// attribute (8..10), kind (12..13), children over all types (16..23), output
// of some type (24)
// stage word: component (bits 0..3), kind (4..5), batch (8..16), executor (20..25)
// executor word e_geo: first stage (bits 0..7), component set (8..15), GPUs index (16..18)
// executor state e_st: iteration kind (bits 0..1), last stage run (4..7, 15: none), members (12..20)

struct RegLds {
  uint32_t info[CF_MAX_COMP][CF_MAX_TYPES];
  uint32_t npar[CF_MAX_TYPES];  // parents on the path, 4 bits per component
  double slo[CF_MAX_TYPES][4];
  double tps[CF_MAX_COMP][8];
  double lat[CF_MAX_COMP][5];   // k0, k1, k2, d0, d1
  uint32_t met[CF_MAX_TYPES], cnt[CF_MAX_TYPES];
  uint32_t geo[CF_MAX_EXEC];    // e_geo, indexed per lane by the deliveries
  uint8_t route[CF_MAX_TYPES][2][CF_MAX_COMP];
  uint8_t nalt[CF_MAX_TYPES], aw[CF_MAX_TYPES][2], path[CF_MAX_TYPES], nout[CF_MAX_TYPES], src[CF_MAX_TYPES];
  uint8_t vbase[CF_MAX_NODES], vrep[CF_MAX_NODES], vminc[CF_MAX_NODES], vcomp[CF_MAX_NODES];
  uint8_t vrep1[CF_MAX_NODES], vw[CF_MAX_NODES];
  uint16_t vbatch[CF_MAX_NODES], vbatch2[CF_MAX_NODES];
};

struct Reg {
  const FineArgs *A;
  RegLds *sh;
  // the wavefront's memory (RReq blocks first) and the offsets in it of the
  // running slots (8 bytes: request, step at which it finishes), members,
  // delay line, queue chunks, their links and the free chunks
  CF_GLOBAL char *slab;
  uint32_t o_run, o_mem, o_dl, o_pool, o_next, o_free;
  GPtr<const uint64_t> ticks;  // the seed's arrival ticks
  uint32_t seed;
  double lam, now, dl_head_t, comm;
  uint64_t events, dirty, busy, runm, done_now;  // executor masks: busy, in a multi-step decode run, ended at `now`
  uint32_t status, dl_head, dl_tail, dl_mask;
  int pool_top, pool_fresh, pool_hot, n_chunks, n_done, nx, lat_slot;
  uint32_t nt;
  bool tp_any;
  bool joins;  // some component has several parents on a path
  uint32_t *hrow;
  // executor x in lane x
  double e_end, e_t1, e_dur;  // end of the iteration (+inf: idle); a decode run's first step end and step time
  uint32_t e_itgt, e_st, e_geo;
  // stage instance s in lane s
  uint32_t s_word, s_roff, s_qn, s_qh, s_qt, s_rn, s_iter, s_minfin;
  // component c in lane c
  uint32_t c_word;
  // request (block of 64 arrivals) i in lane i
  double a_t;
  uint64_t a_ex;
  uint32_t a_type;
};

__device__ __forceinline__ CArgs &args(const Reg &S) { return args(S.A); }

// a T at byte offset off of the wavefront's memory
template <typename T>
__device__ __forceinline__ CF_GLOBAL T &at(const Reg &S, uint32_t off) {
  return *(CF_GLOBAL T *)(S.slab + off);
}
// a T at byte off of request r's block
template <typename T>
__device__ __forceinline__ CF_GLOBAL T &req_at(const Reg &S, uint32_t r, uint32_t off) {
  return at<T>(S, r * (uint32_t)sizeof(RReq) + off);
}

// ------------------------------------------------------------------ queues
// The free chunks are a stack whose top stays in a register: a queue that
// empties and fills again takes its chunk back without a memory access.
__device__ __forceinline__ int chunk_alloc(Reg &S) {
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
__device__ __forceinline__ void chunk_free(Reg &S, int c) {
  if (c < 0 || c >= S.n_chunks || S.pool_top >= S.n_chunks) {
    S.status |= CF_ST_OVERFLOW;
    return;
  }
  if (S.pool_hot >= 0) at<int>(S, S.o_free + 4u * (uint32_t)S.pool_top++) = S.pool_hot;  // every lane, the same word
  S.pool_hot = c;
}

// appends, in lane order, the requests r of the lanes `on` (mask bal) to stage si's queue
__device__ __forceinline__ void q_push(Reg &S, int si, uint64_t bal, bool on, uint32_t r) {
  const int cnt = __popcll(bal);
  const uint32_t qn = rl(S.s_qn, si);
  uint32_t qt = rl(S.s_qt, si);
  if (qn == 0) {
    const int c = chunk_alloc(S);
    if (c < 0) return;
    qt = qend(c, 0);
    wl(S.s_qh, si, qt);
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
  wl(S.s_qt, si, cnt <= room ? qt + (uint32_t)cnt : qend(c1, cnt - room));
  wl(S.s_qn, si, qn + (uint32_t)cnt);
}

// appends one request (wave-uniform r)
__device__ __forceinline__ void q_push1(Reg &S, int si, uint32_t r) {
  const uint32_t qn = rl(S.s_qn, si);
  uint32_t qt = rl(S.s_qt, si);
  if (qn == 0) {
    const int c = chunk_alloc(S);
    if (c < 0) return;
    qt = qend(c, 0);
    wl(S.s_qh, si, qt);
  } else if (qend_pos(qt) == kChunk) {
    const int c = chunk_alloc(S);
    if (c < 0) return;
    at<int>(S, S.o_next + 4u * (uint32_t)qend_chunk(qt)) = c;
    qt = qend(c, 0);
  }
  at<uint32_t>(S, S.o_pool + 4u * (uint32_t)(qend_chunk(qt) * kChunk + qend_pos(qt))) = r;
  wl(S.s_qt, si, qt + 1u);
  wl(S.s_qn, si, qn + 1u);
}

// Takes the first k entries of stage si's queue to offset dst, 64 at a time (a
// block spans at most two chunks), and sums their attributes sel.
__device__ __forceinline__ uint32_t q_take(Reg &S, int si, int k, uint32_t dst, uint32_t sel) {
  const uint32_t qh = rl(S.s_qh, si);
  int hc = qend_chunk(qh), hp = qend_pos(qh);
  const int qn = (int)rl(S.s_qn, si);
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
  wl(S.s_qn, si, (uint32_t)(qn - k));
  if (qn == k) chunk_free(S, hc);
  else wl(S.s_qh, si, qend(hc, hp));
  return dpp_sum_u32(xs);
}

__device__ __forceinline__ int stage_in(uint32_t geo, int c) {
  return (int)(geo & 0xFFu) + __popc((geo >> 8) & 0xFFu & ((1u << c) - 1u));
}

// ------------------------------------------------------------------ arrivals
// Prepares the 64 requests from base on: arrival times, routes and blocks.
__device__ __forceinline__ void load_arrivals(Reg &S, uint32_t base) {
  CArgs &A = args(S);
  CModel &m = A.m;
  const RegLds &sh = *S.sh;
  const uint32_t r = base + (uint32_t)lane_id();
  S.a_t = __builtin_inf();
  S.a_ex = ~0ull;
  S.a_type = CF_MAX_TYPES;
  if (r < (uint32_t)A.n) {
    const size_t o = (size_t)S.seed * (size_t)A.n;
    const uint64_t tk = S.ticks[r];
    const uint32_t t = gload(A.type, o, r), ak = gload(A.akey, o, r);
    const uint64_t k0 = gload(A.rkey0, o, r), k1 = gload(A.rkey1, o, r);
    u32x4 w;
    w.x = (uint32_t)gload(A.prompt, o, r) | ((uint32_t)gload(A.out, o, r) << 16);
    w.y = gload(A.patches, o, r);
    w.z = gload(A.aud_in, o, r);
    w.w = gload(A.aud_out, o, r);
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

__device__ __forceinline__ void arrive(Reg &S, uint32_t r) {
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
    q_push1(S, stage_in(rl(S.e_geo, x), c), r);
    S.dirty |= 1ull << x;
  }
}

// ------------------------------------------------------------------ deliveries
// step 2: the delayed deliveries due now, in production order
__device__ __forceinline__ void deliver_due(Reg &S) {
  while (S.dl_head != S.dl_tail && S.dl_head_t == S.now) {
    const uint32_t n = S.dl_tail - S.dl_head;
    u32x4 e = {0, 0x7FF00000u, 0, 0};
    if ((uint32_t)lane_id() < n)
      e = at<u32x4>(S, S.o_dl + ((S.dl_head + (uint32_t)lane_id()) & S.dl_mask) * 16u);
    const double et = words_double(e.x, e.y);
    const uint64_t late = ballot(et != S.now);
    const int k = late ? ff1(late) : 64;  // entries due
    if (k == 0) {  // the head's time is kept in dl_head_t: cannot happen
      S.status |= CF_ST_OVERFLOW;
      return;
    }
    const bool on = lane_id() < k;
    const uint32_t r = e.z >> 4;
    const int c2 = (int)(e.z & 7u);
    u32x4 q = {0, 0, 0, 0};
    if (on) q = req_at<u32x4>(S, r, 0);
    const uint32_t x = (uint32_t)((((uint64_t)q.y << 32) | q.x) >> (8 * c2)) & 63u;
    const uint32_t st = on ? (uint32_t)stage_in(S.sh->geo[x], c2) : 0u;
    if (!S.joins) {
      // one parent everywhere: every delivery enqueues; one push per stage
      for (uint64_t left = ballot(on); left;) {
        const int f = ff1(left);
        const int si = (int)rl(st, f);
        const bool mine = on && (int)st == si;
        const uint64_t bal = ballot(mine);
        S.events += (uint64_t)__popcll(bal);
        q_push(S, si, bal, mine, r);
        S.dirty |= 1ull << rl(x, f);
        left &= ~bal;
      }
    } else {
      // one after the other: two deliveries of a request may be due together
      for (int i = 0; i < k; i++) {
        const uint32_t ri_ = rl(r, i);
        const int ci = (int)rl((uint32_t)c2, i);
        const uint32_t misc = rl(q.w, i);
        CF_GLOBAL uint32_t &jp = req_at<uint32_t>(S, ri_, 8);
        const uint32_t join = ru(jp) + (1u << (4 * ci));
        jp = join;
        const int t = (int)((misc >> 8) & 7u);
        if (((join >> (4 * ci)) & 15u) == ((ru(S.sh->npar[t]) >> (4 * ci)) & 15u)) {
          S.events++;
          q_push1(S, (int)rl(st, i), ri_);
          S.dirty |= 1ull << rl(x, i);
        }
      }
    }
    S.dl_head += (uint32_t)k;
    if (S.dl_head == S.dl_tail) S.dl_head_t = __builtin_inf();
    else if (k < 64) S.dl_head_t = words_double(rl(e.x, k), rl(e.y, k));
    else S.dl_head_t = rdb(at<double>(S, S.o_dl + (S.dl_head & S.dl_mask) * 16u));
  }
}

// ------------------------------------------------------------------ completions
// The n members of an iteration of stage si (component c) of executor x that
// ended now, in member order, 64 per pass.  KIND:
//   IT_BATCH    ENC/GEN members finish their component;
//   IT_PREFILL  members get their first token and finish or join the running set;
//   IT_FINISH   the running slots that finish at step `it` (slot order) finish;
//               the others close the gaps (a kept slot only moves down, and a
//               page is read before it is written).
// Lanes without a member read request 0's block and are masked afterwards:
// every load of a pass is issued unconditionally, with one wait.
template <int KIND>
__device__ __forceinline__ void members(Reg &S, int x, uint32_t geo, int si, int c, int n, uint32_t it) {
  RegLds &sh = *S.sh;
  const uint32_t cw = rl(S.c_word, c);
  const uint32_t chany = (cw >> 16) & 0xFFu;
  const bool outc = (cw >> 24) & 1u, genc = KIND == IT_BATCH && ((cw >> 12) & 3u) == CF_GEN;
  const uint32_t slots = KIND == IT_BATCH ? 0u : S.o_run + rl(S.s_roff, si) * 8u;
  const double now = S.now;
  uint32_t w = 0, mn = kNone;
  for (int b = 0; b < n; b += 64) {
    const int j = b + lane_id();
    bool valid = j < n;
    uint32_t r;
    if constexpr (KIND == IT_FINISH) {
      const uint64_t sv = at<uint64_t>(S, slots + (uint32_t)j * 8u);
      const uint32_t key = (uint32_t)(sv >> 32);
      const bool keep = valid && key != it;
      const uint64_t kb = ballot(keep);
      if (keep) {
        at<uint64_t>(S, slots + (w + lanes_below(kb)) * 8u) = sv;
        mn = key < mn ? key : mn;
      }
      w += (uint32_t)__popcll(kb);
      valid = valid && key == it;
      if (!ballot(valid)) continue;
      r = valid ? (uint32_t)sv : 0u;
    } else {
      r = at<uint32_t>(S, S.o_mem + (uint32_t)(x * CF_MAX_BATCH + j) * 4u);
      r = valid ? r : 0u;
    }
    const u32x4 q = req_at<u32x4>(S, r, 0);
    u32x4 aw, tw;
    uint64_t tkv;
    if constexpr (KIND == IT_PREFILL) aw = req_at<u32x4>(S, r, kOffAttr);
    if (outc) {
      if constexpr (KIND != IT_PREFILL) tw = req_at<u32x4>(S, r, kOffTim);
      tkv = S.ticks[r];
    }
    const uint32_t t = (q.w >> 8) & 7u;
    const uint32_t info = sh.info[c][t];
    bool fin = valid;
    if constexpr (KIND == IT_PREFILL) {
      uint32_t no = attr_in(aw, (cw >> 8) & 7u);
      no = (info & IN_PFO) || no < 1u ? 1u : no;
      fin = valid && no == 1u;
      const uint64_t nb = (uint64_t)__double_as_longlong(now);
      tw = u32x4{(uint32_t)nb, (uint32_t)(nb >> 32), no, 0u};
      if (valid && (info & IN_TTFT)) req_at<u32x4>(S, r, kOffTim) = tw;
      // running-set appends, in member order
      const bool append = valid && no != 1u;
      const uint64_t ab = ballot(append);
      if (ab) {
        const uint32_t rn = rl(S.s_rn, si), key = rl(S.s_iter, si) + no - 1u;
        if (append) at<uint64_t>(S, slots + (rn + lanes_below(ab)) * 8u) = ((uint64_t)key << 32) | r;
        wl(S.s_rn, si, rn + (uint32_t)__popcll(ab));
        const uint32_t km = dpp_min_u32(append ? key : kNone), om = rl(S.s_minfin, si);
        wl(S.s_minfin, si, km < om ? km : om);
      }
      if (!ballot(fin)) continue;
    }
    uint32_t join = q.z, misc = q.w;
    bool put = false;
    // deliveries to the children: remote ones join the delay line, local ones
    // enqueue when the last input is there
    if (chany) {
      const uint32_t ch = fin ? info & 0xFFu : 0u;
      uint32_t rc = 0, ready = 0;
      for (uint32_t cc = chany; cc; cc &= cc - 1) {
        const int c2 = __builtin_ctz(cc);
        const uint32_t bit = ch & (1u << c2);
        const uint32_t xe = ((c2 < 4 ? q.x : q.y) >> (8 * (c2 & 3))) & 0xFFu;
        const bool local = xe == (uint32_t)x;
        rc |= local ? 0u : bit;
        if (!S.joins) {
          ready |= local ? bit : 0u;
        } else if (local && bit) {
          join += 1u << (4 * c2);
          put = true;
          if (((join >> (4 * c2)) & 15u) == ((sh.npar[t] >> (4 * c2)) & 15u)) ready |= bit;
        }
      }
      const uint64_t db = ballot(rc != 0);
      if (db) {
        const uint32_t ndl = (uint32_t)__popc(rc);
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
        for (uint32_t cc = chany; cc; cc &= cc - 1) {
          const int c2 = __builtin_ctz(cc);
          const bool on = (ready >> c2) & 1u;
          const uint64_t bal = ballot(on);
          if (!bal) continue;
          S.events += (uint64_t)__popcll(bal);
          q_push(S, stage_in(geo, c2), bal, on, r);
        }
      }
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
          if (KIND == IT_PREFILL && !here) tw = req_at<u32x4>(S, r, kOffTim);
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
    // the last token's time, unless the request is complete with it
    if (KIND == IT_FINISH && valid && !done && (info & IN_TTFT)) req_at<double>(S, r, kOffLast) = now;
    if (put) req_at<uint64_t>(S, r, 8) = ((uint64_t)misc << 32) | join;
  }
  if constexpr (KIND == IT_FINISH) {
    wl(S.s_rn, si, w);
    wl(S.s_minfin, si, dpp_min_u32(mn));
  }
}

// the iteration of executor x ended now
__device__ __forceinline__ void complete(Reg &S, int x) {
  const uint32_t st = rl(S.e_st, x), geo = rl(S.e_geo, x);
  const uint64_t xbit = 1ull << x;
  const int si = (int)(geo & 0xFFu) + (int)((st >> 4) & 15u);
  S.busy &= ~xbit;
  S.runm &= ~xbit;
  S.dirty |= xbit;
  S.done_now |= xbit;
  wld(S.e_end, x, __builtin_inf());
  const uint32_t kind = st & 3u;
  const int c = (int)(rl(S.s_word, si) & 15u);
  if (kind == IT_DECODE) {
    const uint32_t it0 = rl(S.s_iter, si), rn = rl(S.s_rn, si), it = rl(S.e_itgt, x);
    wl(S.s_iter, si, it);
    S.events += (uint64_t)rn * (uint64_t)(it - it0);
    if (it == rl(S.s_minfin, si)) members<IT_FINISH>(S, x, geo, si, c, (int)rn, it);
  } else {
    const int n = (int)((st >> 12) & 511u);
    S.events += (uint64_t)n;
    if (kind == IT_PREFILL) members<IT_PREFILL>(S, x, geo, si, c, n, 0u);
    else members<IT_BATCH>(S, x, geo, si, c, n, 0u);
  }
}

// ------------------------------------------------------------------ starts
// Starts the next iteration of idle executor x; mb, mp, md: the stages with a
// batch, a prefill, a decode step to run.
__device__ __forceinline__ void try_start(Reg &S, int x, uint64_t mb, uint64_t mp, uint64_t md) {
  const uint32_t geo = rl(S.e_geo, x);
  const int first = (int)(geo & 0xFFu), ns = __popc((geo >> 8) & 0xFFu);
  const uint32_t can = (uint32_t)((mb | mp | md) >> first) & ((1u << ns) - 1u);
  if (!can) return;
  // round robin: the first stage with work after the one run last
  const uint32_t l0 = (rl(S.e_st, x) >> 4) & 15u;
  const uint32_t after = l0 == 15u ? can : can & ~((2u << l0) - 1u);
  const int l = __builtin_ctz(after ? after : can);
  const int si = first + l;
  const uint64_t sbit = 1ull << si, xbit = 1ull << x;
  const uint32_t sw = rl(S.s_word, si);
  const int c = (int)(sw & 15u);
  const uint32_t rn = rl(S.s_rn, si);
  const double tps = S.tp_any ? S.sh->tps[c][(geo >> 16) & 7u] : 1.0;
  double end;
  uint32_t kind, n = rn;
  if ((mb | mp) & sbit) {
    kind = (mb & sbit) ? IT_BATCH : IT_PREFILL;
    const uint32_t beff = (sw >> 8) & 511u, room = kind == IT_PREFILL ? beff - rn : beff, qn = rl(S.s_qn, si);
    n = qn < room ? qn : room;
    const double *lat = S.sh->lat[c];
    const double k0 = lat[0], k1 = lat[1], k2 = lat[2];
    const uint32_t xs = q_take(S, si, (int)n, S.o_mem + (uint32_t)(x * CF_MAX_BATCH * 4), rl(S.c_word, c) & 0x7Fu);
    double dur = (k0 + k1 * (double)xs) + k2 * (double)n;
    if (S.tp_any) dur = tps * dur;
    // an encoder started on an executor that was idle before this instant
    if (((sw >> 4) & 3u) == CF_ENC && !(S.done_now & xbit)) dur = dur + args(S).m.cpu_pre;
    end = S.now + dur;
  } else {
    kind = IT_DECODE;
    double dur = S.sh->lat[c][3] + S.sh->lat[c][4] * (double)rn;
    if (S.tp_any) dur = tps * dur;
    // Decode run: while no input reaches this executor and no other of its
    // stages has work, its next steps are decode steps of this stage with the
    // same members; run to the first finishing step (cut_run cuts it).
    const uint32_t it1 = rl(S.s_iter, si) + 1u, fin = rl(S.s_minfin, si);
    uint32_t itgt = it1;
    end = S.now + dur;
    if ((can & (can - 1u)) == 0 && fin > it1 && dur > 0.0) {
      wld(S.e_t1, x, end);
      wld(S.e_dur, x, dur);
      const uint32_t more = fin - it1 < 65535u ? fin - it1 : 65535u;
      uint32_t taken = 0;
      end = run_walk(end, dur, more, __builtin_inf(), &taken);
      itgt += taken;
      S.runm |= xbit;
    }
    wl(S.e_itgt, x, itgt);
  }
  wld(S.e_end, x, end);
  S.busy |= xbit;
  wl(S.e_st, x, kind | ((uint32_t)l << 4) | (n << 12));
}

// An input reached executor x, in a decode run: the run stops at the first
// step that ends at or after now (the steps before it are unchanged).
__device__ __forceinline__ void cut_run(Reg &S, int x) {
  if (!(lane_val(S.e_end, x) > S.now)) return;
  const int si = (int)(rl(S.e_geo, x) & 0xFFu) + (int)((rl(S.e_st, x) >> 4) & 15u);
  const uint32_t it1 = rl(S.s_iter, si) + 1u;
  uint32_t taken = 0;
  const double t = run_walk(lane_val(S.e_t1, x), lane_val(S.e_dur, x), rl(S.e_itgt, x) - it1, S.now, &taken);
  wld(S.e_end, x, t);
  wl(S.e_itgt, x, it1 + taken);
  if (taken == 0) S.runm &= ~(1ull << x);
}

// ------------------------------------------------------------------ setup
// Plan p into LDS and registers; false: the plan is malformed.
__device__ __forceinline__ bool setup_plan(Reg &S, int p) {
  CArgs &A = args(S);
  CModel &m = A.m;
  RegLds &sh = *S.sh;
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
  int base = 0, nsi = 0, run_need = 0;
  for (int v = 0; v < nv; v++) {
    const uint32_t cm = ru(sh.vcomp[v]);
    const int rep = ri(sh.vrep[v]), rep1 = ri(sh.vrep1[v]), b1 = ri(sh.vbatch[v]), b2 = ri(sh.vbatch2[v]);
    sh.vbase[v] = (uint8_t)(base < 255 ? base : 255);
    base += rep;
    nsi += rep * __popc(cm);
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
  if (nsi > kRegStages || run_need > A.L.run_cap) {
    S.status |= CF_ST_OVERFLOW;
    return true;
  }
  S.nx = base;
  // executors, one lane each
  if (lane < base) {
    int v = 0, first = 0;
    while (v + 1 < nv && sh.vbase[v + 1] <= lane) {
      first += sh.vrep[v] * __popc((uint32_t)sh.vcomp[v]);
      v++;
    }
    const uint32_t cm = sh.vcomp[v];
    const int j = lane - sh.vbase[v];
    uint32_t tp = 0;
    if (m.tp_any) {
      const uint32_t g = j >= sh.vrep1[v] ? A.node_gpus2[v * P + p] : A.node_gpus[v * P + p];
      tp = g < 1 ? 0 : (g > 8 ? 7 : g - 1);
    }
    S.e_geo = (uint32_t)(first + j * __popc(cm)) | (cm << 8) | (tp << 16);
    sh.geo[lane] = S.e_geo;
  }
  // stage instances, one lane each
  int c = 0, beff = 0, x = 0;
  bool llm = false;
  if (lane < nsi) {
    int v = 0, acc = 0;
    while (acc + sh.vrep[v] * __popc((uint32_t)sh.vcomp[v]) <= lane) {
      acc += sh.vrep[v] * __popc((uint32_t)sh.vcomp[v]);
      v++;
    }
    uint32_t cc = sh.vcomp[v];
    const int per = __popc(cc), e = (lane - acc) / per;
    for (int k = (lane - acc) - e * per; k > 0; k--) cc &= cc - 1;
    c = __builtin_ctz(cc);
    x = sh.vbase[v] + e;
    const int bn = e < sh.vrep1[v] ? sh.vbatch[v] : sh.vbatch2[v];
    beff = bn < m.cap[c] ? bn : m.cap[c];
    llm = m.kind[c] == CF_LLM;
  }
  uint32_t tot;
  S.s_roff = wave_excl_scan(llm ? (uint32_t)beff : 0u, tot);
  S.s_word = (uint32_t)c | ((uint32_t)m.kind[c] << 4) | ((uint32_t)beff << 8) | ((uint32_t)x << 20);
  __syncthreads();
  return true;
}

__device__ __forceinline__ void setup_model(Reg &S) {
  CModel &m = args(S).m;
  RegLds &sh = *S.sh;
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
      if (m.ttft_c[t] >= 0) w |= IN_LLM;
    }
    sh.info[c][t] = w;
    sh.tps[c][t] = m.tps[c][t];
  }
  bool joins = false;
  if (lane < CF_MAX_TYPES) {
    uint32_t np = 0;
    for (int c = 0; c < CF_MAX_COMP; c++) {
      np |= (uint32_t)(m.npar[lane][c] & 15u) << (4 * c);
      joins |= m.npar[lane][c] > 1;
    }
    sh.npar[lane] = np;
    sh.path[lane] = (uint8_t)m.path[lane];
    sh.nout[lane] = (uint8_t)__popc(m.outm[lane]);
    sh.src[lane] = (uint8_t)m.srcm[lane];
  }
  S.joins = ballot(joins) != 0;
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
               (chany << 16) | (out << 24);
  }
}

// 80 VGPRs, 6 wavefronts per SIMD (8 VGPRs and 73 SGPRs spilled): 5 and 7 per
// SIMD measure within 3 % on full launches, 7 is 4 % slower alone.
__global__ void __launch_bounds__(64, 6) k_fine_reg(const FineArgs *__restrict__ Ap) {
  __shared__ RegLds sh;
  const int lane = lane_id();
  Reg S;
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
    S.dl_mask = L.dl_mask;
    S.n_chunks = L.n_chunks;
    S.comm = A.m.comm;
    S.nt = (uint32_t)A.m.nt;
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
    S.e_t1 = per_lane(0.0);
    S.e_dur = per_lane(0.0);
    S.e_itgt = per_lane(0u);
    S.e_st = per_lane(15u << 4);  // no stage run yet
    S.s_qn = per_lane(0u);
    S.s_qh = per_lane(0u);
    S.s_qt = per_lane(0u);
    S.s_rn = per_lane(0u);
    S.s_iter = per_lane(0u);
    S.s_minfin = per_lane(kNone);
    S.a_t = __builtin_inf();
    S.a_ex = ~0ull;
    S.e_geo = S.a_type = S.s_word = S.s_roff = 0;
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
        // --- next pending time: the earliest iteration end (the ends of idle
        // executors are +inf; non-negative doubles order like their bits), the
        // executors ending then, the delay line's head and the next arrival
        const uint64_t eb = (uint64_t)__double_as_longlong(S.e_end);
        const uint32_t hi = (uint32_t)(eb >> 32);
        const uint32_t hmin = dpp_min_u32(hi);
        uint64_t ends = ballot(hi == hmin);
        double te = __builtin_inf();
        if (hmin != 0x7FF00000u) {
          uint32_t lmin;
          if ((ends & (ends - 1)) == 0) {
            lmin = rl((uint32_t)eb, ff1(ends));
          } else {
            lmin = dpp_min_u32(hi == hmin ? (uint32_t)eb : ~0u);
            ends = ballot(hi == hmin && (uint32_t)eb == lmin);
          }
          te = words_double(lmin, hmin);
        } else if (ballot(eb < 0x7FF0000000000000ull) == 0) {
          ends = 0;
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
        // --- step 3: executors whose state changed: cut runs, start iterations
        __syncthreads();
        uint64_t cand = S.dirty & ~S.busy, cut = S.dirty & S.runm;
        S.dirty = 0;
        while (cut) {
          const int x = ff1(cut);
          cut &= cut - 1;
          cut_run(S, x);
        }
        if (cand) {
          const uint32_t sw = S.s_word;
          const bool llm = ((sw >> 4) & 3u) == CF_LLM;
          const uint64_t q = ballot(S.s_qn > 0), ml = ballot(llm);
          const uint64_t mp = ballot(S.s_rn < ((sw >> 8) & 511u)) & q & ml;
          const uint64_t md = ballot(S.s_rn > 0) & ml, mb = q & ~ml;
          do {
            const int x = ff1(cand);
            cand &= cand - 1;
            try_start(S, x, mb, mp, md);
          } while (cand);
        }
        if (S.status & (CF_ST_OVERFLOW | CF_ST_INVALID)) break;
      }
      if (S.n_done < A.n && !(S.status & (CF_ST_OVERFLOW | CF_ST_INVALID))) S.status |= CF_ST_DEADLOCK;
    }
    __syncthreads();
    CArgs &Ao = args(S);
    if (lane < (int)S.nt) {
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

void launch_fine_reg(const FineArgs *args, unsigned waves, hipStream_t s) {
  hipLaunchKernelGGL(k_fine_reg, dim3(waves), dim3(64), 0, s, args);
}

}  // namespace fine
}  // namespace cf
