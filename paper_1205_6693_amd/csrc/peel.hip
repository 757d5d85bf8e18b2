// Peeling (Algorithm 2, made level-synchronous).
//
// Level k removes every live edge whose support is at most k-2 and gives it
// truss number k.  Within a level the frontier F_r of sub-round r is a snapshot:
// an edge joins F_r by having its round stamp set to r, and an edge counts as
// removed once its stamp is non-zero and below the current round.  A triangle
// whose three edges are not removed and which has at least one edge in F_r is
// destroyed in round r; only its F_r edge of smallest id processes it, and that
// edge decrements each of the triangle's other edges that is not in F_r exactly
// once (the two decrements of Algorithm 2).  After round r every live
// edge's support therefore equals its support in the graph without
// F_0 ∪ ... ∪ F_r, which is the sequential invariant, so the truss numbers
// match Algorithm 2 whatever the order of removals inside a level.
//
// Triangles through a frontier edge e = (u, v) are found as in Algorithm 2,
// by its triangle walk: walk the adjacency row of the endpoint with the shorter live row,
// and look each neighbour w up in the other endpoint's row (hash table or
// binary search).  Deleted edges are only marked (Section 3.1); the rows are compacted
// in place whenever the live edge count has fallen below 70 % of their entries.
//
// What bounds a round is a chain of dependent memory accesses (about 0.7 us
// each at the coherent level) up to some 10^6 walk entries, and memory
// throughput above.  So a frontier is kept as finished walk records, appended
// when an edge joins it (its endpoints are at hand then) together with the
// start of its walk among all walks of the round laid end to end: the next
// round cuts that length into equal parts and every workgroup finds the
// records of its part by itself, with no work handed from one workgroup to another.
// Drawing chunks of the frontier and announcing pieces of their walks to idle
// workgroups took 47 us for a round of 580 K entries and 105 us for one of 2 M, this
// 36 and 73 us (R-MAT of 15.7 M edges: rounds 110.8 -> 86.4 ms of a call).
//
// The level loop runs in a persistent kernel, one 1024-thread workgroup per
// compute unit (fewer on small graphs).  The grid is never larger than the number of workgroups the
// device holds at once (one per compute unit, checked against the occupancy
// of the kernel before the first launch), so every workgroup is resident and
// the grid barrier can complete; the launch is an ordinary one on the
// caller's stream (a cooperative launch goes through a queue of its own,
// which profilers tear down at exit after the run's results are written, and
// adds nothing here).  Phases are separated by a grid barrier; the last
// workgroup to arrive runs the control step (next phase, next level
// k = max(k+1, min live support + 2), queue sizes) before releasing the others.
// The kernel returns to the host only to compact the rows (a separate kernel)
// or when every edge is removed.
//
// Memory coherence (see grid_barrier): every value that one phase writes and a
// later phase of another workgroup reads (queues, live lists, round stamps,
// supports) is written and read with agent-scope relaxed atomics.  Adjacency
// rows, offsets and row lengths are immutable inside a launch and use ordinary
// cached loads.
//
// Each level runs in one of four ways, decided when its first frontier is
// known: the frontier mode (SPARSE enqueues an edge the moment its support
// drops from k-1 to k-2, the queue of Section 3.1; DENSE re-scans the live
// edges after every sub-round) and the membership probe (the edge
// hash table, or a binary search of the other endpoint's sorted row).  The scheduler
// (plain, a fixed heuristic, or the learned network evaluated by the control
// wavefront) only picks among these exact methods.
#include "common.hpp"
#include "internal.hpp"
#include "mlp.hpp"

namespace truss {

namespace {

constexpr int kT = 1024;
constexpr int kWaves = kT / kWave;
constexpr int kIntMax = 0x7fffffff;
constexpr int kHistBins = 6;
// Rows are compacted when the live entries fall to kCompactNum / kCompactDen of those
// they hold.  With 0.85 / 0.8 / 0.75 / 0.7 (the list as below): 13.7, 13.4, 13.2 and 13.0 ms
// a call on R-MAT of 1.2 M edges, - / 83.5 / 82.9 / 83.0 on 15.7 M, - / 84.6 / 83.5 / 83.3
// on Chung-Lu of 15.5 M, 1162 / 1145 / 1152 / 1141 on R-MAT 23.
constexpr long long kCompactNum = 7, kCompactDen = 10;
// Rows that hold fewer edges are not compacted any more: the way through the host
// costs some 60 us, more than walking the removed entries to the end does
// (G(2000, 0.01), 20 K edges: the call 0.47 -> 0.36 ms, with the waits below).
constexpr long long kCompactMin = 1 << 15;
constexpr int kStageQ = 16384;  // LDS staging of a list phase's frontier (entries)

// The support of an edge that has joined a frontier is set to kGone, so that the
// list phases tell live edges by their support alone.  Later decrements (fewer than
// the edge has triangles) leave it above kGoneMin; the supports out of reach that
// frozen edges start with (2^29) lie below.
constexpr int kGone = 1 << 30, kGoneMin = 3 << 28;

// The live list is written anew in a sweep once half of its edges are gone: a sweep
// reads 4 bytes of list and a line of supports per some edges, a rewrite takes a
// block scan and an atomic per step.  At 3/4, 1/2, 1/3 and 1/4 left: sweeps 5.48, 4.77,
// 5.06 and 4.99 ms on R-MAT of 15.7 M edges, 57.4, 48.2, 52.0 ms (3/4 to 1/3) on R-MAT 23.
constexpr long long kListNum = 1, kListDen = 2;

// A round's walks, laid end to end in queue order, are cut into parts of equal
// length: one a workgroup while that length lies between kMinChunk and kPartMax
// entries; shorter rounds use fewer workgroups, and longer ones cut parts of
// kPartMax entries which the workgroups draw one after another, so that no
// workgroup waits long for the last one.  Measured (whole calls, R-MAT of 1.2 M
// and 15.7 M edges, Chung-Lu of 15.5 M): kMinChunk 64 / 256 / 1024: 22.1 / 22.6 /
// 23.7, 114.0 / 115.1 / 117.2 and 117.4 / 117.9 / 123.2 ms; kPartMax 8192 / 16384 /
// 32768: 117.9 / 116.0 / 116.3 ms on the second.
constexpr int kMinChunk = 64;  // entries of the smallest part: one a lane of one wavefront
constexpr long long kPartMax = 16384;

enum Phase : int {
  PH_SWEEP = 0,    // minimum live support and the next level's first frontier
  PH_START = 1,    // level start: collect live edges with sup <= k-2
  PH_PROC = 2,     // destroy the triangles of F_r
  PH_DENSE = 4,    // dense mode: collect the next frontier by re-scan
  PH_COMPACT = 5,  // return to the host: drop removed entries from the rows
  PH_DONE = 6
};

// Working counters of one phase, each on its own 128-byte line.  Two sets
// alternate from phase to phase: the control step that reads one resets it
// for the phase after the next, so the release of the next phase need not
// wait for the reset.
struct alignas(128) PhaseCounts {
  alignas(128) int fetch;                  // parts of the round drawn
  alignas(128) unsigned long long q;       // next frontier: (walk units << qbits) | edges
  alignas(128) int alive;                  // entries of the list being written
  alignas(128) int minsup;                 // minimum live support
  alignas(128) unsigned long long fwork;   // level start: sum over F_0 of the shorter live row
};

// what the workgroups need of the control state in a phase (published words)
enum Pub : int { PUB_FLAGS = 0, PUB_K = 1, PUB_R = 2, PUB_UNITS = 3, PUB_ACNT = 4, kPub = 5 };

struct alignas(256) PeelCtl {
  GridBarrier bar;
  PhaseCounts w[2];
  alignas(128) unsigned long long w_work;
  alignas(128) unsigned bar_gen;  // barriers passed before this launch
  // published control state, written only by the control step
  int phase;
  int k;
  int r;
  int qlen;
  unsigned long long qunits;  // walk units of the round
  int acnt;     // length of the live list
  int acur;     // which list
  int first;    // the list is still all edges, in order
  int compact;  // the next sweep writes a new list
  int mode;
  int kmax;
  int levels;
  long long removed_level;
  long long removed;      // edges of the finished levels
  long long csr_live;
  long long subrounds;
  long long heavy_rounds;
  long long max_subrounds;
  long long hist[kHistBins];
  unsigned long long t_last;            // wall clock at the previous barrier
  unsigned long long t_phase[8];        // time spent per phase (100 MHz ticks)
  int err;
  // scheduling
  int probe;               // membership probe of the current level: 0 row hash table, 1 binary search
  int sched;               // TRUSS_SCHED_* in effect
  int fix_bits, fix_vals;  // action bits fixed by the options
  int qbits;               // bits of the edge count in w_q
  int input_err;           // RunHead::err when the peeling began
  unsigned long long sup_total;
  int stop_level;          // > 0: no level above it is started
  long long lvl_sub0;      // sub-rounds before the current level
  long long prev_sub;      // sub-rounds of the previous level
  unsigned long long t_dec;  // wall clock at the current level's decision
};

// What a walk needs of a vertex, in one 16-byte load: its row (a symmetric CSR
// of m < 2^31 edges has fewer than 2^32 entries), the live row length and its
// hash table (offset of up to 2^34 slots, log2 of the slots).
struct alignas(16) VInfo {
  uint32_t base;
  int32_t len;
  unsigned long long tab;  // (offset << 6) | lg
};

// A frontier, as its walks: record x is edge e = (a, b) with a the endpoint of
// the shorter live row, which is walked and whose neighbours are looked up
// in b's table.  pre is the start of the walk among the frontier's walks laid
// end to end, in units of 2^shift entries.
struct FrontierQueue {
  unsigned long long* pre;
  unsigned long long* eb;   // (row start of a << 32) | e
  unsigned long long* ab;   // (b << 32) | a
  unsigned long long* tab;  // b's table
};

struct PeelArgs {
  int32_t n;
  int64_t m;
  const int32_t* col;
  const int32_t* seid;
  const VInfo* vinfo;
  const int32_t* eu;
  const int32_t* ev;
  // support and round stamp, in arrays of their own: a walk's first edges have
  // consecutive ids, and both its stamp reads and its decrements are served by
  // the 64-byte line (atomics at about 25 G lines/s), so 4 bytes an edge halve their
  // number against interleaved pairs
  int32_t* sup;
  int32_t* stamp;
  int32_t* truss;
  int32_t* alist[2];
  FrontierQueue fq[2];
  const int2* rtab;           // row hash tables
  PeelCtl* ctl;
  const RunHead* head;
  const float* model;         // peeling model part (learned scheduler), or null
  float* tr_feat;             // per-level trace (tr_cap rows), or null
  float* tr_ms;
  int32_t* tr_act;
  int tr_cap;
};

__device__ __forceinline__ int hist_bin(long long q) {
  return q <= 1 ? 0 : q <= 16 ? 1 : q <= 256 ? 2 : q <= 4096 ? 3 : q <= 65536 ? 4 : 5;
}

// Entries per walk unit (log2): 0 wherever the longest round the graph allows
// (wbound entries: the sum of the shorter row over all edges) fits in the
// counter's 64 - qbits bits, as on every graph of up to some 100 M edges;
// otherwise the smallest power of two for which the units fit.
__device__ __forceinline__ int walk_shift(unsigned long long wbound, int64_t m, int qbits) {
  int s = 0;
  while ((wbound >> s) + (unsigned long long)m >= (1ULL << (63 - qbits))) ++s;
  return s;
}

// The published state of a phase.
struct PhaseState {
  int phase, acur, mode, probe, first, compact, qlen, k, r, acnt;
  unsigned long long units;
};
__device__ __forceinline__ unsigned long long pub_word(const PhaseState& s, int i) {
  switch (i) {
    case PUB_FLAGS:
      return (unsigned long long)(unsigned)(s.phase | (s.acur << 3) | (s.mode << 4) | (s.probe << 6) | (s.first << 7) |
                                           (s.compact << 8)) |
             ((unsigned long long)(unsigned)s.qlen << 9);
    case PUB_K: return (unsigned)s.k;
    case PUB_R: return (unsigned)s.r;
    case PUB_UNITS: return s.units;
    default: return (unsigned)s.acnt;
  }
}
// from the published words in LDS; the same in all lanes
__device__ __forceinline__ PhaseState phase_state(const unsigned long long* pub) {
  PhaseState s;
  const unsigned long long f = scalar64(pub[PUB_FLAGS]);
  s.phase = (int)(f & 7);
  s.acur = (int)(f >> 3) & 1;
  s.mode = (int)(f >> 4) & 3;
  s.probe = (int)(f >> 6) & 1;
  s.first = (int)(f >> 7) & 1;
  s.compact = (int)(f >> 8) & 1;
  s.qlen = (int)(f >> 9);
  s.k = (int)scalar64(pub[PUB_K]);
  s.r = (int)scalar64(pub[PUB_R]);
  s.acnt = (int)scalar64(pub[PUB_ACNT]);
  s.units = scalar64(pub[PUB_UNITS]);
  return s;
}
static_assert(TRUSS_PEEL_SPARSE < 4 && TRUSS_PEEL_DENSE < 4 && PH_DONE < 8, "fields of PUB_FLAGS");

// ---- control step: the first wavefront of the last workgroup to reach a barrier ---------------
// All inputs are loaded first (independent loads in flight together; the
// published state is at hand), the decision is made in registers and released,
// and lane 0 stores the rest of the state afterwards: the next control step
// reads it after this workgroup's next arrival.  Every value is the same in all
// lanes; the lanes evaluate the scheduler's network together (one hidden unit
// each).  st: the state of the phase that has ended, on return that of the
// next one; gen: barriers passed including this one.
template <typename Release>
__device__ __forceinline__ void control_step(PeelCtl* c, const PeelArgs& P, PhaseState& st, unsigned gen, int shift,
                                             Release release) {
  const bool lead = lane_id() == 0;
  PhaseCounts* const w = &c->w[(gen - 1) & 1];
  int phase = st.phase;
  int k = st.k;
  int r = st.r;
  int acnt = st.acnt;
  int acur = st.acur;
  const int mode_in = st.mode;
  const unsigned long long qunits_in = st.units;
  int levels = ldc(&c->levels);
  long long removed_level = ldc(&c->removed_level);
  long long removed = ldc(&c->removed);
  long long csr_live = ldc(&c->csr_live);
  long long subrounds = ldc(&c->subrounds);
  long long heavy_rounds = ldc(&c->heavy_rounds);
  const long long maxsr = ldc(&c->max_subrounds);
  const unsigned long long t_last = ldc(&c->t_last);
  const int qbits = ldc(&c->qbits);
  const unsigned long long w_q = ldc(&w->q);
  const int w_qlen = (int)(w_q & ((1ULL << qbits) - 1ULL));
  const int w_alive = ldc(&w->alive);
  const int w_minsup = ldc(&w->minsup);
  const unsigned long long w_fwork = ldc(&w->fwork);
  const int sched = ldc(&c->sched);
  const int fix_bits = ldc(&c->fix_bits);
  const int fix_vals = ldc(&c->fix_vals);
  const int stop_level = ldc(&c->stop_level);
  long long lvl_sub0 = ldc(&c->lvl_sub0);
  long long prev_sub = ldc(&c->prev_sub);
  unsigned long long t_dec = ldc(&c->t_dec);
  const int phase_in = phase;
  const unsigned long long t_ph = ldc(&c->t_phase[phase_in]);
  const unsigned long long now = wall_clock64();
  int hist_bin_out = -1;
  bool failed = false;

  auto begin_round = [&](int q) {
    st.qlen = q;
    st.units = w_q >> qbits;
    subrounds += 1;
    hist_bin_out = hist_bin(q);
    phase = PH_PROC;
  };
  auto next_round = [&]() {
    if (w_qlen > 0) {
      r += 1;
      removed_level += w_qlen;
      begin_round(w_qlen);
    } else {
      // level finished
      const int li = levels - 1;
      if (lead && li < P.tr_cap && P.tr_ms) P.tr_ms[li] = (float)((double)(now - t_dec) * 1e-5);
      prev_sub = subrounds - lvl_sub0;
      // compact the rows when the live count has dropped below kCompactNum /
      // kCompactDen of the entries they hold
      removed += removed_level;
      removed_level = 0;
      const long long alive_after = P.m - removed;
      st.compact = alive_after * kListDen < (long long)acnt * kListNum ? 1 : 0;
      if (csr_live >= kCompactMin && alive_after > 0 && alive_after * kCompactDen < csr_live * kCompactNum) {
        csr_live = alive_after;
        phase = PH_COMPACT;
      } else {
        phase = PH_SWEEP;
      }
    }
  };
  // the level's decision, from features that are the same whatever earlier
  // levels chose; then the level's first round
  auto start_level = [&]() {
        float x[kPeelF];
        const float live = (float)(P.m - removed), f0 = (float)w_qlen, wk = (float)w_fwork;
        x[0] = log2f(1.f + live);
        x[1] = log2f(1.f + f0);
        x[2] = f0 / (live > 1.f ? live : 1.f);
        x[3] = log2f((float)k);
        x[4] = log2f(1.f + wk);
        x[5] = log2f(1.f + wk / (f0 > 1.f ? f0 : 1.f));
        x[6] = live / (float)(csr_live > 1 ? csr_live : 1);
        x[7] = log2f(1.f + (float)prev_sub);
        int act;
        if (sched == TRUSS_SCHED_LEARNED && P.model) {
          float sc[kPeelA];
          mlp_scores_wave(P.model, x, sc);
          unsigned mask = 0;
          for (int a = 0; a < kPeelA; ++a)
            if ((a & fix_bits) == fix_vals) mask |= 1u << a;
          act = argmin_allowed(sc, kPeelA, mask);
        } else {
          // the heuristic: sparse and the row hash table, whatever the level
          const int pref = sched == TRUSS_SCHED_PLAIN ? 3 : 0;
          act = (pref & ~fix_bits) | fix_vals;
        }
        st.mode = (act & 2) ? (int)TRUSS_PEEL_DENSE : (int)TRUSS_PEEL_SPARSE;
        st.probe = act & 1;
        const int li = levels - 1;  // trace row of the level
        if (lead && li < P.tr_cap && P.tr_feat) {
          for (int i = 0; i < kPeelF; ++i) P.tr_feat[(int64_t)li * kPeelF + i] = x[i];
          P.tr_act[li] = act;
        }
        lvl_sub0 = subrounds;
        t_dec = now;
        begin_round(w_qlen);
  };
  switch (phase) {
    case PH_SWEEP:
      // the sweep has also taken the live edges with sup <= k-1, the frontier
      // of level k+1 (stamped r+1); it is the level's F_0 unless empty, which
      // happens exactly when the minimum live support is at least k, so that
      // the next level is min + 2 and needs its own start phase
      if (st.compact) {
        acnt = w_alive;
        acur ^= 1;
        st.first = 0;
      }
      if (removed == P.m || (stop_level > 0 && (w_qlen > 0 ? k + 1 : w_minsup + 2) > stop_level)) {
        phase = PH_DONE;
        break;
      }
      levels += 1;
      r += 1;
      if (w_qlen > 0) {
        k = k + 1;
        removed_level = w_qlen;
        start_level();
      } else {
        k = w_minsup + 2;
        removed_level = 0;
        phase = PH_START;
      }
      break;
    case PH_START:
      removed_level = w_qlen;
      if (w_qlen > 0) start_level();
      else phase = PH_SWEEP;
      break;
    case PH_PROC:
      if ((qunits_in << shift) > (unsigned long long)kT) heavy_rounds += 1;
      if (mode_in == TRUSS_PEEL_DENSE) {
        phase = PH_DENSE;
        break;
      }
      next_round();
      break;
    case PH_DENSE:
      next_round();
      break;
    default:
      phase = PH_DONE;
  }
  if (maxsr > 0 && subrounds > maxsr && phase != PH_DONE) {
    failed = true;
    phase = PH_DONE;
  }
  st.phase = phase;
  st.k = k;
  st.r = r;
  st.acnt = acnt;
  st.acur = acur;
  release(pub_word(st, lane_id()));
  if (!lead) return;
  if (failed) stc(&c->err, (int)TRUSS_E_INTERNAL);
  if (t_last != 0) stc(&c->t_phase[phase_in], t_ph + (now - t_last));
  stc(&c->t_last, now);
  if (hist_bin_out >= 0) stc(&c->hist[hist_bin_out], ldc(&c->hist[hist_bin_out]) + 1);
  stc(&w->fetch, 0);
  stc(&w->q, 0ULL);
  stc(&w->alive, 0);
  stc(&w->minsup, kIntMax);
  stc(&w->fwork, 0ULL);
  stc(&c->bar_gen, gen);
  stc(&c->k, k);
  stc(&c->kmax, k);
  stc(&c->r, r);
  stc(&c->acnt, acnt);
  stc(&c->acur, acur);
  stc(&c->first, st.first);
  stc(&c->compact, st.compact);
  stc(&c->mode, st.mode);
  stc(&c->probe, st.probe);
  stc(&c->qlen, st.qlen);
  stc(&c->qunits, st.units);
  stc(&c->levels, levels);
  stc(&c->removed_level, removed_level);
  stc(&c->removed, removed);
  stc(&c->csr_live, csr_live);
  stc(&c->subrounds, subrounds);
  stc(&c->heavy_rounds, heavy_rounds);
  stc(&c->lvl_sub0, lvl_sub0);
  stc(&c->prev_sub, prev_sub);
  stc(&c->t_dec, t_dec);
  stc(&c->phase, phase);
}

// The grid barrier between two phases; on return st is the state of the next one.
__device__ __forceinline__ bool phase_barrier(PeelCtl* c, const PeelArgs& P, PhaseState& st, unsigned gen, int shift,
                                              unsigned long long* pub) {
  const bool ok = grid_barrier<kPub>(&c->bar, gen, pub,
                                     [&](auto release) { control_step(c, P, st, gen, shift, release); });
  st = phase_state(pub);
  return ok;
}

__device__ __forceinline__ bool removed_at(int rnd, int r) { return rnd != 0 && rnd < r; }

// The frontier records of one part being walked (LDS).
struct WalkTabs {
  int pre[kT + 1];          // start of the walk, in units, relative to the part
  int e[kT], a[kT], b[kT];
  uint32_t base[kT];
  unsigned long long tab[kT];
  int len[kT];              // only with more than one entry a unit
};

// NI adjacency entries of walks, one step at a time for all of them so that
// their memory accesses are in flight together.  Entry q is position j[q] of
// the row walked for the frontier record x[q] of W (edge e = (a, b)), valid if
// ok[q].  HALF: a lookup reads the other half of a bucket only when the home half
// does not settle it, which costs short rounds a hop through memory and saves
// long ones accesses.  Outputs the (up to two) edges per entry whose support crossed
// k-1 -> k-2 and must be enqueued: f1 = (a, w) and f2 = (b, w).
template <int NI, bool HALF>
__device__ __forceinline__ void process_entries(const PeelArgs& P, const WalkTabs& W, const int (&x)[NI],
                                                const uint32_t (&j)[NI], bool (&ok)[NI], int r, int l, int k,
                                                bool sparse, int probe, int32_t (&w)[NI], int32_t (&f1)[NI],
                                                int32_t (&f2)[NI]) {
  int32_t e1[NI], e2[NI], s1[NI], s2[NI];
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    f1[q] = -1;
    f2[q] = -1;
    w[q] = -1;
    e1[q] = 0;
    e2[q] = 0;
    s1[q] = 0;
    s2[q] = 0;
    if (ok[q]) {
      w[q] = P.col[j[q]];
      e1[q] = P.seid[j[q]];
    }
  }
  // the first other edge (a, w) must not be removed
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    ok[q] = ok[q] && w[q] != W.b[x[q]];
    if (ok[q]) s1[q] = ldc(&P.stamp[e1[q]]);
  }
#pragma unroll
  for (int q = 0; q < NI; ++q) ok[q] = ok[q] && !removed_at(s1[q], r);
  // the second other edge (b, w): b's row hash table, or a binary search of
  // b's sorted row (the entries of one walk look up the same row, so they
  // touch the same few cached lines either way)
  if (probe == 0) {
    const int2* tb[NI];
    uint32_t h[NI], mask[NI];
    int4 sa[NI], sb[NI];
#pragma unroll
    for (int q = 0; q < NI; ++q) {  // the home buckets of all lookups in flight together
      tb[q] = P.rtab;
      h[q] = 0;
      mask[q] = 0;
      sa[q] = make_int4(-1, 0, -1, 0);
      sb[q] = sa[q];
      if (ok[q]) {
        const unsigned long long tab = W.tab[x[q]];
        const int lg = (int)(tab & 63);
        tb[q] = P.rtab + (tab >> 6);
        mask[q] = (1u << lg) - 1u;
        h[q] = row_slot(w[q], lg) & ~1u;
        sa[q] = *(const int4*)(tb[q] + h[q]);
        if (!HALF) sb[q] = *(const int4*)(tb[q] + (h[q] ^ 2u));
      }
    }
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      if (!ok[q]) continue;
      for (;;) {
        const int4 a = sa[q];
        if (HALF) {
          e2[q] = half_find(a, w[q]);
          if (e2[q] >= 0 || half_open(a)) break;
          sb[q] = *(const int4*)(tb[q] + (h[q] ^ 2u));
        }
        const int4 b = sb[q];
        if (!HALF) e2[q] = half_find(a, w[q]);
        if (e2[q] < 0) e2[q] = half_find(b, w[q]);
        if (e2[q] >= 0 || half_open(a) || half_open(b)) break;
        h[q] = (h[q] + 4) & mask[q];
        sa[q] = *(const int4*)(tb[q] + h[q]);
        if (!HALF) sb[q] = *(const int4*)(tb[q] + (h[q] ^ 2u));
      }
      ok[q] = e2[q] >= 0;
    }
  } else {
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      if (!ok[q]) continue;
      const VInfo vb = P.vinfo[W.b[x[q]]];
      const int64_t rb = vb.base;
      const int64_t re = rb + vb.len;
      const int64_t p = lower_bound_i32<int64_t>(P.col, rb, re, w[q]);
      if (p < re && P.col[p] == w[q]) e2[q] = P.seid[p];
      else ok[q] = false;
    }
  }
#pragma unroll
  for (int q = 0; q < NI; ++q)
    if (ok[q]) s2[q] = ldc(&P.stamp[e2[q]]);
  // the triangle is destroyed now unless an edge is removed, and it belongs
  // to its frontier edge of smallest id; each other edge not in F_r loses one
  bool d1[NI], d2[NI];
  int old1[NI], old2[NI];
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    const int e = W.e[x[q]];
    const bool live = ok[q] && !removed_at(s2[q], r) && !(s1[q] == r && e1[q] < e) && !(s2[q] == r && e2[q] < e);
    d1[q] = live && s1[q] != r;
    d2[q] = live && s2[q] != r;
    old1[q] = 0;
    old2[q] = 0;
    if (d1[q]) old1[q] = atomicSub(&P.sup[e1[q]], 1);
    if (d2[q]) old2[q] = atomicSub(&P.sup[e2[q]], 1);
  }
  if (!sparse) return;
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    if (d1[q] && old1[q] == l + 1) {
      stc(&P.stamp[e1[q]], r + 1);
      stc(&P.sup[e1[q]], kGone);
      P.truss[e1[q]] = k;
      f1[q] = e1[q];
    }
    if (d2[q] && old2[q] == l + 1) {
      stc(&P.stamp[e2[q]], r + 1);
      stc(&P.sup[e2[q]], kGone);
      P.truss[e2[q]] = k;
      f2[q] = e2[q];
    }
  }
}

// One edge of a new frontier with endpoints u, v: which row is walked (the
// shorter live one, ties by id), where it starts and its length.
struct Walk {
  int32_t a, b;
  uint32_t base;
  int len;
  unsigned long long tab;
};
__device__ __forceinline__ Walk walk_of(const PeelArgs& P, int32_t u, int32_t v) {
  const VInfo x = P.vinfo[u], y = P.vinfo[v];
  const bool ua = x.len < y.len || (x.len == y.len && u < v);
  Walk r;
  r.a = ua ? u : v;
  r.b = ua ? v : u;
  r.base = ua ? x.base : y.base;
  r.len = ua ? x.len : y.len;
  r.tab = ua ? y.tab : x.tab;
  return r;
}

__device__ __forceinline__ void put_record(const FrontierQueue& Q, int64_t at, unsigned long long pre, int32_t e,
                                           const Walk& w) {
  stc(&Q.pre[at], pre);
  stc(&Q.eb[at], ((unsigned long long)w.base << 32) | (uint32_t)e);
  stc(&Q.ab[at], ((unsigned long long)(uint32_t)w.b << 32) | (uint32_t)w.a);
  stc(&Q.tab[at], w.tab);
}

// A frontier queue being appended to.  Its counter holds the walk units and
// the edges appended so far in one word, so that one atomic gives a group of
// edges both its places in the queue and its stretch of the walks, in the same
// order.
struct QueueOut {
  FrontierQueue q;
  unsigned long long* count;  // (units << qbits) | edges
  int qbits, shift;
};

__device__ __forceinline__ unsigned long long walk_units(int len, int shift) {
  return ((unsigned long long)len + (1ULL << shift) - 1ULL) >> shift;
}

// Next-frontier edges are gathered per wavefront in LDS and appended to the
// global queue 64 or more at a time, so the queue counter sees one atomic per
// flush instead of one per wavefront iteration.  A flush looks up both
// endpoints' rows and appends the finished walk record, so that the next
// round starts from the records alone.
constexpr int kWq = 192;  // capacity: a flush happens before 64 + 2 * 64 entries are exceeded
struct WaveQueue {
  int* e;       // LDS, kWq entries each, private to the wavefront: edge and endpoints
  int* u;
  int* v;
  int cnt;      // wave-uniform fill level
};

__device__ __forceinline__ void wq_flush(const PeelArgs& P, WaveQueue& wq, const QueueOut& out) {
  if (wq.cnt == 0) return;
  wave_sync();
  const int lane = lane_id();
  for (int i0 = 0; i0 < wq.cnt; i0 += kWave) {
    const int i = i0 + lane;
    const bool in = i < wq.cnt;
    int32_t e = 0;
    Walk w = {0, 0, 0u, 0, 0ULL};
    if (in) {
      e = wq.e[i];
      w = walk_of(P, wq.u[i], wq.v[i]);
    }
    const unsigned long long units = in ? walk_units(w.len, out.shift) : 0ULL;
    const unsigned long long inc = wave_inclusive_sum(units);
    const int n = wq.cnt - i0 < kWave ? wq.cnt - i0 : kWave;
    unsigned long long at = 0;
    if (lane == kWave - 1) at = atomicAdd(out.count, (inc << out.qbits) | (unsigned)n);
    at = __shfl(at, kWave - 1, kWave);
    if (in)
      put_record(out.q, (int64_t)(at & ((1ULL << out.qbits) - 1ULL)) + lane,
                 (at >> out.qbits) + inc - units, e, w);
  }
  wq.cnt = 0;
  wave_sync();
}

// What the wavefronts of a workgroup still hold at the end of a round (fewer
// than kWave edges each), appended together with one atomic.  Same-address
// atomics are served one after another (about 17 ns each): with one per
// wavefront instead, the 4096 of a full grid held up a round of some 500 K
// entries by 30 us.  qe, qu, qv: all wavefronts' buffers; tmp: kWaves ints, tmp64:
// kWaves entries of LDS.
__device__ __forceinline__ void block_flush(const PeelArgs& P, const WaveQueue& wq, const int (*qe)[kWq],
                                            const int (*qu)[kWq], const int (*qv)[kWq], const QueueOut& out, int* tmp,
                                            unsigned long long* tmp64) {
  __shared__ unsigned long long s_at;
  const int tid = threadIdx.x, wv = tid / kWave;
  if (lane_id() == 0) tmp[wv] = wq.cnt;
  __syncthreads();
  int n = 0, src = 0, first = 0;
#pragma unroll 4
  for (int q = 0; q < kWaves; ++q) {
    const int c = tmp[q];
    if (tid >= n && tid < n + c) {
      src = q;
      first = n;
    }
    n += c;
  }
  if (n == 0) return;
  const bool in = tid < n;
  int32_t e = 0;
  Walk w = {0, 0, 0u, 0, 0ULL};
  if (in) {
    e = qe[src][tid - first];
    w = walk_of(P, qu[src][tid - first], qv[src][tid - first]);
  }
  const unsigned long long units = in ? walk_units(w.len, out.shift) : 0ULL;
  const unsigned long long inc = wave_inclusive_sum(units);
  if (lane_id() == kWave - 1) tmp64[wv] = inc;
  __syncthreads();
  unsigned long long base = 0, all = 0;
#pragma unroll 4
  for (int q = 0; q < kWaves; ++q) {
    const unsigned long long v = tmp64[q];
    if (q < wv) base += v;
    all += v;
  }
  if (tid == 0) s_at = atomicAdd(out.count, (all << out.qbits) | (unsigned)n);
  __syncthreads();
  const unsigned long long at = s_at;
  if (in)
    put_record(out.q, (int64_t)(at & ((1ULL << out.qbits) - 1ULL)) + tid, (at >> out.qbits) + base + inc - units, e, w);
}

__device__ __forceinline__ void wq_push(WaveQueue& wq, int32_t f, int32_t u, int32_t v) {
  const uint64_t m = ballot(f >= 0);
  if (f >= 0) {
    const int at = wq.cnt + rank_below(m);
    wq.e[at] = f;
    wq.u[at] = u;
    wq.v[at] = v;
  }
  wq.cnt += __popcll(m);
}

// Frontier edges of a list phase gathered in LDS; a flush appends their walk
// records, one atomic per kT of them.  Every thread of the workgroup calls
// flush().  tmp: kWaves entries of LDS.
struct StagedQueue {
  int* buf;   // LDS, kStageQ entries
  int* fill;  // LDS: entries held
  unsigned long long* tmp;
  QueueOut out;
};

__device__ __forceinline__ void staged_flush(const PeelArgs& P, StagedQueue& L) {
  __shared__ unsigned long long s_at;
  __syncthreads();
  const int n = *L.fill;
  if (n == 0) return;
  const int wv = threadIdx.x / kWave;
  for (int i0 = 0; i0 < n; i0 += kT) {
    const int i = i0 + (int)threadIdx.x;
    const bool in = i < n;
    int32_t e = 0;
    Walk w = {0, 0, 0u, 0, 0ULL};
    if (in) {
      e = L.buf[i];
      w = walk_of(P, P.eu[e], P.ev[e]);
    }
    const unsigned long long units = in ? walk_units(w.len, L.out.shift) : 0ULL;
    const unsigned long long inc = wave_inclusive_sum(units);
    if (lane_id() == kWave - 1) L.tmp[wv] = inc;
    __syncthreads();
    unsigned long long base = 0, all = 0;
#pragma unroll 4
    for (int q = 0; q < kWaves; ++q) {
      const unsigned long long v = L.tmp[q];
      if (q < wv) base += v;
      all += v;
    }
    if (threadIdx.x == 0) s_at = atomicAdd(L.out.count, (all << L.out.qbits) | (unsigned)(n - i0 < kT ? n - i0 : kT));
    __syncthreads();
    const unsigned long long at = s_at;
    if (in)
      put_record(L.out.q, (int64_t)(at & ((1ULL << L.out.qbits) - 1ULL)) + (int)threadIdx.x,
                 (at >> L.out.qbits) + base + inc - units, e, w);
    __syncthreads();
  }
  if (threadIdx.x == 0) *L.fill = 0;
  __syncthreads();
}

// minimum over the workgroup into *dst (one atomic per workgroup); tmp: kWaves ints
__device__ __forceinline__ void block_min_to(int x, int* tmp, int* dst) {
  x = wave_min(x);
  if (lane_id() == 0) tmp[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int v = kIntMax;
    for (int q = 0; q < kWaves; ++q) v = tmp[q] < v ? tmp[q] : v;
    if (v != kIntMax) atomicMin(dst, v);
  }
  __syncthreads();
}

// sum over the workgroup into *dst (one atomic per workgroup); tmp: kWaves entries
__device__ __forceinline__ void block_sum_to(unsigned long long x, unsigned long long* tmp,
                                             unsigned long long* dst) {
  x = wave_sum(x);
  if (lane_id() == 0) tmp[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long v = 0;
    for (int q = 0; q < kWaves; ++q) v += tmp[q];
    if (v) atomicAdd(dst, v);
  }
  __syncthreads();
}

// Block-wide inclusive prefix sum of one int per thread; total in *total; tmp: kWaves ints of LDS.
__device__ __forceinline__ int block_inclusive_sum(int x, int* tmp, int* total) {
  const int w = threadIdx.x / kWave;
  const int inc = wave_inclusive_sum(x);
  if (lane_id() == kWave - 1) tmp[w] = inc;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll 4
  for (int q = 0; q < kWaves; ++q) {
    const int v = tmp[q];
    if (q < w) base += v;
    all += v;
  }
  *total = all;
  __syncthreads();
  return base + inc;
}

// Number of threads of the workgroup with `p` set; tmp: kWaves ints of LDS.
__device__ __forceinline__ int block_count(bool p, int* tmp) {
  const uint64_t m = ballot(p);
  if (lane_id() == 0) tmp[threadIdx.x / kWave] = __popcll(m);
  __syncthreads();
  int n = 0;
  for (int q = 0; q < kWaves; ++q) n += tmp[q];
  __syncthreads();
  return n;
}

using KernArgs = const __attribute__((address_space(4))) PeelArgs*;

// The same for two conditions: (threads with q << 16) | threads with p (kT < 2^16).
__device__ __forceinline__ int block_count2(bool p, bool q, int* tmp) {
  const uint64_t mp = ballot(p), mq = ballot(q);
  if (lane_id() == 0) tmp[threadIdx.x / kWave] = (__popcll(mq) << 16) | __popcll(mp);
  __syncthreads();
  int n = 0;
#pragma unroll 4
  for (int i = 0; i < kWaves; ++i) n += tmp[i];
  __syncthreads();
  return n;
}

// NI: walk entries in flight per thread; SU: live-list entries per thread and
// step of the list phases
template <int NI, int SU, bool HALF>
__device__ __forceinline__ void peel_body() {
  static_assert(2 * SU * kT <= kStageQ, "a step's frontier fits beside the last one's");
  // the walking phase and the list phases use the same LDS
  struct RoundLds {
    WalkTabs W;
    int qe[kWaves][kWq], qu[kWaves][kWq], qv[kWaves][kWq];
  };
  struct ListLds {
    int q[kStageQ];
  };
  __shared__ union {
    RoundLds r;
    ListLds l;
  } S;
  __shared__ int s_tmp[kWaves + 2];
  __shared__ int s_part;
  __shared__ unsigned long long s_w64[kWaves];
  __shared__ int s_fill, s_list;
  KernArgs ka = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  PeelCtl* const c = ((const PeelArgs*)ka)->ctl;
  if (threadIdx.x == 0) s_fill = 0;
  __syncthreads();
  const int tid = threadIdx.x;
  const int wv = tid / kWave;
  const int qbits = ldc(&c->qbits);
  const int shift = walk_shift(((const PeelArgs*)ka)->head->wbound, ((const PeelArgs*)ka)->m, qbits);
  if (blockIdx.x == 0 && threadIdx.x == 0) stc(&c->sup_total, ((const PeelArgs*)ka)->head->sup_total);
  unsigned long long my_work = 0;  // entries walked by this wavefront

  __shared__ unsigned long long s_pub[kPub];
  // the state left by the previous launch (or k_peel_init)
  unsigned gen = ldc(&c->bar_gen);
  PhaseState st;
  st.phase = ldc(&c->phase);
  st.acur = ldc(&c->acur);
  st.mode = ldc(&c->mode);
  st.probe = ldc(&c->probe);
  st.first = ldc(&c->first);
  st.compact = ldc(&c->compact);
  st.qlen = 0;
  st.k = ldc(&c->k);
  st.r = ldc(&c->r);
  st.acnt = ldc(&c->acnt);
  st.units = 0;

  for (;;) {
    // the arguments are read anew in each phase: kept in scalar registers over
    // all phases they would spill, and take vector registers with them
    asm volatile("" : "+s"(ka));
    const PeelArgs& P = *(const PeelArgs*)ka;
    const int phase = st.phase;
    if (phase == PH_DONE || phase == PH_COMPACT) break;
    const int k = st.k;
    const int l = k - 2;
    const int r = st.r;
    const int acur = st.acur;
    PhaseCounts* const cw = &c->w[gen & 1];
    if (phase != PH_PROC) {
      // Sweep: the minimum live support, and at once the live edges with
      // sup <= k-1 as the frontier of level k+1 (the control step keeps them only
      // if that level is not skipped, in which case none is taken); with
      // compact set the live edges are also written as the new list.  Level start
      // after a skip, or dense re-scan: the live edges with sup <= k-2.
      const bool sweep = phase == PH_SWEEP;
      const int kt = sweep ? k + 1 : k;
      const int stamp = phase == PH_START ? r : r + 1;
      const bool ids = st.first != 0, write = sweep && st.compact != 0;
      const int64_t cnt = ids ? P.m : (int64_t)st.acnt;
      const int32_t* A = P.alist[acur];
      int32_t* const B = P.alist[acur ^ 1];
      StagedQueue LQ{S.l.q, &s_fill, s_w64, QueueOut{P.fq[stamp & 1], &cw->q, qbits, shift}};
      int mins = kIntMax;
      unsigned long long wsum = 0;  // shorter live row over the frontier
      // SU list entries a thread, their loads in flight together; the few that
      // are taken (or written to the new list) are read again afterwards, so
      // that only their bits are held.  What bounds a sweep is the lines of sup
      // that sparse lists touch; SU of 2, 4 and 8 measured 57.6, 67.5 and 77.1 ms
      // of sweeps on R-MAT 23 (the list written anew in every sweep, with stamps
      // read as well: 74.4), since larger steps leave workgroups idle on the
      // shorter lists.
      for (int64_t base = (int64_t)blockIdx.x * kT * SU; base < cnt; base += (int64_t)gridDim.x * kT * SU) {
        unsigned live = 0, taken = 0;
        {
          int32_t e[SU];
          int sv[SU];
#pragma unroll
          for (int u = 0; u < SU; ++u) {
            const int64_t i = base + u * kT + tid;
            e[u] = i < cnt ? (ids ? (int32_t)i : ldc(&A[i])) : -1;
          }
#pragma unroll
          for (int u = 0; u < SU; ++u) sv[u] = e[u] >= 0 ? ldc(&P.sup[e[u]]) : kGone;
#pragma unroll
          for (int u = 0; u < SU; ++u) {
            if (sv[u] < kGoneMin) {
              mins = sv[u] < mins ? sv[u] : mins;
              live |= 1u << u;
              if (sv[u] <= kt - 2) taken |= 1u << u;
            }
          }
        }
        if (ballot(taken != 0)) {
#pragma unroll 1
          for (int u = 0; u < SU; ++u) {
            const bool take = (taken >> u & 1u) != 0;
            const uint64_t m = ballot(take);
            if (m == 0) continue;
            int at = 0;
            if (lane_id() == 0) at = atomicAdd(&s_fill, __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            if (take) {
              const int64_t i = base + u * kT + tid;
              const int32_t e = ids ? (int32_t)i : ldc(&A[i]);
              S.l.q[at + rank_below(m)] = e;
              stc(&P.stamp[e], stamp);
              stc(&P.sup[e], kGone);
              P.truss[e] = kt;
              const int du = P.vinfo[P.eu[e]].len, dv = P.vinfo[P.ev[e]].len;
              wsum += (unsigned long long)(du < dv ? du : dv);
            }
          }
        }
        if (write) {
          int total;
          const int keep = __popc(live);
          const int inc = block_inclusive_sum(keep, s_tmp, &total);
          if (tid == 0) s_list = atomicAdd(&cw->alive, total);
          __syncthreads();
          int at = s_list + inc - keep;
#pragma unroll 1
          for (int u = 0; u < SU; ++u) {
            if (!(live >> u & 1u)) continue;
            const int64_t i = base + u * kT + tid;
            stc(&B[at++], ids ? (int32_t)i : ldc(&A[i]));
          }
        }
        __syncthreads();
        const int held = s_fill;
        __syncthreads();  // every thread has read it before the next append
        if (held > kStageQ - SU * kT) staged_flush(P, LQ);
      }
      staged_flush(P, LQ);
      if (sweep) block_min_to(mins, s_tmp, &cw->minsup);
      if (phase != PH_DENSE) block_sum_to(wsum, s_w64, &cw->fwork);
    } else if (phase == PH_PROC) {
      // The round's walks, laid end to end, in parts of equal length (see
      // kMinChunk): every workgroup finds the record its part starts in by a
      // search of the records' starts, kT probes at a time, stages the part's
      // records in LDS and walks its entries, a thread taking NI of them at
      // once.  Nothing is handed from one workgroup to another.
      const int qn = st.qlen;
      const unsigned long long units = st.units;
      const bool sparse = st.mode == TRUSS_PEEL_SPARSE;
      const int probe = st.probe;
      const FrontierQueue Q = P.fq[r & 1];
      const QueueOut out{P.fq[(r + 1) & 1], &cw->q, qbits, shift};
      WaveQueue wq{S.r.qe[wv], S.r.qu[wv], S.r.qv[wv], 0};
      WalkTabs& W = S.r.W;
      const int umask = (1 << shift) - 1;
      unsigned long long pu = (units + gridDim.x - 1) / gridDim.x;  // units a part
      if (pu < (unsigned long long)(kMinChunk >> shift)) pu = (unsigned long long)(kMinChunk >> shift);
      if (pu > (unsigned long long)(kPartMax >> shift)) pu = (unsigned long long)(kPartMax >> shift);
      if (pu < (units >> 30)) pu = units >> 30;  // the draw counter is an int
      if (pu < 1) pu = 1;
      const unsigned long long parts = (units + pu - 1) / pu;
      const bool drawn = parts > gridDim.x;  // more parts than workgroups: the later ones are drawn
      for (unsigned long long part = blockIdx.x; part < parts;) {
        // the next part is drawn early: its number is needed after this one's walk
        if (drawn && tid == 0) s_part = atomicAdd(&cw->fetch, 1);
        const unsigned long long lo = part * pu;
        const unsigned long long hi = lo + pu < units ? lo + pu : units;
        // x0: the last record that starts at or before unit lo.  A frontier of
        // up to kT records is read whole, and x0 found among the records read.
        int64_t x0 = 0;
        const bool whole = qn <= kT;
        for (int64_t span = lo > 0 && !whole ? qn : 1; span > 1;) {
          const int64_t sp = (span + kT - 1) / kT;
          const int64_t d = tid * sp;
          const int n = block_count(d < span && ldc(&Q.pre[x0 + d]) <= lo, s_tmp);
          x0 += (int64_t)(n - 1) * sp;
          span = span - (int64_t)(n - 1) * sp < sp ? span - (int64_t)(n - 1) * sp : sp;
        }
        for (;;) {
          // up to kT records from x0 on
          const int64_t x = x0 + tid;
          unsigned long long pre = ~0ULL, eb = 0, ab = 0, tab = 0, next = hi;
          if (x < qn) {
            pre = ldc(&Q.pre[x]);
            eb = ldc(&Q.eb[x]);
            ab = ldc(&Q.ab[x]);
            tab = ldc(&Q.tab[x]);
          }
          if (x0 + kT < qn) {
            next = ldc(&Q.pre[x0 + kT]);
            next = next < hi ? next : hi;
          }
          // records before x0 (whole only) and records in the part
          const int cnt2 = block_count2(whole && pre <= lo, pre < hi, s_tmp);
          const int skip = whole ? (cnt2 & 0xffff) - 1 : 0;
          const int nrec = (cnt2 >> 16) - skip;
          const int y0 = tid - skip;
          if (y0 >= 0 && pre < hi) {
            W.pre[y0] = (int)((long long)pre - (long long)lo);
            W.e[y0] = (int32_t)(uint32_t)eb;
            W.base[y0] = (uint32_t)(eb >> 32);
            W.a[y0] = (int32_t)(uint32_t)ab;
            W.b[y0] = (int32_t)(ab >> 32);
            W.tab[y0] = tab;
            if (shift > 0) W.len[y0] = P.vinfo[(uint32_t)ab].len;
          }
          __syncthreads();
          const int ub = W.pre[0] > 0 ? W.pre[0] : 0, ue = (int)(next - lo);
          int top = 1;
          while (2 * top < nrec) top <<= 1;
          const int hi_t = ue << shift;
          for (int t0 = ub << shift; t0 < hi_t; t0 += NI * kT) {
            int x_[NI];
            int32_t w[NI], f1[NI], f2[NI];
            uint32_t j[NI];
            bool ok[NI];
#pragma unroll
            for (int q = 0; q < NI; ++q) x_[q] = 0;
            // the record of each entry: the last whose walk starts at or before it
            for (int st = top; st > 0; st >>= 1) {
#pragma unroll
              for (int q = 0; q < NI; ++q) {
                const int y = x_[q] + st;
                if (y < nrec && W.pre[y] <= ((t0 + q * kT + tid) >> shift)) x_[q] = y;
              }
            }
#pragma unroll
            for (int q = 0; q < NI; ++q) {
              const int t = t0 + q * kT + tid;
              const int off = (((t >> shift) - W.pre[x_[q]]) << shift) + (t & umask);
              ok[q] = t < hi_t && (shift == 0 || off < W.len[x_[q]]);
              j[q] = W.base[x_[q]] + (uint32_t)off;
              my_work += __popcll(ballot(ok[q]));
            }
            process_entries<NI, HALF>(P, W, x_, j, ok, r, l, k, sparse, probe, w, f1, f2);
            if (sparse) {
#pragma unroll
              for (int q = 0; q < NI; ++q) {
                wq_push(wq, f1[q], W.a[x_[q]], w[q]);
                wq_push(wq, f2[q], W.b[x_[q]], w[q]);
                if (wq.cnt >= kWave) wq_flush(P, wq, out);
              }
            }
          }
          __syncthreads();
          x0 += kT;
          if (x0 >= qn || next >= hi) break;
        }
        if (!drawn) break;
        part = (unsigned long long)gridDim.x + (unsigned)s_part;
        __syncthreads();
      }
      if (sparse) block_flush(P, wq, S.r.qe, S.r.qu, S.r.qv, out, s_tmp, s_w64);
    }
    ++gen;
    if (!phase_barrier(c, P, st, gen, shift, s_pub)) break;
  }
  if (lane_id() == 0 && my_work) atomicAdd(&c->w_work, my_work);
}

// The persistent peeling kernel in two shapes over the same state machine:
// one 1024-thread workgroup per compute unit with two walk entries in flight
// per thread, or two workgroups per compute unit (registers capped for eight
// wavefronts per SIMD) with one entry per thread, which hides more latency
// when walks are long.  Entries per thread, measured: narrow 1 / 2 / 3 / 4: 13.2 / 13.3 /
// 13.8 / 14.3 ms on R-MAT of 1.2 M edges, 90.7 / 83.5 / 85.7 / 87.2 on 15.7 M; wide
// 1 / 2: 1173 / 1202 ms on R-MAT 23 (at 64 registers both spill, 40 and 52 bytes of scratch a
// lane).  Buckets read by halves / at once:
// narrow 86.4 / 83.8 ms on 15.7 M edges, wide 1173 / 1224 on R-MAT 23.  All state lives in global
// memory between launches.
__global__ void __launch_bounds__(kT) k_peel(PeelArgs) { peel_body<2, 2, false>(); }
__global__ void __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(8, 8))) k_peel_wide(PeelArgs) {
  peel_body<1, 2, true>();
}

// One bit per edge, set when the edge is removed: the liveness test of the
// row compaction reads this bitmap (m/8 bytes, cache-resident) instead of
// one scattered stamp per row entry.
__global__ void __launch_bounds__(256) k_dead_bits(const int32_t* __restrict__ stamp, int64_t m,
                                                   unsigned long long* __restrict__ dead) {
  const int lane = lane_id();
  const int64_t gw = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  for (int64_t base = gw * kWave; base < m; base += nw * kWave) {
    const int64_t e = base + lane;
    const unsigned long long bits = ballot(e < m && stamp[e] != 0);
    if (lane == 0) dead[base / kWave] = bits;
  }
}

// Stable in-place compaction of every row to its live entries (a wavefront a row).
constexpr int kCompactUnroll = 4;
__global__ void __launch_bounds__(256) k_compact(int32_t* __restrict__ col,
                                                 int32_t* __restrict__ seid, VInfo* __restrict__ vinfo, int32_t n,
                                                 const unsigned long long* __restrict__ dead, PeelCtl* c) {
  const int lane = lane_id();
  const int64_t gw = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  if (gw == 0 && lane == 0) {
    c->phase = PH_SWEEP;
    c->t_last = 0;
  }
  for (int64_t v = gw; v < n; v += nw) {
    const VInfo vi = vinfo[v];
    const int64_t rb = vi.base;
    const int len = vi.len;
    int wpos = 0;
    // kCompactUnroll chunks of kWave entries are read before any is written
    // back, so their loads overlap; entries only move to lower positions, so
    // the writes never reach an entry that has not been read
    for (int c0 = 0; c0 < len; c0 += kCompactUnroll * kWave) {
      int32_t x[kCompactUnroll], ed[kCompactUnroll];
      bool keep[kCompactUnroll];
#pragma unroll
      for (int u = 0; u < kCompactUnroll; ++u) {
        const int i = c0 + u * kWave + lane;
        x[u] = 0;
        ed[u] = 0;
        if (i < len) {
          x[u] = col[rb + i];
          ed[u] = seid[rb + i];
        }
      }
#pragma unroll
      for (int u = 0; u < kCompactUnroll; ++u) {
        const int i = c0 + u * kWave + lane;
        keep[u] = i < len && ((dead[ed[u] >> 6] >> (ed[u] & 63)) & 1ULL) == 0;
      }
#pragma unroll
      for (int u = 0; u < kCompactUnroll; ++u) {
        const uint64_t km = ballot(keep[u]);
        if (keep[u]) {
          const int64_t dst = rb + wpos + rank_below(km);
          col[dst] = x[u];
          seid[dst] = ed[u];
        }
        wpos += __popcll(km);
      }
    }
    if (lane == 0) vinfo[v].len = wpos;
  }
}

// The vertices' walk records and the control block.  head->wbound receives the sum
// of the shorter row over all edges: with the ids ranked by degree an edge's
// shorter row is that of its first endpoint in the orientation, so the sum is
// that of out-degree times degree.  head->sup_total receives the sum of the
// supports (sup nullable).
__global__ void __launch_bounds__(256) k_peel_init(PeelCtl* c, const int64_t* __restrict__ row_ptr,
                                                   const int64_t* __restrict__ orow, const int64_t* __restrict__ rtoff,
                                                   VInfo* __restrict__ vinfo, int32_t n, int64_t m,
                                                   long long max_subrounds, int sched, int fix_bits, int fix_vals,
                                                   int qbits, int first_level, int stop_level,
                                                   const int32_t* __restrict__ sup, RunHead* head) {
  __shared__ unsigned long long s_s[4];
  __shared__ unsigned long long s_w[4];
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  unsigned long long wsum = 0, ssum = 0;
  if (sup)
    for (int64_t e = i; e < m; e += (int64_t)gridDim.x * blockDim.x) ssum += (unsigned long long)sup[e];
  if (i < n) {
    const int64_t rb = row_ptr[i], d = row_ptr[i + 1] - rb;
    const int64_t to = rtoff[i], slots = rtoff[i + 1] - to;
    VInfo v;
    v.base = (uint32_t)rb;
    v.len = (int32_t)d;
    v.tab = ((unsigned long long)to << 6) | (unsigned)(slots > 0 ? row_table_lg(slots) : 0);
    vinfo[i] = v;
    wsum = (unsigned long long)(orow[i + 1] - orow[i]) * (unsigned long long)d;
  }
  wsum = wave_sum(wsum);
  ssum = wave_sum(ssum);
  if (lane_id() == 0) {
    s_w[threadIdx.x / kWave] = wsum;
    s_s[threadIdx.x / kWave] = ssum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long w = s_w[0] + s_w[1] + s_w[2] + s_w[3], t = s_s[0] + s_s[1] + s_s[2] + s_s[3];
    if (w) atomicAdd(&head->wbound, w);
    if (t) atomicAdd(&head->sup_total, t);
  }
  if (i == 0) {
    grid_barrier_init(&c->bar);
    c->bar_gen = 0;
    for (int i = 0; i < 2; ++i) {
      c->w[i].fetch = 0;
      c->w[i].q = 0ULL;
      c->w[i].alive = 0;
      c->w[i].minsup = kIntMax;
      c->w[i].fwork = 0ULL;
    }
    c->w_work = 0ULL;
    c->input_err = head->err;
    c->sup_total = 0ULL;
    c->phase = head->err == kNoErr ? PH_SWEEP : PH_DONE;
    c->k = first_level - 1;  // the first sweep takes the frontier of level first_level
    c->r = 0;
    c->qlen = 0;
    c->qunits = 0ULL;
    c->acnt = (int)m;
    c->acur = 0;
    c->first = 1;
    c->compact = 0;
    c->mode = TRUSS_PEEL_SPARSE;
    c->kmax = 0;
    c->levels = 0;
    c->removed_level = 0;
    c->removed = 0;
    c->csr_live = m;
    c->subrounds = 0;
    c->heavy_rounds = 0;
    c->max_subrounds = max_subrounds;
    for (int b = 0; b < kHistBins; ++b) c->hist[b] = 0;
    c->t_last = 0;
    for (int b = 0; b < 8; ++b) c->t_phase[b] = 0;
    c->err = 0;
    c->probe = 0;
    c->sched = sched;
    c->fix_bits = fix_bits;
    c->fix_vals = fix_vals;
    c->stop_level = stop_level;
    c->qbits = qbits;
    c->lvl_sub0 = 0;
    c->prev_sub = 0;
    c->t_dec = 0;
  }
}

// truss numbers in the caller's order (nothing for an invalid input or a peeling
// that did not come to its end)
__global__ void __launch_bounds__(256) k_peel_out(const int32_t* __restrict__ truss, const int32_t* __restrict__ perm,
                                                  int64_t m, int32_t* __restrict__ out, const PeelCtl* c) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool done = c->input_err == kNoErr && c->err == 0 && c->bar.abort == 0 && c->phase == PH_DONE;
  if (e < m && done) out[perm[e]] = truss[e];
}

struct PeelLayout {
  PeelCtl* ctl;
  VInfo* vinfo;
  int32_t* alist[2];
  FrontierQueue fq[2];
  unsigned long long* dead;  // removed-edge bitmap for the row compaction
};

void carve(int64_t m, Arena& a, PeelLayout& L) {
  L.ctl = a.take<PeelCtl>(1);
  for (int i = 0; i < 2; ++i) L.alist[i] = a.take<int32_t>(m + 1);
}

// what lies in the build's temporaries
void carve_records(int32_t n, int64_t m, Arena& t, PeelLayout& L) {
  L.vinfo = t.take<VInfo>((size_t)n + 1);
  for (int i = 0; i < 2; ++i) {
    L.fq[i].pre = t.take<unsigned long long>((size_t)m + 1);
    L.fq[i].eb = t.take<unsigned long long>((size_t)m + 1);
    L.fq[i].ab = t.take<unsigned long long>((size_t)m + 1);
    L.fq[i].tab = t.take<unsigned long long>((size_t)m + 1);
  }
  L.dead = t.take<unsigned long long>((size_t)(m / kWave + 2));
}

// Small graphs take one workgroup per kGridEdges edges, at least kGridMin: fewer start
// (each fetches the code anew) and meet at the barriers.  Whole calls, 256 workgroups /
// this rule: 20 K edges 0.357 -> 0.323 ms, 40 K 0.406 -> 0.375, 110 K 0.496 -> 0.481; with 128
// workgroups R-MAT of 1.2 M edges takes 15.6 ms instead of 14.8, with 16 G(2000, 0.01)
// 0.394 instead of 0.326.
constexpr int64_t kGridEdges = 512;
constexpr int kGridMin = 64;

int g_peel_blocks = 0;       // grid of k_peel: one workgroup per compute unit
int g_peel_wide_blocks = -1;  // grid of k_peel_wide (two per compute unit), 0 if it does not fit

// TRUSS_SHAPE_AUTO takes the wide shape from this many edges on: there its
// extra wavefronts hide the latency of long walks in every launch, while on
// smaller graphs the shorter rounds favour the narrow shape (fewer workgroups
// at each barrier, more entries in flight per thread; 1173 against 1470 ms on
// R-MAT 23, 161 M edges).
constexpr long long kWideMinEdges = 1LL << 27;

}  // namespace

size_t peel_workspace(const DevGraph& dg, Arena& a) {
  PeelLayout L;
  carve(dg.m, a, L);
  return a.used;
}

size_t peel_record_bytes(int32_t n, int64_t m) {
  PeelLayout L;
  Arena t;
  t.counting = true;
  carve_records(n, m, t, L);
  return t.used;
}

int peel(const DevGraph& dg, const PeelPlan& plan, int32_t* sup, int32_t* stamp, int32_t* truss_canon, Arena& a, PeelResult* res,
         hipStream_t s, truss_trace* trace) {
  PeelLayout L;
  carve(dg.m, a, L);
  Arena t;
  t.base = static_cast<char*>(dg.tmp);
  t.cap = dg.tmp_bytes;
  carve_records(dg.n, dg.m, t, L);
  if (a.overflow() || t.overflow()) return TRUSS_E_WORKSPACE;
  *res = PeelResult();
  if (dg.m == 0) return TRUSS_OK;
  const long long maxsr = plan.max_subrounds;
  int qbits = 1;
  while ((dg.m >> qbits) != 0) ++qbits;  // a frontier holds up to m edges
  // a thread a vertex; with the sum of the supports at least up to 1024 workgroups
  int64_t init = ((int64_t)(dg.n > 0 ? dg.n : 1) + 255) / 256;
  const int64_t for_sum = (dg.m + 255) / 256 < 1024 ? (dg.m + 255) / 256 : 1024;
  if (plan.sum && init < for_sum) init = for_sum;
  hipLaunchKernelGGL(k_peel_init, dim3((unsigned)init), dim3(256), 0, s,
                     L.ctl, dg.row_ptr, dg.orow, dg.rtoff, L.vinfo, dg.n, dg.m, maxsr, plan.sched, plan.fix_bits,
                     plan.fix_vals, qbits, plan.first_level < 2 ? 2 : plan.first_level, plan.stop_level,
                     plan.sum ? sup : nullptr, plan.head);
  if (g_peel_blocks == 0) {
    int dev = 0, cus = 0, occ = 0;
    TRUSS_HIP(hipGetDevice(&dev));
    TRUSS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    TRUSS_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void*)k_peel, kT, 0));
    if (occ < 1) {
      set_last_error("peeling kernel does not fit on a compute unit");
      return TRUSS_E_DEVICE;
    }
    g_peel_blocks = cus;
    int occw = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occw, (const void*)k_peel_wide, kT, 0) != hipSuccess) occw = 0;
    g_peel_wide_blocks = occw >= 2 ? 2 * cus : 0;
  }
  int blocks = g_peel_blocks;
  if (plan.grid_blocks > 0) {
    if (plan.grid_blocks < blocks) blocks = plan.grid_blocks;
  } else {
    const int64_t few = dg.m / kGridEdges < kGridMin ? kGridMin : dg.m / kGridEdges;
    if (few < blocks) blocks = (int)few;
  }
  // a caller-fixed grid keeps the narrow shape
  const bool wide = plan.grid_blocks <= 0 && g_peel_wide_blocks > 0 &&
                    (plan.shape == TRUSS_SHAPE_WIDE || (plan.shape == TRUSS_SHAPE_AUTO && dg.m >= kWideMinEdges));
  PeelArgs P;
  P.n = dg.n;
  P.m = dg.m;
  P.col = dg.col;
  P.seid = dg.seid;
  P.vinfo = L.vinfo;
  P.eu = dg.eu;
  P.ev = dg.ev;
  P.sup = sup;
  P.stamp = stamp;
  P.truss = truss_canon;
  for (int i = 0; i < 2; ++i) {
    P.alist[i] = L.alist[i];
    P.fq[i] = L.fq[i];
  }
  P.rtab = dg.rtab;
  P.ctl = L.ctl;
  P.head = plan.head;
  P.model = plan.sched == TRUSS_SCHED_LEARNED ? plan.model : nullptr;
  P.tr_cap = trace && trace->level_feat && trace->level_ms && trace->level_action ? trace->level_cap : 0;
  P.tr_feat = P.tr_cap > 0 ? trace->level_feat : nullptr;
  P.tr_ms = P.tr_cap > 0 ? trace->level_ms : nullptr;
  P.tr_act = P.tr_cap > 0 ? trace->level_action : nullptr;
  PeelCtl h;
  // below kCompactMin edges the kernel never returns for a compaction, so the
  // output can follow it without asking (k_peel_out looks at how it ended)
  const bool once = dg.m < kCompactMin;
  auto output = [&]() {
    hipLaunchKernelGGL(k_peel_out, dim3((unsigned)((dg.m + 255) / 256)), dim3(256), 0, s, truss_canon, plan.perm, dg.m,
                       plan.out, L.ctl);
    if (plan.done) (void)hipEventRecord(plan.done, s);
  };
  int launches = 0;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  const bool timed = plan.timed && hipEventCreate(&ev0) == hipSuccess && hipEventCreate(&ev1) == hipSuccess;
  double kernel_ms = 0.0;
  for (;;) {
    if (timed) (void)hipEventRecord(ev0, s);
    if (wide)
      hipLaunchKernelGGL(k_peel_wide, dim3(g_peel_wide_blocks), dim3(kT), 0, s, P);
    else
      hipLaunchKernelGGL(k_peel, dim3(blocks), dim3(kT), 0, s, P);
    TRUSS_HIP(hipGetLastError());
    if (timed) (void)hipEventRecord(ev1, s);
    ++launches;
    if (once) output();
    TRUSS_HIP(hipMemcpyAsync(&h, L.ctl, sizeof(PeelCtl), hipMemcpyDeviceToHost, s));
    TRUSS_HIP(hipStreamSynchronize(s));
    if (timed) {
      float t = 0.f;
      if (hipEventElapsedTime(&t, ev0, ev1) == hipSuccess) kernel_ms += t;
    }
    if (h.bar.abort || h.err || h.phase != PH_COMPACT) break;
    hipLaunchKernelGGL(k_dead_bits, dim3(4096), dim3(256), 0, s, stamp, dg.m, L.dead);
    hipLaunchKernelGGL(k_compact, dim3(2048), dim3(256), 0, s, dg.col, dg.seid, L.vinfo, dg.n, L.dead, L.ctl);
  }
  if (ev0) (void)hipEventDestroy(ev0);
  if (ev1) (void)hipEventDestroy(ev1);
  if (h.input_err != kNoErr) return input_error(h.input_err);
  if (!once) {
    output();
    TRUSS_HIP(hipStreamSynchronize(s));
  }
  TRUSS_HIP(hipGetLastError());
  res->sup_total = h.sup_total;
  res->kernel_ms = kernel_ms;
  if (trace) trace->levels = h.levels < P.tr_cap ? h.levels : P.tr_cap;
  res->kmax = h.kmax;
  res->levels = h.levels;
  res->subrounds = h.subrounds;
  res->work = (int64_t)h.w_work;
  res->launches = launches;
  res->heavy_rounds = h.heavy_rounds;
  for (int b = 0; b < kHistBins; ++b) res->hist[b] = h.hist[b];
  for (int b = 0; b < 6; ++b) res->phase_ms[b] = (double)h.t_phase[b] * 1e-5;
  if (h.bar.abort) {
    set_last_error("peeling kernel barrier timed out");
    return TRUSS_E_INTERNAL;
  }
  if (h.err) {
    set_last_error("peeling exceeded the sub-round cap (%lld)", (long long)h.max_subrounds);
    return h.err;
  }
  if (h.phase != PH_DONE) {
    set_last_error("peeling stopped in phase %d", h.phase);
    return TRUSS_E_INTERNAL;
  }
  return TRUSS_OK;
}

}  // namespace truss
