// Core numbers (the c-core is the largest subgraph with minimum degree >= c)
// and the per-vertex sums behind the cohesion statistics of Section 7
// (Table 6: the k_max-truss against the c_max-core).
//
// Core numbers peel vertices level by level, like the edges of Algorithm 2:
// level c takes every live vertex of degree <= c (core number c), and removing
// a taken vertex lowers the degree of each of its neighbours by one; a live
// neighbour whose degree falls from c+1 to c is taken in the same level.  The
// order of the removals inside a level does not matter, so a taken vertex may be
// processed at any time: vertices are claimed by a compare-and-swap of their
// core number, the level start and the decrements race for them freely, and a
// workgroup goes on with the vertices it has claimed itself, from LDS, until it
// has walked kBudget entries; only then does it hand the rest to the grid through
// a queue.  An empty level jumps to the smallest live degree.
//
// All levels run in one persistent kernel, one workgroup per compute unit: what
// bounds it is the number of grid barriers (about 5 us each) and the chain of
// dependent accesses of a level.  R-MAT 20 (c_max 611): 832 kernel launches with a
// fence in every workgroup took 30 ms, this one kernel 5.5.
//
// Its barriers need every workgroup resident, which the device alone can not
// promise: beside another persistent kernel (a second call of this one, a
// peeling) on another stream or of another process, each could hold part of the
// compute units and wait for the rest.  So the grid agrees, before its first
// barrier, on whether all of it is there within kAdmitTicks; if not, it ends,
// and the levels are stepped by ordinary launches, which finish beside anything.
#include "common.hpp"
#include "internal.hpp"

namespace truss {

namespace {

constexpr int kT = 256;
constexpr int kIntMax = 0x7fffffff;

constexpr int kCoreT = 1024;
constexpr int kCoreWaves = kCoreT / kWave;
constexpr int kCoreNI = 4;         // row entries in flight per thread
constexpr int kCoreList = 4096;    // claimed vertices held in LDS
// A workgroup walks the vertices it has claimed itself until they come to kBudget row
// entries in a phase, and no list of more than kListMax: it would take longer than a
// grid barrier and the queue (kListMax 16384: a graph of 2000 vertices 0.305 -> 0.312 ms,
// the call on a ring of 1 M vertices of degree 10 3 % slower).
constexpr int kBudget = 16384;
constexpr int kListMax = 65536;

enum CorePhase : int { kLevel = 0, kRound = 1, kDone = 2 };
enum CorePub : int { kPubFlags = 0, kPubLevel = 1, kPubHead = 2, kPubTail = 3, kPubCnt = 4, kCorePub = 5 };

enum CoreAdmit : int { kUndecided = 0, kAdmitted = 1, kRefused = 2 };
// Longest wait for the rest of the grid, in ticks of the 100 MHz clock (0.5 ms).
constexpr unsigned long long kAdmitTicks = 50000;

struct CoreCounts {  // one phase's counters, by arrival group (a line each) where many workgroups add
  alignas(128) int minv[kGridGroups][32];   // smallest degree of a live vertex left
  alignas(128) int taken[kGridGroups][32];  // vertices claimed
  alignas(128) int list;                    // entries of the compacted live list
};

struct alignas(256) CoreCtl {
  GridBarrier bar;
  CoreCounts w[2];
  alignas(128) int tail;  // entries of the queue; a vertex enters it at most once
  alignas(128) int dead;  // vertices claimed so far
  int cmax;
  int phase;
  int admit;  // CoreAdmit, changed once
  alignas(128) unsigned arrived[kGridGroups][32];  // workgroups that have started, per group (a line each)
  alignas(128) unsigned groups;                    // groups all of whose workgroups have
};

// The stepped form: a sequence of identical launches of one kernel; the state says
// what a step does.  The last workgroup to finish a step decides the next one, so
// launches follow each other without a host round trip; the host checks for
// the end every kStepsPerCheck launches.
enum StepPhase : int { kStart = 0, kTake = 1, kEnd = 2 };

struct CoreState {
  int phase;  // kStart: take live vertices of degree <= level; kTake: remove the queue's vertices
  int level;
  int cur;    // queue holding the current frontier
  int qn;     // its length (kTake)
  int cmax;
  // counters of the running step, cleared by the workgroup that decides
  int next;   // vertices appended by this step
  int alive;  // kStart: live vertices left
  int minv;   // kStart: their smallest degree
  unsigned arrived;
};

constexpr unsigned kStepBlocks = 1024;
constexpr int kStepsPerCheck = 16;

struct CoreArgs {
  const int64_t* row_ptr;
  const int32_t* col;
  int32_t* deg;
  int32_t* core;
  int32_t n;
  int32_t* queue;    // n
  int32_t* list[2];  // live lists of n entries, or null: every level looks at all vertices
  CoreCtl* ctl;
};

inline unsigned blocks(int64_t n) {
  const int64_t b = (n + kT - 1) / kT;
  return (unsigned)(b < 1 ? 1 : b);
}

__global__ void k_core_init(const int64_t* __restrict__ row_ptr, int32_t n, int32_t* __restrict__ deg,
                            int32_t* __restrict__ core, CoreCtl* c, CoreState* st) {
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v < n) {
    deg[v] = (int32_t)(row_ptr[v + 1] - row_ptr[v]);
    core[v] = -1;
  }
  if (v == 0) {
    grid_barrier_init(&c->bar);
    for (int i = 0; i < 2; ++i) {
      for (int g = 0; g < kGridGroups; ++g) {
        c->w[i].minv[g][0] = kIntMax;
        c->w[i].taken[g][0] = 0;
      }
      c->w[i].list = 0;
    }
    c->tail = 0;
    c->dead = 0;
    c->cmax = 0;
    c->phase = kLevel;
    c->admit = kUndecided;
    for (int g = 0; g < kGridGroups; ++g) c->arrived[g][0] = 0;
    c->groups = 0;
    *st = CoreState{kStart, 0, 0, 0, 0, 0, 0, kIntMax, 0u};
  }
}

// Whether the whole grid is resident, the same answer for every workgroup: the last
// one to arrive says yes, one that has waited too long says no, and the first to
// change the word decides.  A workgroup arrives as it starts (core_arrive, one
// thread) and asks after its first phase, when the others have long arrived: asked at
// once, the answer took 8 us.
__device__ __forceinline__ void core_arrive(CoreCtl* c) {
  const unsigned g = blockIdx.x % kGridGroups, size = (gridDim.x - g + kGridGroups - 1) / kGridGroups;
  const unsigned ngroups = gridDim.x < (unsigned)kGridGroups ? gridDim.x : (unsigned)kGridGroups;
  if (atomicAdd(&c->arrived[g][0], 1u) + 1 == size && atomicAdd(&c->groups, 1u) + 1 == ngroups)
    atomicCAS(&c->admit, kUndecided, kAdmitted);
}
__device__ __forceinline__ bool core_admitted(CoreCtl* c) {
  __shared__ int s_yes;
  if (threadIdx.x == 0) {
    const uint64_t t0 = wall_clock64();
    while (ldc(&c->admit) == kUndecided) {
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > kAdmitTicks) atomicCAS(&c->admit, kUndecided, kRefused);
    }
    s_yes = ldc(&c->admit) == kAdmitted ? 1 : 0;
  }
  __syncthreads();
  return s_yes != 0;
}

// A workgroup's claimed vertices (LDS): one list being walked, one being filled.
struct CoreLds {
  int list[2][kCoreList];
  int cnt[2];
  uint32_t pre[kCoreT];
  uint32_t base[kCoreT];
  int tmp[kCoreWaves];
  int at;
  unsigned long long pub[kCorePub];
};

__device__ __forceinline__ bool claim(int32_t* core, int level) { return atomicCAS(core, -1, level) == -1; }

// v (if want) into the list being filled, into the queue when that is full
__device__ __forceinline__ void core_push(const CoreArgs& P, CoreLds& L, int to, bool want, int32_t v) {
  const uint64_t m = ballot(want);
  if (m == 0) return;
  const int leader = __builtin_ctzll(m), n = __popcll(m);
  int at = 0;
  if (lane_id() == leader) at = atomicAdd(&L.cnt[to], n);
  at = __shfl(at, leader, kWave) + rank_below(m);
  const bool over = want && at >= kCoreList;
  if (want && !over) L.list[to][at] = v;
  const uint64_t mo = ballot(over);
  if (mo) {
    const int lo = __builtin_ctzll(mo);
    int q = 0;
    if (lane_id() == lo) q = atomicAdd(&P.ctl->tail, __popcll(mo));
    q = __shfl(q, lo, kWave) + rank_below(mo);
    if (over) stc(&P.queue[q], v);
  }
}

// Walks the rows of the vertices in list `from` (cnt of them) and claims into the
// other list, up to the kCoreT vertices whose rows would pass `room` entries (kIntMax:
// all).  Returns the row entries walked; done: the vertices walked.
__device__ __forceinline__ int core_walk(const CoreArgs& P, CoreLds& L, int from, int cnt, int level, int room,
                                         int& done, int& taken) {
  const int tid = threadIdx.x, wv = tid / kWave;
  int total = 0;
  done = 0;
  for (int c0 = 0; c0 < cnt; c0 += kCoreT) {
    int len = 0;
    uint32_t base = 0;
    if (c0 + tid < cnt) {
      const int32_t v = L.list[from][c0 + tid];
      const int64_t rb = P.row_ptr[v];
      base = (uint32_t)rb;  // 2m < 2^32
      len = (int)(P.row_ptr[v + 1] - rb);
    }
    const int n = cnt - c0 < kCoreT ? cnt - c0 : kCoreT;
    // distinct rows of fewer than 2^32 entries in all: 32-bit sums suffice
    const uint32_t inc = wave_inclusive_sum((uint32_t)len);
    __syncthreads();
    if (lane_id() == kWave - 1) L.tmp[wv] = (int)inc;
    __syncthreads();
    uint32_t off = 0, W = 0;
#pragma unroll 4
    for (int q = 0; q < kCoreWaves; ++q) {
      if (q < wv) off += (uint32_t)L.tmp[q];
      W += (uint32_t)L.tmp[q];
    }
    if (room != kIntMax && W > (uint32_t)(room - total)) break;
    done = c0 + n;
    L.pre[tid] = off + inc - (uint32_t)len;
    L.base[tid] = base;
    __syncthreads();
    int top = 1;
    while (2 * top < n) top <<= 1;
    for (int64_t t0 = 0; t0 < W; t0 += kCoreNI * kCoreT) {
      int x[kCoreNI], u[kCoreNI], k[kCoreNI];
      bool ok[kCoreNI];
#pragma unroll
      for (int q = 0; q < kCoreNI; ++q) x[q] = 0;
      for (int st = top; st > 0; st >>= 1) {
#pragma unroll
        for (int q = 0; q < kCoreNI; ++q) {
          const int y = x[q] + st;
          if (y < n && L.pre[y] <= t0 + q * kCoreT + tid) x[q] = y;
        }
      }
#pragma unroll
      for (int q = 0; q < kCoreNI; ++q) {
        const int64_t t = t0 + q * kCoreT + tid;
        ok[q] = t < W;
        u[q] = ok[q] ? P.col[L.base[x[q]] + ((uint32_t)t - L.pre[x[q]])] : 0;
      }
#pragma unroll
      for (int q = 0; q < kCoreNI; ++q) k[q] = ok[q] ? ldc(&P.core[u[q]]) : 0;
#pragma unroll
      for (int q = 0; q < kCoreNI; ++q) {
        ok[q] = ok[q] && k[q] < 0;
        k[q] = ok[q] ? atomicSub(&P.deg[u[q]], 1) : 0;
      }
#pragma unroll
      for (int q = 0; q < kCoreNI; ++q) {
        const bool got = ok[q] && k[q] == level + 1 && claim(&P.core[u[q]], level);
        taken += __popcll(ballot(got));
        core_push(P, L, from ^ 1, got, u[q]);
      }
    }
    total = W < (uint32_t)(kIntMax - total) ? total + (int)W : kIntMax;
    __syncthreads();
  }
  return total;
}

// Walks list 0 and then, in turn, what has been claimed meanwhile, within kBudget
// and kListMax; hands the rest to the queue.  must: list 0 is walked whatever its
// length (it comes from the queue, cut into equal shares, or is full, and then the
// other workgroups' are, too).  Otherwise a level start's list is cut like the
// others: where one level takes a whole dense graph, two workgroups would walk all
// its rows (K_2000: the call 2.4 ms, handed over 0.29).  Every thread of the workgroup calls it; both lists are empty on return.
__device__ __forceinline__ void core_drain(const CoreArgs& P, CoreLds& L, int level, bool must, int& spent,
                                           int& taken) {
  int from = 0;
  bool first = true;
  for (;;) {
    __syncthreads();
    const int cnt = L.cnt[from] < kCoreList ? L.cnt[from] : kCoreList;
    __syncthreads();
    if (cnt == 0) break;
    if (threadIdx.x == 0) L.cnt[from ^ 1] = 0;
    __syncthreads();
    const int room = first && must ? kIntMax : spent < kBudget ? kListMax : 0;
    int done;
    const int w = core_walk(P, L, from, cnt, level, room, done, taken);
    if (done < cnt) {
      if (threadIdx.x == 0) L.at = atomicAdd(&P.ctl->tail, cnt - done);
      __syncthreads();
      for (int i = done + threadIdx.x; i < cnt; i += kCoreT) stc(&P.queue[L.at + i - done], L.list[from][i]);
      __syncthreads();
    }
    if (!first) spent += w;
    first = false;
    if (threadIdx.x == 0) L.cnt[from] = 0;
    from ^= 1;
  }
  if (threadIdx.x == 0) L.cnt[0] = L.cnt[1] = 0;
  __syncthreads();
}

__global__ void __launch_bounds__(kCoreT) k_core(CoreArgs P) {
  __shared__ CoreLds L;
  CoreCtl* const c = P.ctl;
  const int tid = threadIdx.x, lane = lane_id();
  if (tid == 0) core_arrive(c);
  const unsigned g = blockIdx.x % kGridGroups;
  if (tid < 2) L.cnt[tid] = 0;
  __syncthreads();
  int phase = kLevel, level = 0, head = 0, tail = 0;
  int cnt = P.n;         // entries of the live list
  int cur = 0;           // which list
  bool ids = true;       // the list is 0..n-1
  bool compact = false;  // write the next list in this level
  for (unsigned gen = 1;; ++gen) {
    CoreCounts* const w = &c->w[(gen - 1) & 1];
    int taken = 0, spent = 0, mins = kIntMax;
    if (phase == kLevel) {
      for (int64_t i0 = (int64_t)blockIdx.x * kCoreT; i0 < cnt; i0 += (int64_t)gridDim.x * kCoreT) {
        const int64_t i = i0 + tid;
        int32_t v = 0;
        bool keep = false, got = false;
        if (i < cnt) {
          v = ids ? (int32_t)i : ldc(&P.list[cur][i]);
          const int k = ldc(&P.core[v]), d = ldc(&P.deg[v]);
          if (k < 0) {
            if (d <= level) {
              got = claim(&P.core[v], level);
            } else {
              keep = true;
              mins = d < mins ? d : mins;
            }
          }
        }
        taken += __popcll(ballot(got));
        core_push(P, L, 0, got, v);
        if (compact) {
          const uint64_t m = ballot(keep);
          if (lane == 0) L.tmp[tid / kWave] = __popcll(m);
          __syncthreads();
          int before = 0, all = 0;
#pragma unroll 4
          for (int q = 0; q < kCoreWaves; ++q) {
            if (q < tid / kWave) before += L.tmp[q];
            all += L.tmp[q];
          }
          if (tid == 0 && all) L.at = atomicAdd(&w->list, all);
          __syncthreads();
          if (keep) stc(&P.list[cur ^ 1][L.at + before + rank_below(m)], v);
        }
        __syncthreads();
        const int held = L.cnt[0];
        __syncthreads();  // every thread has read it before the next append
        if (held > kCoreList - kCoreT) core_drain(P, L, level, true, spent, taken);
      }
      core_drain(P, L, level, false, spent, taken);
    } else {
      // the queue's vertices [head, tail), spread over the workgroups
      const int per = (tail - head + (int)gridDim.x - 1) / (int)gridDim.x;
      const int64_t q0 = (int64_t)head + (int64_t)blockIdx.x * per;
      const int64_t q1 = q0 + per < tail ? q0 + per : tail;
      for (int64_t i0 = q0; i0 < q1; i0 += kCoreList) {
        const int n = (int)(q1 - i0 < kCoreList ? q1 - i0 : kCoreList);
        for (int i = tid; i < n; i += kCoreT) L.list[0][i] = ldc(&P.queue[i0 + i]);
        if (tid == 0) L.cnt[0] = n;
        core_drain(P, L, level, true, spent, taken);
      }
    }
    // smallest live degree seen, vertices claimed (taken is the same in a wavefront's lanes)
    mins = wave_min(mins);
    if (lane == 0) L.tmp[tid / kWave] = mins;
    __syncthreads();
    if (tid == 0) {
      for (int q = 1; q < kCoreWaves; ++q) mins = L.tmp[q] < mins ? L.tmp[q] : mins;
      if (mins != kIntMax) atomicMin(&w->minv[g][0], mins);
    }
    __syncthreads();
    if (lane == 0) L.tmp[tid / kWave] = taken;
    __syncthreads();
    if (tid == 0) {
      for (int q = 1; q < kCoreWaves; ++q) taken += L.tmp[q];
      if (taken) atomicAdd(&w->taken[g][0], taken);
    }
    if (gen == 1 && !core_admitted(c)) return;
    const bool ok = grid_barrier<kCorePub>(&c->bar, gen, L.pub, [&](auto release) {
      const int q = lane < kGridGroups ? lane : 0;
      const int mv = ldc(&w->minv[q][0]), tk = lane < kGridGroups ? ldc(&w->taken[q][0]) : 0;
      const int tl = ldc(&c->tail), ll = ldc(&w->list);
      int dead = ldc(&c->dead), cmax = ldc(&c->cmax);
      const int m_all = wave_min(mv), t_all = wave_sum(tk);
      dead += t_all;
      if (t_all > 0) cmax = level;
      int ncnt = cnt, ncur = cur, nids = ids ? 1 : 0, nphase = phase, nlevel = level;
      if (phase == kLevel && compact) {
        ncnt = ll;
        ncur = cur ^ 1;
        nids = 0;
      }
      if (tl > tail) {
        nphase = kRound;
      } else if (phase == kLevel && t_all == 0) {
        // nothing left the graph in this level: the smallest live degree is exact
        nlevel = m_all;
        if (m_all == kIntMax) nphase = kDone;
      } else {
        nphase = kLevel;
        nlevel = level + 1;
      }
      // a new list once a fifth of this one is dead
      const bool comp = P.list[0] != nullptr && (long long)(P.n - dead) * 5 < (long long)ncnt * 4;
      unsigned long long word = (unsigned)ncnt;
      if (lane == kPubFlags) word = (unsigned)(nphase | (ncur << 2) | (nids << 3) | ((comp ? 1 : 0) << 4));
      if (lane == kPubLevel) word = (unsigned)nlevel;
      if (lane == kPubHead) word = (unsigned)tail;
      if (lane == kPubTail) word = (unsigned)tl;
      release(word);
      if (lane < kGridGroups) {
        stc(&w->minv[lane][0], kIntMax);
        stc(&w->taken[lane][0], 0);
      }
      if (lane == 0) {
        stc(&w->list, 0);
        stc(&c->dead, dead);
        stc(&c->cmax, cmax);
        stc(&c->phase, nphase);
      }
    });
    if (!ok) break;
    const unsigned f = (unsigned)scalar64(L.pub[kPubFlags]);
    phase = (int)(f & 3u);
    cur = (int)(f >> 2) & 1;
    ids = ((f >> 3) & 1u) != 0;
    compact = ((f >> 4) & 1u) != 0;
    level = (int)scalar64(L.pub[kPubLevel]);
    head = (int)scalar64(L.pub[kPubHead]);
    tail = (int)scalar64(L.pub[kPubTail]);
    cnt = (int)scalar64(L.pub[kPubCnt]);
    if (phase == kDone) break;
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kT) k_core_step(const int64_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ col, int32_t* __restrict__ deg,
                                                  int32_t* __restrict__ core, int32_t n, int32_t* __restrict__ q0,
                                                  int32_t* __restrict__ q1, CoreState* st) {
  __shared__ int s_min[kT / kWave], s_cnt[kT / kWave];
  __shared__ int s_last;
  const int phase = st->phase;  // written by an earlier launch
  if (phase == kEnd) return;
  const int level = st->level, cur = st->cur;
  int32_t* qc = cur ? q1 : q0;
  int32_t* qx = cur ? q0 : q1;
  const int lane = lane_id();
  if (phase == kStart) {
    // live vertices of degree <= level are taken (core number = level)
    int dmin = kIntMax, alive = 0;
    for (int64_t v0 = (int64_t)blockIdx.x * kT; v0 < n; v0 += (int64_t)gridDim.x * kT) {
      const int64_t v = v0 + threadIdx.x;
      bool take = false;
      if (v < n && core[v] < 0) {
        const int d = deg[v];
        if (d <= level) {
          take = true;
          core[v] = level;
        } else {
          dmin = d < dmin ? d : dmin;
          alive += 1;
        }
      }
      const int pos = wave_append(&st->next, take);
      if (take) qc[pos] = (int32_t)v;
    }
    dmin = wave_min(dmin);
    alive = wave_sum(alive);
    const int w = threadIdx.x / kWave;
    if (lane == 0) {
      s_min[w] = dmin;
      s_cnt[w] = alive;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int x = 0, y = kIntMax;
      for (int i = 0; i < kT / kWave; ++i) {
        x += s_cnt[i];
        y = s_min[i] < y ? s_min[i] : y;
      }
      if (x) atomicAdd(&st->alive, x);
      if (y != kIntMax) atomicMin(&st->minv, y);
    }
  } else {
    // every queued vertex removes its edges to live vertices; a neighbour
    // whose degree falls from level + 1 to level joins the next queue
    const int qn = st->qn;
    const int64_t gw = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
    for (int64_t i = gw; i < qn; i += nw) {
      const int32_t v = qc[i];
      const int64_t rb = row_ptr[v], re = row_ptr[v + 1];
      for (int64_t j0 = rb; j0 < re; j0 += kWave) {
        const int64_t j = j0 + lane;
        bool take = false;
        int32_t u = 0;
        if (j < re) {
          u = col[j];
          if (__hip_atomic_load(&core[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < 0) {
            const int old = atomicSub(&deg[u], 1);
            if (old == level + 1) {
              __hip_atomic_store(&core[u], level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              take = true;
            }
          }
        }
        const int pos = wave_append(&st->next, take);
        if (take) qx[pos] = u;
      }
    }
  }
  // the last workgroup of the step decides the next one
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(&st->arrived, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (s_last && threadIdx.x == 0) {
    __threadfence();
    const int next = __hip_atomic_load(&st->next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (phase == kStart) {
      if (next == 0) {
        if (__hip_atomic_load(&st->alive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
          st->phase = kEnd;
        } else {
          // no vertex at this level: the next level is the smallest live degree
          st->level = __hip_atomic_load(&st->minv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else {
        st->cmax = level;
        st->qn = next;
        st->phase = kTake;
      }
    } else if (next == 0) {
      st->level = level + 1;
      st->phase = kStart;
    } else {
      st->cur = cur ^ 1;
      st->qn = next;
    }
    st->next = 0;
    st->alive = 0;
    st->minv = kIntMax;
    st->arrived = 0;
  }
}

// per-vertex degree and triangle sums over a subgraph's edges (sup = support
// of each subgraph edge inside the subgraph)
__global__ void k_vertex_sums(const int32_t* __restrict__ su, const int32_t* __restrict__ sv,
                              const int32_t* __restrict__ sup, int64_t ms, int32_t* __restrict__ deg,
                              unsigned long long* __restrict__ tri) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= ms) return;
  atomicAdd(&deg[su[e]], 1);
  atomicAdd(&deg[sv[e]], 1);
  atomicAdd(&tri[su[e]], (unsigned long long)sup[e]);
  atomicAdd(&tri[sv[e]], (unsigned long long)sup[e]);
}

// local clustering coefficient of every vertex (0 for degree < 2)
__global__ void k_local_cc(const int32_t* __restrict__ deg, const unsigned long long* __restrict__ tri, int32_t n,
                           double* __restrict__ cc) {
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v >= n) return;
  const double d = (double)deg[v];
  cc[v] = deg[v] >= 2 ? (double)(tri[v] / 2) / (d * (d - 1.0) / 2.0) : 0.0;
}

// vertices with degree > 0 and the sum of their coefficients, in a fixed order
__global__ void __launch_bounds__(1024) k_cc_reduce(const int32_t* __restrict__ deg, const double* __restrict__ cc,
                                                    int32_t n, double* __restrict__ out) {
  __shared__ double s_sum[1024];
  __shared__ double s_cnt[1024];
  double a = 0.0, b = 0.0;
  for (int64_t v = threadIdx.x; v < n; v += blockDim.x) {
    if (deg[v] > 0) {
      a += cc[v];
      b += 1.0;
    }
  }
  s_sum[threadIdx.x] = a;
  s_cnt[threadIdx.x] = b;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      s_sum[threadIdx.x] += s_sum[threadIdx.x + st];
      s_cnt[threadIdx.x] += s_cnt[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = s_cnt[0];
    out[1] = s_sum[0];
  }
}

}  // namespace

size_t core_workspace(int32_t n, Arena& a) {
  for (int i = 0; i < 3; ++i) a.take<int32_t>((size_t)n + 1);
  a.take<CoreCtl>(1);
  a.take<CoreState>(1);
  return a.used;
}

// The levels by ordinary launches.
static int core_steps(const CoreArgs& P, int32_t* q0, int32_t* q1, CoreState* st, int32_t* cmax_out, hipStream_t s) {
  // (a refused grid may have taken vertices)
  hipLaunchKernelGGL(k_core_init, dim3(blocks(P.n)), dim3(kT), 0, s, P.row_ptr, P.n, P.deg, P.core, P.ctl, st);
  // a level with takes costs its start, at most one empty start before it and
  // at most one sub-round per vertex taken: at most 3n + 1 steps in all (a
  // guard against a stuck loop)
  const long long max_steps = 4LL * P.n + 2 * kStepsPerCheck;
  CoreState h;
  for (long long launched = 0;;) {
    for (int i = 0; i < kStepsPerCheck; ++i)
      hipLaunchKernelGGL(k_core_step, dim3(kStepBlocks), dim3(kT), 0, s, P.row_ptr, P.col, P.deg, P.core, P.n, q0, q1,
                         st);
    TRUSS_HIP(hipGetLastError());
    launched += kStepsPerCheck;
    TRUSS_HIP(hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, s));
    TRUSS_HIP(hipStreamSynchronize(s));
    if (h.phase == kEnd) break;
    if (launched > max_steps) {
      set_last_error("core numbers did not finish within %lld steps", max_steps);
      return TRUSS_E_INTERNAL;
    }
  }
  *cmax_out = h.cmax;
  return TRUSS_OK;
}

int compute_core_numbers(const DevGraph& dg, int32_t* core, int32_t* cmax_out, Arena& a, hipStream_t s) {
  CoreArgs P;
  P.deg = a.take<int32_t>((size_t)dg.n + 1);
  P.queue = a.take<int32_t>((size_t)dg.n + 1);
  int32_t* const second = a.take<int32_t>((size_t)dg.n + 1);  // live list, or the steps' second queue
  P.list[0] = second;
  P.list[1] = nullptr;
  P.ctl = a.take<CoreCtl>(1);
  CoreState* const st = a.take<CoreState>(1);
  if (a.overflow()) return TRUSS_E_WORKSPACE;
  // the second live list lies in what the build leaves unused; on a graph of
  // almost only isolated vertices that is too little, and no lists are kept
  if (dg.tmp_bytes >= sizeof(int32_t) * ((size_t)dg.n + 1)) P.list[1] = static_cast<int32_t*>(dg.tmp);
  else P.list[0] = nullptr;
  *cmax_out = 0;
  if (dg.n == 0) return TRUSS_OK;
  P.row_ptr = dg.row_ptr;
  P.col = dg.col;
  P.core = core;
  P.n = dg.n;
  int dev = 0, cus = 0, occ = 0;
  TRUSS_HIP(hipGetDevice(&dev));
  TRUSS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  TRUSS_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void*)k_core, kCoreT, 0));
  if (occ < 1 || cus < 1) return core_steps(P, P.queue, second, st, cmax_out, s);
  hipLaunchKernelGGL(k_core_init, dim3(blocks(dg.n)), dim3(kT), 0, s, dg.row_ptr, dg.n, P.deg, core, P.ctl, st);
  hipLaunchKernelGGL(k_core, dim3((unsigned)cus), dim3(kCoreT), 0, s, P);
  TRUSS_HIP(hipGetLastError());
  int aborted = 0;
  int res[3] = {0, 0, 0};  // cmax, phase, admit
  TRUSS_HIP(hipMemcpyAsync(&aborted, &P.ctl->bar.abort, sizeof(int), hipMemcpyDeviceToHost, s));
  TRUSS_HIP(hipMemcpyAsync(res, &P.ctl->cmax, sizeof(res), hipMemcpyDeviceToHost, s));
  TRUSS_HIP(hipStreamSynchronize(s));
  if (res[2] != kAdmitted) return core_steps(P, P.queue, second, st, cmax_out, s);
  if (aborted || res[1] != kDone) {
    set_last_error("core number kernel barrier timed out");
    return TRUSS_E_INTERNAL;
  }
  *cmax_out = res[0];
  return TRUSS_OK;
}

int subgraph_vertex_stats(int32_t n, const int32_t* su, const int32_t* sv, const int32_t* sup, int64_t ms, Arena& a,
                          double* nv_out, double* cc_out, hipStream_t s) {
  int32_t* deg = a.take<int32_t>((size_t)n + 1);
  unsigned long long* tri = a.take<unsigned long long>((size_t)n + 1);
  double* cc = a.take<double>((size_t)n + 1);
  double* red = a.take<double>(4);
  if (a.overflow()) return TRUSS_E_WORKSPACE;
  TRUSS_HIP(hipMemsetAsync(deg, 0, sizeof(int32_t) * ((size_t)n + 1), s));
  TRUSS_HIP(hipMemsetAsync(tri, 0, sizeof(unsigned long long) * ((size_t)n + 1), s));
  if (ms > 0) hipLaunchKernelGGL(k_vertex_sums, dim3(blocks(ms)), dim3(kT), 0, s, su, sv, sup, ms, deg, tri);
  hipLaunchKernelGGL(k_local_cc, dim3(blocks(n)), dim3(kT), 0, s, deg, tri, n, cc);
  hipLaunchKernelGGL(k_cc_reduce, dim3(1), dim3(1024), 0, s, deg, cc, n, red);
  double h[2] = {0.0, 0.0};
  TRUSS_HIP(hipMemcpyAsync(h, red, sizeof(h), hipMemcpyDeviceToHost, s));
  TRUSS_HIP(hipStreamSynchronize(s));
  *nv_out = h[0];
  *cc_out = h[0] > 0.0 ? h[1] / h[0] : 0.0;
  return TRUSS_OK;
}

}  // namespace truss
