// Graph build: validation of the simple-graph contract (Section 2), canonical
// edge ids, the symmetric CSR with edge ids, and the (degree, id) orientation
// used for triangle listing (the in-memory triangle counting that Algorithm 2,
// starts from; the smaller-degree rule of its triangle walk and Theorem 1).
#include <utility>

#include "common.hpp"
#include "internal.hpp"

namespace truss {

namespace {

constexpr int kT = 256;

inline unsigned grid_for(int64_t n, int per_block = kT) {
  int64_t b = (n + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > (1LL << 30)) b = 1LL << 30;
  return (unsigned)b;
}

inline int bits_for(int64_t n) {
  int b = 0;
  while (b < 62 && (1LL << b) < n) ++b;
  return b;
}

__device__ __forceinline__ void report(int* err, int code) { atomicMin(err, code); }

// the head, and counters of n + 1 entries (nullable) cleared
__global__ void k_build_init(RunHead* head, int32_t* __restrict__ deg, int64_t n) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    head->err = kNoErr;
    head->sup_total = 0ULL;
    head->wbound = 0ULL;
  }
  if (!deg) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x) deg[i] = 0;
}

// ---- row hash tables (the membership test of Algorithm 2) -----------------------------------

// slots of v's table: the power of two >= 2 deg(v), at least a bucket of four (0 for an
// isolated vertex, and throughout for an invalid input)
__global__ void k_rtab_sizes(const int64_t* __restrict__ row_ptr, int32_t n, int32_t* __restrict__ tsz, const int* err) {
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int64_t d = row_ptr[v + 1] - row_ptr[v];
  int64_t sz = 0;
  if (d > 0 && !invalid(err)) {
    sz = 4;
    while (sz < 2 * d) sz <<= 1;
  }
  tsz[v] = (int32_t)sz;
}

__global__ void k_rtab_clear(int2* __restrict__ rtab, const int64_t* __restrict__ rtoff, int32_t n, int64_t cap) {
  const int64_t total = rtoff[n];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total && i < cap;
       i += (int64_t)gridDim.x * blockDim.x)
    rtab[i] = make_int2(-1, 0);
}

__device__ __forceinline__ void rtab_put(int2* __restrict__ rtab, const int64_t* __restrict__ rtoff, int32_t v,
                                         int32_t w, int32_t e) {
  if (!rtab) return;
  const int64_t off = rtoff[v];
  const int lg = row_table_lg(rtoff[v + 1] - off);
  const uint32_t mask = (1u << lg) - 1u;
  const uint32_t h = row_slot(w, lg);
  // neighbours are distinct and the table is at most half full: a free slot is found
  // the home bucket's slots, its home half first, then the next buckets'
  for (uint32_t p = 0;; ++p) {
    const int64_t at = off + (((h + (p & ~3u)) & mask) ^ (p & 3u));
    if (atomicCAS(&rtab[at].x, -1, w) != -1) continue;
    rtab[at].y = e;
    return;
  }
}

// capacity bound: max(4, 2^ceil(log2(2d))) <= 4d for d >= 1, so all tables fit in 8m slots
inline int64_t rtab_capacity(int64_t m) { return 8 * m + 2; }

// ---- edge-list input ----------------------------------------------------------------

__global__ void k_canon(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t m, int32_t n,
                        int vb, uint64_t* __restrict__ key, int32_t* __restrict__ val, int* err) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= m) return;
  int32_t u = src[i], v = dst[i];
  int code = 0;
  if (u < 0 || u >= n || v < 0 || v >= n) code = kErrRange;
  else if (u == v) code = kErrSelfloop;
  if (code) { report(err, code); u = 0; v = 0; }
  uint64_t a = (uint64_t)(u < v ? u : v), b = (uint64_t)(u < v ? v : u);
  key[i] = (a << vb) | b;
  val[i] = (int32_t)i;
}

// and, for the rows, the larger endpoint and the edge id as sort key and value.
// Repeats count only in an input without errors so far: pairs that have been
// set to key 0 repeat that key, and a CSR with too few upper entries is asymmetric
// (a larger code than a repeat's, so it would be hidden).
__global__ void k_edges_from_keys(const uint64_t* __restrict__ key, const int32_t* __restrict__ val, int64_t m,
                                  int vb, int32_t* __restrict__ eu, int32_t* __restrict__ ev,
                                  int32_t* __restrict__ perm, uint32_t* __restrict__ tkey,
                                  int32_t* __restrict__ tval, int* err) {
  int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= m) return;
  uint64_t k = key[e];
  if (e > 0 && key[e - 1] == k && !invalid(err)) report(err, kErrDup);
  eu[e] = (int32_t)(k >> vb);
  const int32_t v = (int32_t)(k & ((1ULL << vb) - 1));
  ev[e] = v;
  perm[e] = val[e];
  if (tkey) {
    tkey[e] = (uint32_t)v;
    tval[e] = (int32_t)e;
  }
}

// Row offsets without counters: the canonical edges are sorted by their
// smaller endpoint (eu) and, in a second copy, by their larger one (lo_v), so
// uppre[x] / lowpre[x] = edges whose smaller / larger endpoint is below x
// are lower bounds in those arrays; row x of the symmetric CSR starts at
// uppre[x] + lowpre[x] and holds its lower neighbours, then its upper ones.
// (lo_v null: uppre alone.)
__global__ void k_row_bounds(const int32_t* __restrict__ eu, const int32_t* __restrict__ lo_v, int64_t m, int32_t n,
                             int64_t* __restrict__ uppre, int64_t* __restrict__ lowpre,
                             int64_t* __restrict__ row_ptr) {
  const int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (x > n) return;
  const int64_t a = lower_bound_i32<int64_t>(eu, 0, m, (int)x);
  uppre[x] = a;
  if (!lo_v) return;
  const int64_t b = lower_bound_i32<int64_t>(lo_v, 0, m, (int)x);
  lowpre[x] = b;
  row_ptr[x] = a + b;
}

// upper entry of canonical edge e = (u, v): the tail of u's row, after its
// lower entries (row_ptr[u+1] = uppre[u+1] + lowpre[u+1]); and v into u's row table
// (the threads of a block share u, so their inserts land in one table)
__global__ void k_sym_upper(const int32_t* __restrict__ eu, const int32_t* __restrict__ ev, int64_t m,
                            const int64_t* __restrict__ row_ptr, const int64_t* __restrict__ lowpre,
                            int32_t* __restrict__ col, int32_t* __restrict__ seid,
                            const int64_t* __restrict__ rtoff, int2* __restrict__ rtab, const int* err) {
  int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= m) return;
  const bool bad = invalid(err);  // (tested where the other loads have come)
  int32_t u = eu[e], v = ev[e];
  int64_t pos = lowpre[u + 1] + e;
  if (bad) return;
  col[pos] = v;
  seid[pos] = (int32_t)e;
  rtab_put(rtab, rtoff, u, v, (int32_t)e);
}

// lower entry of edge tval[t] = (u, v) with v = tkey[t]: the head of v's row,
// in canonical order (row_ptr[v] = uppre[v] + lowpre[v]); and u into v's row
// table (threads sorted by v, so again one table per run of threads)
__global__ void k_sym_lower(const uint32_t* __restrict__ tkey, const int32_t* __restrict__ tval, int64_t m,
                            const int64_t* __restrict__ row_ptr, const int64_t* __restrict__ uppre,
                            const int32_t* __restrict__ eu, int32_t* __restrict__ col,
                            int32_t* __restrict__ seid, const int64_t* __restrict__ rtoff,
                            int2* __restrict__ rtab, const int* err) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= m) return;
  const bool bad = invalid(err);
  int32_t e = tval[t];
  int32_t v = (int32_t)tkey[t];
  int32_t u = eu[e];
  int64_t pos = uppre[v] + t;
  if (bad) return;
  col[pos] = u;
  seid[pos] = e;
  rtab_put(rtab, rtoff, v, u, e);
}

// ---- locality relabelling ------------------------------------------------------------
// Vertices are renumbered by (degree, id) ascending before the graph is built:
// the orientation order of triangle listing becomes the id order, and the edges
// among high-degree vertices -- the ones the late levels of peeling walk over
// and over -- get the highest canonical ids, so that their supports, stamps and
// rows share lines and stay in cache.  perm maps each relabelled edge back to
// the caller's edge (input pair, or canonical CSR position), so outputs keep
// the caller's order.

// Edge-list input: range and self-loop checks, degrees over the valid pairs.
// A workgroup counts in an LDS table first, one counter a slot, claimed by the
// first vertex that hashes there (another one counts in memory at once): device
// atomics are served at some 27 G a second, and those on one address at one per
// 17 ns, so a hub's count cost 185 us of an R-MAT graph of 592 K edges.
constexpr int kDegT = 1024, kDegSlots = 8192;
__global__ void __launch_bounds__(kDegT) k_edge_degrees(const int32_t* __restrict__ src,
                                                        const int32_t* __restrict__ dst, int64_t m, int32_t n,
                                                        int32_t* __restrict__ deg, int* err) {
  __shared__ int owner[kDegSlots], cnt[kDegSlots];
  for (int x = threadIdx.x; x < kDegSlots; x += kDegT) {
    owner[x] = -1;
    cnt[x] = 0;
  }
  __syncthreads();
  auto count = [&](int32_t v) {
    const int h = (int)((uint32_t)v % kDegSlots);
    int o = owner[h];
    if (o < 0) o = atomicCAS(&owner[h], -1, v);
    if (o < 0 || o == v) atomicAdd(&cnt[h], 1);
    else atomicAdd(&deg[v], 1);
  };
  for (int64_t i = blockIdx.x * (int64_t)kDegT + threadIdx.x; i < m; i += (int64_t)gridDim.x * kDegT) {
    const int32_t u = src[i], v = dst[i];
    if (u < 0 || u >= n || v < 0 || v >= n) {
      report(err, kErrRange);
    } else if (u == v) {
      report(err, kErrSelfloop);
    } else {
      count(u);
      count(v);
    }
  }
  __syncthreads();
  for (int x = threadIdx.x; x < kDegSlots; x += kDegT)
    if (cnt[x]) atomicAdd(&deg[owner[x]], cnt[x]);
}

// sort keys of the vertices: the degree, from the CSR offsets or from deg; in id
// order, so that a stable sort ranks by (degree, id)
__global__ void k_degree_keys(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ deg, int32_t n, int vb,
                              uint32_t* __restrict__ key, int32_t* __restrict__ val) {
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v >= n) return;
  int64_t d = row_ptr ? row_ptr[v + 1] - row_ptr[v] : deg[v];
  const int64_t dmax = (1LL << vb) - 1;  // a simple graph has d < n <= 2^vb; larger only on invalid input
  key[v] = (uint32_t)(d < 0 ? 0 : d > dmax ? dmax : d);
  val[v] = (int32_t)v;
}

__global__ void k_ranks(const int32_t* __restrict__ order, int32_t n, int32_t* __restrict__ rank) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) rank[order[i]] = (int32_t)i;
}

// Canonical keys of the relabelled edges.  The input may still turn out to be
// invalid (its errors are read once, when the build is done): a pair with an id
// out of range or beyond the *valid pairs there are (nullable) gets key 0, so
// that the keys can be sorted and searched like any others.
__global__ void k_canon_relabel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t m,
                                const int64_t* __restrict__ valid, int32_t n, int vb,
                                const int32_t* __restrict__ rank, uint64_t* __restrict__ key,
                                int32_t* __restrict__ val) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= m) return;
  const bool in = !valid || i < *valid;
  const int32_t s = in ? src[i] : -1, d = in ? dst[i] : -1;
  const bool ok = s >= 0 && s < n && d >= 0 && d < n;
  const int32_t u = ok ? rank[s] : 0, v = ok ? rank[d] : 0;
  const uint64_t a = (uint64_t)(u < v ? u : v), b = (uint64_t)(u < v ? v : u);
  key[i] = (a << vb) | b;
  val[i] = (int32_t)i;
}

// ---- CSR input -------------------------------------------------------------------------

__global__ void k_rowptr_check(const int64_t* __restrict__ row_ptr, int32_t n, int64_t m2, int* err) {
  int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v > n) return;
  int64_t r = row_ptr[v];
  if (v == 0 && r != 0) report(err, kErrRowptr);
  if (v == n && r != m2) report(err, kErrRowptr);
  if (v < n && row_ptr[v + 1] < r) report(err, kErrRowptr);
  if (r < 0 || r > m2) report(err, kErrRowptr);
}

// one wavefront per row writes the row id of each entry
__global__ void k_rowid(const int64_t* __restrict__ row_ptr, int32_t n, int32_t* __restrict__ rowid) {
  const int lane = lane_id();
  const int64_t wid = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  for (int64_t v = wid; v < n; v += nw) {
    const int64_t b = row_ptr[v], e = row_ptr[v + 1];
    for (int64_t j = b + lane; j < e; j += kWave) rowid[j] = (int32_t)v;
  }
}

__global__ void k_csr_check(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n,
                            int64_t m2, const int32_t* __restrict__ rowid, int32_t* __restrict__ uf, int* err) {
  int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= m2) return;
  const int32_t v = rowid[j], w = col[j];
  int code = 0;
  if (w < 0 || w >= n) code = kErrRange;
  else if (w == v) code = kErrSelfloop;
  else if (j + 1 < row_ptr[v + 1]) {
    const int32_t x = col[j + 1];
    if (x == w) code = kErrDup;
    else if (x < w && x >= 0) code = kErrUnsorted;
  }
  if (code) report(err, code);
  uf[j] = (w > v && w < n) ? 1 : 0;
}

__global__ void k_csr_upper(const int32_t* __restrict__ col, const int32_t* __restrict__ rowid,
                            const int64_t* __restrict__ upos, int64_t m2, int64_t m, int32_t* __restrict__ colcopy,
                            int32_t* __restrict__ seid, int32_t* __restrict__ eu, int32_t* __restrict__ ev) {
  int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= m2) return;
  const int32_t v = rowid[j], w = col[j];
  if (colcopy) {
    colcopy[j] = w;
    if (w > v) seid[j] = (int32_t)upos[j];
  }
  if (w > v) {
    const int64_t e = upos[j];
    if (e < m) {  // more than m upper entries: an asymmetric input, reported by k_check_total
      eu[e] = v;
      ev[e] = w;
    }
  }
}

__global__ void k_csr_lower(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                            const int32_t* __restrict__ rowid, const int64_t* __restrict__ upos, int64_t m2,
                            int32_t* __restrict__ seid, int* err) {
  int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= m2) return;
  const int32_t v = rowid[j], w = col[j];
  if (w < v) {
    const int64_t lo = row_ptr[w], hi = row_ptr[w + 1];
    const int64_t p = lower_bound_i32<int64_t>(col, lo, hi, v);
    if (p >= hi || col[p] != v) report(err, kErrAsym);
    else if (seid) seid[j] = (int32_t)upos[p];
  }
}

// Symmetry of a CSR input built through the relabelled path: the graph was
// built from the upper entries alone (m of them, no repeats), so the input is
// symmetric iff every lower entry (v, w), w < v, is an edge of that graph --
// looked up in the row table of v's new id or, where no tables are built, in
// the sorted out-neighbours of the smaller new id.
__global__ void k_csr_sym_check(const int32_t* __restrict__ col_in, const int32_t* __restrict__ rowid, int64_t m2,
                                int32_t n, const int32_t* __restrict__ rank, const int2* __restrict__ rtab,
                                const int64_t* __restrict__ rtoff, const int64_t* __restrict__ orow,
                                const int32_t* __restrict__ ocol, int* err) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= m2) return;
  const bool bad = invalid(err);
  const int32_t v = rowid[j], w = col_in[j];
  if (bad || w >= v || w < 0) return;  // (an id out of range is reported by k_csr_check)
  const int32_t x = rank[v], y = rank[w];
  if (rtab) {
    const int64_t off = rtoff[x], slots = rtoff[x + 1] - off;
    if (slots == 0 || row_lookup(rtab + off, row_table_lg(slots), y) < 0) report(err, kErrAsym);
  } else {
    const int32_t a = x < y ? x : y, b = x < y ? y : x;
    const int64_t end = orow[a + 1];
    const int64_t p = lower_bound_i32<int64_t>(ocol, orow[a], end, b);
    if (p >= end || ocol[p] != b) report(err, kErrAsym);
  }
}

__global__ void k_check_total(const int64_t* __restrict__ upos, int64_t m2, int64_t m, int* err) {
  if (upos[m2] != m) report(err, kErrAsym);
}

int read_err(const int* d_err, hipStream_t s) {
  int h = kNoErr;
  TRUSS_HIP(hipMemcpyAsync(&h, d_err, sizeof(int), hipMemcpyDeviceToHost, s));
  TRUSS_HIP(hipStreamSynchronize(s));
  return input_error(h);
}

// buffers of the build, laid out identically for the size query and the run
struct Layout {
  // resident
  int32_t *col, *seid, *eu, *ev, *perm;
  int64_t *row_ptr, *orow;
  // temporaries
  uint64_t *key, *key_alt;
  int32_t *val, *val_alt;
  int64_t *uppre, *lowpre;
  int32_t *rowid, *uf;
  int64_t *opos;
  int32_t *rtmp;
  int64_t *stmp;
  int2* rtab;
  int64_t* rtoff;
  int32_t* tsz;
  size_t tmp_at, tmp_bytes;  // the temporaries' place in the arena
  // relabelling: vertex sort keys and values (ping-pong), their radix scratch, ranks, degrees
  uint32_t *vkey, *vkey_alt;
  int32_t *vval, *vval_alt, *vtmp, *rank, *vdeg;
};

void carve(const truss_graph* g, bool relabel, Arena& a, Layout& L) {
  const int64_t n = g->n, m = g->m, m2 = 2 * m;
  // the edge-list build runs for edge-list input and, after validation, for
  // relabelled CSR input
  const bool edges = g->fmt == TRUSS_FMT_EDGES || relabel;
  L.col = a.take<int32_t>(m2 + 1);
  L.seid = a.take<int32_t>(m2 + 1);
  L.eu = a.take<int32_t>(m + 1);
  L.ev = a.take<int32_t>(m + 1);
  L.orow = a.take<int64_t>(n + 1);
  L.perm = edges ? a.take<int32_t>(m + 1) : nullptr;
  // row tables: of relabelled builds alone
  L.rtab = relabel ? a.take<int2>((size_t)rtab_capacity(m)) : nullptr;
  L.rtoff = relabel ? a.take<int64_t>(n + 1) : nullptr;
  L.tsz = relabel ? a.take<int32_t>(n + 1) : nullptr;
  L.row_ptr = edges ? a.take<int64_t>(n + 1) : nullptr;
  // temporaries: free once the build has returned (DevGraph::tmp)
  L.tmp_at = a.used;
  L.uf = a.take<int32_t>(m2 + 1);
  L.opos = a.take<int64_t>(m2 + 1);
  L.stmp = a.take<int64_t>(scan_tmp_elems(m2 + 1) + scan_tmp_elems(n + 1));
  if (edges) {
    L.key = a.take<uint64_t>(m + 1);
    L.key_alt = a.take<uint64_t>(m + 1);
    L.val = a.take<int32_t>(m + 1);
    L.val_alt = a.take<int32_t>(m + 1);
    L.uppre = a.take<int64_t>(n + 1);
    L.lowpre = a.take<int64_t>(n + 1);
    L.rtmp = a.take<int32_t>(radix_tmp_elems(m + 1));
    L.rowid = g->fmt == TRUSS_FMT_CSR ? a.take<int32_t>(m2 + 1) : nullptr;
  } else {
    L.rowid = a.take<int32_t>(m2 + 1);
    L.key = L.key_alt = nullptr;
    L.val = L.val_alt = nullptr;
    L.uppre = L.lowpre = nullptr;
    L.rtmp = nullptr;
  }
  if (relabel) {
    L.vkey = a.take<uint32_t>(n + 1);
    L.vkey_alt = a.take<uint32_t>(n + 1);
    L.vval = a.take<int32_t>(n + 1);
    L.vval_alt = a.take<int32_t>(n + 1);
    L.vtmp = a.take<int32_t>(radix_tmp_elems(n + 1));
    L.rank = a.take<int32_t>(n + 1);
    L.vdeg = a.take<int32_t>(n + 1);
  } else {
    L.vkey = L.vkey_alt = nullptr;
    L.vval = L.vval_alt = L.vtmp = L.rank = L.vdeg = nullptr;
  }
  // what the peeling keeps there goes in whole: placed by what happens to fit, the
  // workspace would shrink where n or m grows a little
  if (relabel && a.used - L.tmp_at < peel_record_bytes(n, m)) a.used = L.tmp_at + peel_record_bytes(n, m);
  L.tmp_bytes = a.used - L.tmp_at;
}

// ranks of the vertices in (degree, id) order; degrees from row_ptr, else from deg
void degree_ranks(const int64_t* row_ptr, const int32_t* deg, int32_t n, int vb, Layout& L, hipStream_t s) {
  hipLaunchKernelGGL(k_degree_keys, dim3(grid_for(n > 0 ? n : 1)), dim3(kT), 0, s, row_ptr, deg, n, vb, L.vkey,
                     L.vval);
  const bool alt = radix_sort_u32(L.vkey, L.vval, L.vkey_alt, L.vval_alt, n, vb, L.vtmp, s);
  hipLaunchKernelGGL(k_ranks, dim3(grid_for(n > 0 ? n : 1)), dim3(kT), 0, s, alt ? L.vval_alt : L.vval, n, L.rank);
}

// sizes, offsets and cleared slots of the row tables for the rows at row_ptr
void table_layout(const int64_t* row_ptr, int32_t n, int64_t m, Layout& L, const int* d_err, hipStream_t s) {
  hipLaunchKernelGGL(k_rtab_sizes, dim3(grid_for(n > 0 ? n : 1)), dim3(kT), 0, s, row_ptr, n, L.tsz, d_err);
  scan_exclusive_i32_to_i64(L.tsz, L.rtoff, n, L.stmp, s);
  const int64_t cap = rtab_capacity(m);
  hipLaunchKernelGGL(k_rtab_clear, dim3(grid_for(cap) < 65536 ? grid_for(cap) : 65536), dim3(kT), 0, s, L.rtab,
                     L.rtoff, n, cap);
}

// canonical edges and perm, and by `needs` the symmetric rows and their tables,
// from the unsorted canonical keys in L.key / L.val (val: the caller's index of
// each edge).
void rows_from_keys(int32_t n, int64_t m, int vb, Layout& L, int needs, int* d_err, hipStream_t s) {
  if (radix_sort_u64(L.key, L.val, L.key_alt, L.val_alt, m, 2 * vb, L.rtmp, s)) {
    std::swap(L.key, L.key_alt);
    std::swap(L.val, L.val_alt);
  }
  const bool rows = (needs & kBuildRows) != 0;
  uint32_t* tkey = reinterpret_cast<uint32_t*>(L.key_alt);
  uint32_t* tkey_alt = reinterpret_cast<uint32_t*>(L.key);
  hipLaunchKernelGGL(k_edges_from_keys, dim3(grid_for(m)), dim3(kT), 0, s, L.key, L.val, m, vb, L.eu, L.ev, L.perm,
                     rows ? tkey : nullptr, L.val_alt, d_err);
  const int32_t* lo_v = nullptr;
  if (rows) {
    // the canonical order, stably sorted by the larger endpoint (lower halves of the rows)
    if (radix_sort_u32(tkey, L.val_alt, tkey_alt, L.val, m, vb, L.rtmp, s)) std::swap(tkey, tkey_alt);
    else std::swap(L.val, L.val_alt);
    lo_v = reinterpret_cast<const int32_t*>(tkey);
  }
  hipLaunchKernelGGL(k_row_bounds, dim3(grid_for((int64_t)n + 1)), dim3(kT), 0, s, L.eu, lo_v, m, n, L.uppre,
                     L.lowpre, L.row_ptr);
  if (!rows) return;
  int2* rtab = nullptr;
  if (needs & kBuildTables) {
    table_layout(L.row_ptr, n, m, L, d_err, s);
    rtab = L.rtab;
  }
  hipLaunchKernelGGL(k_sym_upper, dim3(grid_for(m)), dim3(kT), 0, s, L.eu, L.ev, m, L.row_ptr, L.lowpre, L.col,
                     L.seid, L.rtoff, rtab, d_err);
  hipLaunchKernelGGL(k_sym_lower, dim3(grid_for(m)), dim3(kT), 0, s, tkey, L.val, m, L.row_ptr, L.uppre, L.eu,
                     L.col, L.seid, L.rtoff, rtab, d_err);
}

}  // namespace

int input_error(int h) {
  if (h == kNoErr) return TRUSS_OK;
  switch (h) {
    case kErrRowptr: set_last_error("CSR row_ptr is not a valid offset array for 2m entries"); break;
    case kErrRange: set_last_error("vertex id outside [0, n)"); break;
    case kErrSelfloop: set_last_error("self-loop in input (simple graphs only)"); break;
    case kErrUnsorted: set_last_error("CSR row not strictly ascending"); break;
    case kErrDup: set_last_error("edge listed more than once"); break;
    case kErrAsym: set_last_error("CSR is not symmetric"); break;
    default: set_last_error("validation failed (%d)", h); break;
  }
  return -h;
}

size_t build_workspace(const truss_graph* g, Arena& a, bool relabel) {
  Layout L;
  carve(g, relabel, a, L);
  return a.used;
}

// Renumbered graph: the canonical edges are sorted by (smaller new id, larger new
// id) and new ids rank the degrees, so the oriented CSR is the edge list itself
// (entry j is edge j, its row offsets uppre).  The input's errors are read once,
// at the end or with the caller's results (and, for CSR input, those of row_ptr at
// the start: the entries are found through it).
static int build_relabelled(const truss_graph* g, Layout& L, DevGraph& dg, int vb, RunHead* head, hipStream_t s,
                            int needs, bool defer) {
  int* const d_err = &head->err;
  const int32_t n = g->n;
  const int64_t m = g->m, m2 = 2 * m;
  const bool edges = g->fmt == TRUSS_FMT_EDGES;
  L.uppre = L.orow;  // kept
  const unsigned gn = grid_for((int64_t)n + 1) < 4096 ? grid_for((int64_t)n + 1) : 4096;
  hipLaunchKernelGGL(k_build_init, dim3(gn), dim3(kT), 0, s, head, edges ? L.vdeg : nullptr, (int64_t)n);
  const int64_t* valid = nullptr;
  const int32_t *src = g->src, *dst = g->dst;
  if (edges) {
    const int64_t groups = (m + 4 * kDegT - 1) / (4 * kDegT);
    hipLaunchKernelGGL(k_edge_degrees, dim3((unsigned)(groups < 1 ? 1 : groups > 2048 ? 2048 : groups)), dim3(kDegT), 0,
                       s, src, dst, m, n, L.vdeg, d_err);
    degree_ranks(nullptr, L.vdeg, n, vb, L, s);
  } else {
    hipLaunchKernelGGL(k_rowptr_check, dim3(grid_for((int64_t)n + 1)), dim3(kT), 0, s, g->row_ptr, n, m2, d_err);
    const int rc = read_err(d_err, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_rowid, dim3(grid_for((int64_t)n * kWave > 0 ? (int64_t)n * kWave : 1)), dim3(kT), 0, s,
                       g->row_ptr, n, L.rowid);
    hipLaunchKernelGGL(k_csr_check, dim3(grid_for(m2)), dim3(kT), 0, s, g->row_ptr, g->col, n, m2, L.rowid, L.uf,
                       d_err);
    scan_exclusive_i32_to_i64(L.uf, L.opos, m2, L.stmp, s);
    hipLaunchKernelGGL(k_check_total, dim3(1), dim3(1), 0, s, L.opos, m2, m, d_err);
    // the upper entries, renamed, go through the edge-list build; perm then maps
    // each edge to its canonical CSR position
    hipLaunchKernelGGL(k_csr_upper, dim3(grid_for(m2)), dim3(kT), 0, s, g->col, L.rowid, L.opos, m2, m,
                       (int32_t*)nullptr, L.seid, L.eu, L.ev);
    src = L.eu;
    dst = L.ev;
    valid = L.opos + m2;
    degree_ranks(g->row_ptr, nullptr, n, vb, L, s);
  }
  hipLaunchKernelGGL(k_canon_relabel, dim3(grid_for(m)), dim3(kT), 0, s, src, dst, m, valid, n, vb, L.rank, L.key,
                     L.val);
  rows_from_keys(n, m, vb, L, needs, d_err, s);
  const bool tables = (needs & kBuildTables) != 0;
  if (!edges && m2 > 0)
    hipLaunchKernelGGL(k_csr_sym_check, dim3(grid_for(m2)), dim3(kT), 0, s, g->col, L.rowid, m2, n, L.rank,
                       tables ? L.rtab : nullptr, L.rtoff, L.uppre, L.ev, d_err);
  TRUSS_HIP(hipGetLastError());
  if (!defer) {
    const int rc = read_err(d_err, s);
    if (rc) return rc;
  }
  dg.orow = L.orow;
  dg.ocol = L.ev;
  dg.row_ptr = L.row_ptr;
  dg.perm = L.perm;
  return TRUSS_OK;
}

int build_graph(const truss_graph* g, Arena& a, DevGraph& dg, RunHead* head, hipStream_t s, bool relabel, int needs,
                bool defer) {
  Layout L;
  carve(g, relabel, a, L);
  if (a.overflow()) return TRUSS_E_WORKSPACE;
  const int32_t n = g->n;
  const int64_t m = g->m, m2 = 2 * m;
  const int vb = bits_for(n) > 0 ? bits_for(n) : 1;
  dg.n = n;
  dg.m = m;
  // no id is in range, and there is no row that could hold the pairs meanwhile
  if (g->fmt == TRUSS_FMT_EDGES && n == 0 && m > 0) return input_error(kErrRange);
  dg.tmp = a.base + L.tmp_at;
  dg.tmp_bytes = L.tmp_bytes;
  dg.col = L.col;
  dg.seid = L.seid;
  dg.eu = L.eu;
  dg.ev = L.ev;
  dg.rtab = L.rtab;
  dg.rtoff = L.rtoff;
  dg.err = &head->err;
  if (relabel) return build_relabelled(g, L, dg, vb, head, s, needs, defer);

  int* const d_err = &head->err;
  hipLaunchKernelGGL(k_build_init, dim3(1), dim3(1), 0, s, head, (int32_t*)nullptr, (int64_t)0);
  int rc;
  if (g->fmt == TRUSS_FMT_EDGES) {
    hipLaunchKernelGGL(k_canon, dim3(grid_for(m)), dim3(kT), 0, s, g->src, g->dst, m, n, vb, L.key, L.val, d_err);
    rows_from_keys(n, m, vb, L, needs, d_err, s);
    if ((rc = read_err(d_err, s))) return rc;
    dg.row_ptr = L.row_ptr;
    dg.perm = L.perm;
  } else {
    hipLaunchKernelGGL(k_rowptr_check, dim3(grid_for((int64_t)n + 1)), dim3(kT), 0, s, g->row_ptr, n, m2, d_err);
    if ((rc = read_err(d_err, s))) return rc;
    hipLaunchKernelGGL(k_rowid, dim3(grid_for((int64_t)n * kWave > 0 ? (int64_t)n * kWave : 1)), dim3(kT), 0, s,
                       g->row_ptr, n, L.rowid);
    hipLaunchKernelGGL(k_csr_check, dim3(grid_for(m2)), dim3(kT), 0, s, g->row_ptr, g->col, n, m2, L.rowid, L.uf,
                       d_err);
    int64_t* upos = L.opos;
    scan_exclusive_i32_to_i64(L.uf, upos, m2, L.stmp, s);
    hipLaunchKernelGGL(k_check_total, dim3(1), dim3(1), 0, s, upos, m2, m, d_err);
    if ((rc = read_err(d_err, s))) return rc;
    const bool own = needs != kBuildRows;  // rows alone: the input's are used as they are
    if (own)
      hipLaunchKernelGGL(k_csr_upper, dim3(grid_for(m2)), dim3(kT), 0, s, g->col, L.rowid, upos, m2, m, L.col, L.seid,
                         L.eu, L.ev);
    hipLaunchKernelGGL(k_csr_lower, dim3(grid_for(m2)), dim3(kT), 0, s, g->row_ptr, g->col, L.rowid, upos, m2,
                       own ? L.seid : nullptr, d_err);
    if ((rc = read_err(d_err, s))) return rc;
    dg.row_ptr = g->row_ptr;
    dg.perm = nullptr;
    if (!own) dg.col = const_cast<int32_t*>(g->col);  // read only
  }
  TRUSS_HIP(hipGetLastError());
  return TRUSS_OK;
}

}  // namespace truss
