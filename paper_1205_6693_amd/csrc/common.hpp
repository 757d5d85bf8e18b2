// Device-side helpers shared by the truss kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace truss {

constexpr int kWave = 64;

// ---- lane / wave helpers --------------------------------------------------

__device__ __forceinline__ int lane_id() {
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// number of set bits of `mask` strictly below this lane
__device__ __forceinline__ int rank_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p ? 1 : 0); }

// Orders LDS traffic between lanes of one wavefront (no block barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T x) {
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T y = __shfl_up(x, d, kWave);
    if (lane >= d) x += y;
  }
  return x;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, kWave);
  return x;
}

template <typename T>
__device__ __forceinline__ T wave_min(T x) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    T y = __shfl_xor(x, d, kWave);
    x = y < x ? y : x;
  }
  return x;
}

template <typename T>
__device__ __forceinline__ T wave_max(T x) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    T y = __shfl_xor(x, d, kWave);
    x = y > x ? y : x;
  }
  return x;
}

// Inclusive maximum over the lanes 0..lane (DPP row shifts within rows of 16,
// then the row broadcasts 15 and 31 of the gfx9 wave64 scan).
__device__ __forceinline__ int wave_incl_max(int x) {
  constexpr int lo = (int)0x80000000;
  int y;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x = y > x ? y : x;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x = y > x ? y : x;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x = y > x ? y : x;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x = y > x ? y : x;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x = y > x ? y : x;
  y = __builtin_amdgcn_update_dpp(lo, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  x = y > x ? y : x;
  return x;
}

// ---- device-scope atomics ---------------------------------------------------

__device__ __forceinline__ int atomic_load_relaxed(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-aggregated append: every lane with `want` gets a distinct slot from
// *counter; returns the slot (undefined for lanes without `want`).
__device__ __forceinline__ int wave_append(int* counter, bool want) {
  const uint64_t m = ballot(want);
  if (m == 0) return 0;
  const int leader = __builtin_ctzll(m);
  int base = 0;
  if (lane_id() == leader) base = atomicAdd(counter, __popcll(m));
  base = __shfl(base, leader, kWave);
  return base + rank_below(m);
}

// ---- persistent kernels: coherent accesses and the grid barrier -----------------
// The L2 caches of the XCDs are not coherent with each other, and an
// agent-scope fence writes back and invalidates a whole L2.  So what one phase
// of a persistent kernel writes and another workgroup reads later is accessed with
// agent-scope relaxed atomics, and each lane waits for its own memory
// operations before its workgroup arrives at the barrier; no fences.
template <typename T>
__device__ __forceinline__ T ldc(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void stc(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// wait until this lane's global loads, stores and atomics have completed
__device__ __forceinline__ void mem_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ unsigned long long scalar64(unsigned long long x) {
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
         (unsigned)__builtin_amdgcn_readfirstlane((int)x);
}

constexpr int kGridGroups = 8;  // arrival groups (workgroup id mod 8: one per XCD under round-robin dispatch)
constexpr int kPubMax = 8;
constexpr int kPubBits = 48;    // value bits of a published word

struct GridBarrier {
  alignas(256) unsigned count;                       // groups arrived at all barriers so far
  alignas(256) unsigned long long pub[kPubMax];      // published words
  alignas(256) unsigned grp[kGridGroups][32];        // workgroups arrived so far, per group (a 128-byte line each)
  alignas(128) int abort;                            // set when a wait has timed out
};

__device__ __forceinline__ void grid_barrier_init(GridBarrier* b) {
  b->count = 0;
  for (int i = 0; i < kPubMax; ++i) b->pub[i] = 0ULL;  // tag 0: the first barrier waits for 1
  for (int g = 0; g < kGridGroups; ++g) b->grp[g][0] = 0;
  b->abort = 0;
}

// Barrier over the grid, whose workgroups must all be resident.  The first
// wavefront of the last workgroup to arrive runs control(release), which decides
// the next phase and calls release(word) with the word its lane publishes (lanes
// below NPUB; kPubBits bits) as soon as that is known; what it stores
// afterwards is complete before this workgroup's next arrival.  Each published
// word carries the low 16 bits of the generation above its value and the
// others poll the words themselves, so the release takes one store and one
// load instead of state, flag and state again.  The arrival counters only
// grow, so none has to be reset.  gen: barriers passed, including this one;
// pub: NPUB words of LDS, on return the published values.  Returns false if the
// wait timed out; the kernel then winds down.
template <int NPUB, typename Control>
__device__ __forceinline__ bool grid_barrier(GridBarrier* b, unsigned gen, unsigned long long* pub, Control control) {
  static_assert(NPUB <= kPubMax, "published words");
  __shared__ int s_ok;
  mem_wait();
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int lane = lane_id();
    // two-level arrival: the last workgroup of a group arrives for the group
    int last = 0;
    if (lane == 0) {
      const unsigned g = blockIdx.x % kGridGroups;
      const unsigned gsize = (gridDim.x - g + kGridGroups - 1) / kGridGroups;
      const unsigned ngroups = gridDim.x < (unsigned)kGridGroups ? gridDim.x : (unsigned)kGridGroups;
      const unsigned pg = __hip_atomic_fetch_add(&b->grp[g][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (pg + 1 == gen * gsize) {
        const unsigned prev = __hip_atomic_fetch_add(&b->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = prev + 1 == gen * ngroups ? 1 : 0;
      }
    }
    last = __builtin_amdgcn_readfirstlane(last);
    const unsigned long long want = (unsigned long long)(gen & 0xffffu);
    int ok = 1;
    if (last) {
      control([&](unsigned long long word) {
        if (lane < NPUB) {
          stc(&b->pub[lane], (want << kPubBits) | word);
          pub[lane] = word;
        }
      });
    } else {
      const uint64_t t0 = wall_clock64();
      unsigned long long x = 0;
      for (int spin = 1;; ++spin) {
        x = ldc(&b->pub[lane < NPUB ? lane : 0]);
        if (ballot((x >> kPubBits) != want) == 0) break;
        __builtin_amdgcn_s_sleep(1);
        if ((spin & 63) != 0) continue;
        // 100 MHz constant clock: give up after 30 s
        const bool late = wall_clock64() - t0 > 3000000000ULL;
        if (late && lane == 0) stc(&b->abort, 1);
        if (__builtin_amdgcn_readfirstlane(late || ldc(&b->abort) != 0 ? 1 : 0)) {
          ok = 0;
          break;
        }
      }
      if (lane < NPUB) pub[lane] = x & ((1ULL << kPubBits) - 1ULL);
    }
    if (lane == 0) s_ok = ok;
  }
  __syncthreads();
  return s_ok != 0;
}

// ---- searches in sorted rows ----------------------------------------------------
// lower_bound of `key` in the sorted range a[lo, hi)
template <typename IdxT>
__device__ __forceinline__ IdxT lower_bound_i32(const int* __restrict__ a, IdxT lo, IdxT hi, int key) {
  while (lo < hi) {
    IdxT mid = lo + ((hi - lo) >> 1);
    if (a[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// ---- row hash tables ------------------------------------------------------------
// The membership test of Algorithm 2 (is (v, w) an edge of E_G?) through a
// hash table over E_G (Section 3.2), kept per vertex: the table of v holds
// v's neighbours w with the edge id of (v, w) in 2^lg >= max(4, 2 deg(v)) slots (at
// most half full); an empty slot has w = -1.  The tables of all vertices lie back
// to back (offsets rtoff), so a walk whose entries all look up the same vertex's
// neighbours touches one compact region, which stays in cache, instead of
// lines scattered over one table of all edges.
//
// Slots are probed in buckets of four (32 bytes, aligned), which a lookup reads in
// one step: an entry lies in its home bucket unless that was full, so a lookup ends
// at a match or at a bucket with an empty slot, nearly always the first one.  With slot
// after slot the slowest of a wavefront's 64 lookups took several dependent loads,
// and every peeling round waits for the slowest: R-MAT of 15.7 M edges 94.9 -> 83.5 ms,
// Chung-Lu of 15.5 M 92.0 -> 85.3, R-MAT 23 1192 -> 1173.
__device__ __forceinline__ int row_table_lg(int64_t slots) { return 63 - __builtin_clzll((unsigned long long)slots); }

__device__ __forceinline__ uint32_t row_slot(int32_t w, int lg) { return ((uint32_t)w * 2654435769u) >> (32 - lg); }

// the edge id of w in half a bucket, or -1; whether it has an empty slot.  Entries
// fill the home half before the other one, so an empty slot in it ends a lookup.
__device__ __forceinline__ int half_find(const int4& a, int32_t w) { return a.x == w ? a.y : a.z == w ? a.w : -1; }
__device__ __forceinline__ bool half_open(const int4& a) { return a.x < 0 || a.z < 0; }

// edge id of (v, w) from v's table tb of 2^lg slots, or -1
__device__ __forceinline__ int row_lookup(const int2* __restrict__ tb, int lg, int32_t w) {
  const uint32_t mask = (1u << lg) - 1u;
  for (uint32_t h = row_slot(w, lg) & ~1u;; h = (h + 4) & mask) {
    const int4 a = *(const int4*)(tb + h), b = *(const int4*)(tb + (h ^ 2u));
    int e = half_find(a, w);
    if (e < 0) e = half_find(b, w);
    if (e >= 0 || half_open(a) || half_open(b)) return e;
  }
}

}  // namespace truss
