// Weakly connected components on the level-switching framework.
//
// The paper expects its per-iteration choice among interchangeable kernels
// to carry over to other traversal algorithms (Section VI).  Components are
// computed here in two phases:
//
//  1. On a symmetric graph, the component of a vertex of largest degree is
//     found by the level-switched BFS itself (the tree picks each level's
//     kernel, Sections III-A and IV-A): its reached vertices take the
//     smallest id among them as their label.  On scale-free and mesh-like
//     graphs this one component holds almost every arc.
//  2. Every other vertex with arcs starts with its own id as label, and
//     minimum-label propagation runs until no label changes.  Each
//     iteration runs one of two interchangeable kernels, chosen per
//     iteration from the active set (the vertices whose label fell in the
//     previous iteration), as BFS levels are chosen from the frontier:
//       push  one lane per active vertex lowers its neighbours' labels with
//             atomicMin; a lowered vertex joins the next active list once
//             (a bitmap claim);
//       pull  one lane per remaining vertex takes the minimum over all its
//             neighbours' labels (no atomics; every arc of the remaining
//             vertices is read).
//     The switching rule pulls once the active vertices' arcs exceed a
//     fraction of the remaining vertices' arcs (the frontier-arc criterion
//     of direction-optimising traversal), else pushes.
//
// Arcs join their ends whatever their direction: on a directed graph both
// the out-arcs and the in-arcs (the transpose the library keeps) of a vertex
// are its neighbours, and phase 1 is skipped (a BFS over out-arcs does not
// reach a weak component).  Labels fall monotonically, so a stale read of a
// label (higher than its current value) only delays a change to a later
// iteration; an iteration that changes nothing read every label as the
// previous iteration left it, which is the fixed point: every arc's ends carry
// the same label, the smallest id of the component.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "gsw_internal.h"

namespace gsw {

using u64 = unsigned long long;

struct CcWorkspace {
  int64_t n = 0;
  int32_t* tmp = nullptr;   // labels when the caller passes host memory
  int32_t* rest = nullptr;  // vertices left to phase 2 (with arcs, not reached in phase 1)
  int32_t* q[2] = {};       // active lists
  u64* mark = nullptr;      // bit per vertex: already on the next active list (push)
  u64* ctr = nullptr;       // device counters (kCcCtr words)
  u64* h_ctr = nullptr;     // pinned copy
  u64* res = nullptr;       // mapped host memory: what k_cc_small found (kCcRes words) ...
  u64* d_res = nullptr;     // ... as seen by the device
  double tick_ms = 0.0;     // milliseconds per wall-clock tick
  hipEvent_t ev[2] = {};
  int32_t seed = -1;        // a vertex of largest out-degree (computed once per graph)
  size_t bytes = 0;
};

namespace {

constexpr int kCcBlock = 256;
constexpr int64_t kCcLane = 32;  // rows of at most this many arcs are walked by their own lane
constexpr int kCcBatch = 8;      // arcs a lane keeps in flight (column loads, then label loads)
constexpr int kCcGridMax = 2048;
// counters, 16 words apart; kCtrClock: when the call began on the device;
// kCtrState: what k_cc_small goes on with (begun, active vertices, their arcs,
// the active list's index, or -1 for `rest`)
enum : int {
  kCtrCount = 0,
  kCtrArcs = 16,
  kCtrKey = 32,
  kCtrReached = 48,
  kCtrRoots = 64,
  kCtrIso = 80,
  kCtrClock = 96,
  kCtrState = 112,
  kCcCtr = 128
};

// k_cc_small: propagation over at most kCcSmall remaining vertices with at
// most kCcSmallArcs arcs runs in one workgroup, kCcRows iterations a launch.
constexpr int kCcWide = 1024;
constexpr int64_t kCcSmall = 4096;
constexpr int64_t kCcSmallArcs = 32768;
constexpr int kCcRows = 64;
constexpr int kCcRow = 5;  // words per iteration: kernel, active, their arcs, changed, ticks
enum : int { kResDone = 0, kResRest, kResArcs, kResReached, kResIso, kResRoots, kResRows, kResTicks, kResRow = 8 };
constexpr int kCcRes = kResRow + kCcRows * kCcRow;

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline unsigned cc_grid(int64_t items) {
  const int64_t b = cdiv(items < 1 ? 1 : items, kCcBlock);
  return (unsigned)(b < kCcGridMax ? b : kCcGridMax);
}

__device__ __forceinline__ int cc_lane() { return (int)__lane_id(); }

__device__ __forceinline__ u64 wave_sum(u64 x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

__device__ __forceinline__ int32_t wave_min(int32_t x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = min(x, __shfl_xor(x, off));
  return x;
}

// Combines one value per thread over the workgroup (op: max, min or sum);
// the result is valid in thread 0.  Reductions over all n vertices end with
// one global atomic per workgroup: one per wave (8192 on one counter for a
// launch of 2048 workgroups) serialise into tens of microseconds.
template <class Op>
__device__ __forceinline__ u64 cc_block_reduce(u64 x, Op op) {
  __shared__ u64 part[kCcBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = op(x, __shfl_xor(x, off));
  if (cc_lane() == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kCcBlock / 64; ++w) x = op(x, part[w]);
  return x;
}
struct CcMax {
  __device__ u64 operator()(u64 a, u64 b) const { return a > b ? a : b; }
};
struct CcMin {
  __device__ u64 operator()(u64 a, u64 b) const { return a < b ? a : b; }
};
struct CcSum {
  __device__ u64 operator()(u64 a, u64 b) const { return a + b; }
};

// Appends the lanes with `take` set to list (one atomic per wave); every
// active lane of the wave calls it with the same control flow.
__device__ __forceinline__ void cc_append(bool take, int32_t v, int32_t* list, u64* count) {
  const u64 m = __ballot(take);
  if (m == 0ull) return;
  const int lane = cc_lane();
  const int leader = __ffsll((long long)m) - 1;
  u64 pos = 0;
  if (lane == leader) pos = atomicAdd(count, (u64)__popcll(m));
  pos = __shfl(pos, leader);
  if (take) list[pos + (u64)__popcll(m & ((1ull << lane) - 1ull))] = v;
}

// Workgroup staging of list appends for loops whose trip count is uniform
// over the workgroup: entries gather in LDS and go out with one global
// atomic per kCcStage of them (appends to one counter serialise, about 11 ns
// each, so one atomic per wave would cost more than the kernel's reads when
// millions of vertices change).  Every thread calls cc_stage_add and
// cc_stage_flush at the same points.
constexpr int kCcStage = 2048;
struct CcStage {
  int32_t buf[kCcStage];
  uint32_t n;
  uint32_t valid;
  unsigned long long base;
};

__device__ __forceinline__ void cc_stage_init(CcStage& S) {
  if (threadIdx.x == 0) S.n = 0u;
  __syncthreads();
}

__device__ __forceinline__ void cc_stage_flush(CcStage& S, int32_t* list, u64* count) {
  __syncthreads();
  const uint32_t m = S.n;
  if (m == 0u) return;  // uniform: every thread read the same S.n after the barrier
  if (threadIdx.x == 0) S.base = atomicAdd(count, (u64)m);
  __syncthreads();
  const u64 b = S.base;
  for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) list[b + i] = S.buf[i];
  __syncthreads();
  if (threadIdx.x == 0) S.n = 0u;
  __syncthreads();
}

// Adds the threads with `take` set (at most one entry per thread per call);
// flushes first when the buffer could overflow.
__device__ __forceinline__ void cc_stage_add(CcStage& S, bool take, int32_t v, int32_t* list, u64* count) {
  __syncthreads();
  if (S.n + blockDim.x > (uint32_t)kCcStage) cc_stage_flush(S, list, count);
  const u64 m = __ballot(take);
  if (m == 0ull) return;
  const int lane = cc_lane();
  const int leader = __ffsll((long long)m) - 1;
  uint32_t pos = 0;
  if (lane == leader) pos = atomicAdd(&S.n, (uint32_t)__popcll(m));
  pos = (uint32_t)__shfl((int)pos, leader);
  if (take) S.buf[pos + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = v;
}

__device__ __forceinline__ int64_t cc_degree(const int64_t* offs, const int64_t* roffs, int32_t v) {
  int64_t d = offs[v + 1] - offs[v];
  if (roffs) d += roffs[v + 1] - roffs[v];
  return d;
}

// A vertex of largest out-degree, the smallest id among ties: the maximum of
// (degree << 32 | (2^31 - 1 - v)).
__global__ void __launch_bounds__(kCcBlock) k_cc_argmax(const int64_t* __restrict__ offs, int64_t n, u64* key) {
  u64 best = 0ull;
  for (int64_t v = (int64_t)blockIdx.x * kCcBlock + threadIdx.x; v < n; v += (int64_t)gridDim.x * kCcBlock) {
    int64_t d = offs[v + 1] - offs[v];
    if (d > 0x7fffffff) d = 0x7fffffff;
    const u64 k = ((u64)d << 32) | (u64)(0x7fffffffu - (uint32_t)v);
    best = k > best ? k : best;
  }
  best = cc_block_reduce(best, CcMax());
  if (threadIdx.x == 0) atomicMax(key, best);
}

// The smallest reached id, from the search's visited bitmap and the degree-0
// bitmap.  Every workgroup walks its own run of words, low ones first, four
// per thread at a time, and stops at its first hit or once a lower one is
// known: a component of most of the graph is found in the first step.
__global__ void __launch_bounds__(kCcBlock) k_cc_first(const u64* __restrict__ vis, const u64* __restrict__ iso,
                                                       int64_t n, int64_t nw, u64* first) {
  const int64_t per = (nw + gridDim.x - 1) / gridDim.x;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = lo + per < nw ? lo + per : nw;
  for (int64_t base = lo; base < hi; base += 4 * kCcBlock) {
    const bool below = threadIdx.x == 0 &&
                       __hip_atomic_load(first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (u64)base * 64;
    if (__syncthreads_or(below)) return;  // (the same in every thread)
    u64 r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t w = base + k * kCcBlock + threadIdx.x;
      r[k] = w < hi ? vis[w] & ~iso[w] : 0ull;
    }
    u64 best = (u64)n;
#pragma unroll
    for (int k = 3; k >= 0; --k)
      if (r[k]) best = (u64)(base + k * kCcBlock + threadIdx.x) * 64 + (u64)(__ffsll((long long)r[k]) - 1);
    best = cc_block_reduce(best, CcMin());  // (padding bits are at or past n)
    if (threadIdx.x == 0 && best < (u64)n) atomicMin(first, best);
    if (__syncthreads_or(threadIdx.x == 0 && best < (u64)n)) return;
  }
}

// Initial labels after phase 1, from the same bitmaps: reached vertices take
// *first, every other vertex its own id; the vertices with arcs among those
// form the list `rest` (count and arcs in the counters); reached and degree-0
// vertices are counted, marks cleared.  A lane takes four vertices (one
// 16-byte store where the labels allow it), a wave four words; its rest
// vertices go to the workgroup's LDS buffer, or past it to the list, with one
// reservation, so there is no barrier in the loop.  At most 256 workgroups:
// their closing atomics on one counter serialise (about 11 ns each), and the
// 2048 that read 4-byte levels here took 28 us at R-MAT scale 22.
__global__ void __launch_bounds__(kCcWide) k_cc_seed_bits(const u64* __restrict__ vis, const u64* __restrict__ iso,
                                                          const int64_t* __restrict__ offs, int64_t n, int64_t nw,
                                                          int32_t* label, int32_t* rest, u64* mark, u64* ctr) {
  __shared__ CcStage S;
  __shared__ u64 s_arcs, s_reached, s_iso;
  if (threadIdx.x == 0) {
    S.n = 0u;
    S.valid = (uint32_t)kCcStage;
    s_arcs = s_reached = s_iso = 0ull;
  }
  __syncthreads();
  const int lane = cc_lane();
  const int32_t gmin = (int32_t)ctr[kCtrKey];
  const bool vec = ((uintptr_t)label & 15u) == 0u;
  const int64_t nwaves = (int64_t)gridDim.x * (kCcWide / 64);
  u64 arcs = 0ull, reached = 0ull, isolated = 0ull;
  for (int64_t w0 = (((int64_t)blockIdx.x * kCcWide + threadIdx.x) >> 6) * 4; w0 < nw; w0 += nwaves * 4) {
    const int64_t w = w0 + (lane >> 4);
    const u64 vw = w < nw ? vis[w] : ~0ull, iw = w < nw ? iso[w] : 0ull;
    const int q = (lane & 15) * 4;
    const int64_t v = w * 64 + q;
    const u64 hit = (vw & ~iw) >> q;
    int32_t lab[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) lab[k] = (hit >> k) & 1ull ? gmin : (int32_t)(v + k);
    if (vec && v + 3 < n) {
      reinterpret_cast<int4*>(label)[v >> 2] = make_int4(lab[0], lab[1], lab[2], lab[3]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (v + k < n) label[v + k] = lab[k];
    }
    if ((lane & 15) == 0 && w < nw) {
      const u64 in = n - w * 64 >= 64 ? ~0ull : (1ull << (n - w * 64)) - 1ull;
      mark[w] = 0ull;
      reached += (u64)__popcll(vw & ~iw & in);
      isolated += (u64)__popcll(iw & in);
    }
    const uint32_t left = (uint32_t)(~vw >> q) & 15u;  // (padding counts as visited)
    if (__ballot(left != 0u) == 0ull) continue;
    const uint32_t cnt = (uint32_t)__popc(left);
    uint32_t inc = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)inc, off);
      if (lane >= off) inc += y;
    }
    const uint32_t total = (uint32_t)__shfl((int)inc, 63);
    u64 at = 0ull;
    if (lane == 0) {
      at = atomicAdd(&S.n, total);
      if (at + total > (u64)kCcStage) {  // (the buffer's use ends at the first that does not fit)
        atomicMin(&S.valid, (uint32_t)at);
        at = (u64)kCcStage + atomicAdd(ctr + kCtrCount, (u64)total);
      }
    }
    at = __shfl(at, 0) + (u64)(inc - cnt);
    for (uint32_t m = left; m != 0u; m &= m - 1u) {
      const int32_t x = (int32_t)v + __ffs((int)m) - 1;
      arcs += (u64)(offs[x + 1] - offs[x]);
      if (at < (u64)kCcStage) S.buf[at] = x; else rest[at - (u64)kCcStage] = x;
      ++at;
    }
  }
  arcs = wave_sum(arcs);
  reached = wave_sum(reached);
  isolated = wave_sum(isolated);
  if (lane == 0) {
    if (arcs) atomicAdd(&s_arcs, arcs);
    if (reached) atomicAdd(&s_reached, reached);
    if (isolated) atomicAdd(&s_iso, isolated);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t m = S.n < S.valid ? S.n : S.valid;
    S.n = m;
    if (m) S.base = atomicAdd(ctr + kCtrCount, (u64)m);
    if (s_arcs) atomicAdd(ctr + kCtrArcs, s_arcs);
    if (s_reached) atomicAdd(ctr + kCtrReached, s_reached);
    if (s_iso) atomicAdd(ctr + kCtrIso, s_iso);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < S.n; i += kCcWide) rest[S.base + i] = S.buf[i];
}

// Initial labels without phase 1: every vertex its own id; the vertices with
// arcs form the list `rest` (count and arcs in the counters), the others are
// counted, marks cleared.
__global__ void __launch_bounds__(kCcBlock) k_cc_seed(const int64_t* __restrict__ offs,
                                                      const int64_t* __restrict__ roffs, int64_t n, int32_t* label,
                                                      int32_t* rest, u64* mark, u64* ctr) {
  __shared__ CcStage S;
  cc_stage_init(S);
  u64 arcs = 0ull, isolated = 0ull;
  for (int64_t base = (int64_t)blockIdx.x * kCcBlock; base < n; base += (int64_t)gridDim.x * kCcBlock) {
    const int64_t v = base + threadIdx.x;
    bool take = false;
    if (v < n) {
      label[v] = (int32_t)v;
      if ((v & 63) == 0) mark[v >> 6] = 0ull;
      const int64_t d = cc_degree(offs, roffs, (int32_t)v);
      take = d > 0;
      isolated += take ? 0ull : 1ull;
      arcs += (u64)d;
    }
    cc_stage_add(S, take, (int32_t)v, rest, ctr + kCtrCount);
  }
  cc_stage_flush(S, rest, ctr + kCtrCount);
  arcs = cc_block_reduce(arcs, CcSum());
  __syncthreads();  // the partials are reused by the second reduction
  isolated = cc_block_reduce(isolated, CcSum());
  if (threadIdx.x == 0 && arcs) atomicAdd(ctr + kCtrArcs, arcs);
  if (threadIdx.x == 0 && isolated) atomicAdd(ctr + kCtrIso, isolated);
}

// A label as the calling kernel has to read and write it: within one launch
// (kOne) iterations follow each other, and what the last one stored or
// lowered has to be seen, so these go to the device's coherence point.
template <bool kOne>
__device__ __forceinline__ int32_t cc_label(const int32_t* p) {
  if constexpr (kOne) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool kOne>
__device__ __forceinline__ void cc_set_label(int32_t* p, int32_t x) {
  if constexpr (kOne) __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = x;
}

// Lowers v's label to lu; true when it fell and v was not yet on the next
// active list (the caller appends it).  A stale plain read of label[v] is
// never below its current value, so the test only skips arcs atomicMin
// would not change.
template <bool kOne>
__device__ __forceinline__ bool cc_lower(int32_t* label, u64* mark, int32_t v, int32_t lu) {
  if (lu >= cc_label<kOne>(label + v)) return false;
  if (lu >= atomicMin(label + v, lu)) return false;
  const u64 bit = 1ull << (v & 63);
  return (atomicOr(mark + (v >> 6), bit) & bit) == 0ull;
}

// Push: every active vertex lowers the labels of its neighbours (out-arcs,
// and in-arcs on a directed graph).  Rows of at most kCcLane arcs are walked
// by their own lane, one arc per step; longer ones by the whole wavefront,
// 64 arcs per step, one row after another.
// Entries base0 + threadIdx.x, base0 + step + threadIdx.x, ...
template <bool kOne>
__device__ __forceinline__ u64 cc_push_rows(const int32_t* qin, int64_t nin, int64_t base0, int64_t step,
                                            int32_t* label, const int64_t* __restrict__ offs,
                                            const int32_t* __restrict__ cols, const int64_t* __restrict__ roffs,
                                            const int32_t* __restrict__ rcols, u64* mark, int32_t* qout, u64* count) {
  const int lane = cc_lane();
  u64 arcs = 0ull;
  const int nrows = roffs ? 2 : 1;
  for (int64_t base = base0; base < nin; base += step) {
    const int64_t i = base + threadIdx.x;
    const bool mine = i < nin;
    const int32_t u = mine ? qin[i] : 0;
    const int32_t lu = mine ? cc_label<kOne>(label + u) : 0;
    for (int r = 0; r < nrows; ++r) {
      const int64_t* ro = r == 0 ? offs : roffs;
      const int32_t* co = r == 0 ? cols : rcols;
      int64_t beg = 0, end = 0;
      if (mine) {
        beg = ro[u];
        end = ro[u + 1];
      }
      const bool own = end - beg <= kCcLane;
      for (int64_t k = 0; __any(own && beg + k < end); k += kCcBatch) {
        int32_t v[kCcBatch], lw[kCcBatch];
#pragma unroll
        for (int q = 0; q < kCcBatch; ++q) v[q] = own && beg + k + q < end ? co[beg + k + q] : -1;
#pragma unroll
        for (int q = 0; q < kCcBatch; ++q) lw[q] = v[q] >= 0 ? cc_label<kOne>(label + v[q]) : 0x7fffffff;
#pragma unroll
        for (int q = 0; q < kCcBatch; ++q) {
          // the plain read filters: only arcs that would lower a label reach the atomics
          const bool take = v[q] >= 0 && lu < lw[q] && cc_lower<kOne>(label, mark, v[q], lu);
          if (take) arcs += (u64)cc_degree(offs, roffs, v[q]);
          cc_append(take, v[q], qout, count);
        }
      }
      u64 longs = __ballot(!own);
      while (longs != 0ull) {
        const int owner = __ffsll((long long)longs) - 1;
        longs &= longs - 1ull;
        const int64_t lo = __shfl(beg, owner), hi = __shfl(end, owner);
        const int32_t lw = __shfl(lu, owner);
        for (int64_t c = lo; c < hi; c += 64) {
          const int64_t e = c + lane;
          bool take = false;
          int32_t v = 0;
          if (e < hi) {
            v = co[e];
            take = cc_lower<kOne>(label, mark, v, lw);
            if (take) arcs += (u64)cc_degree(offs, roffs, v);
          }
          cc_append(take, v, qout, count);
        }
      }
    }
  }
  return arcs;
}

__global__ void __launch_bounds__(kCcBlock) k_cc_push(const int32_t* __restrict__ qin, int64_t nin, int32_t* label,
                                                      const int64_t* __restrict__ offs,
                                                      const int32_t* __restrict__ cols,
                                                      const int64_t* __restrict__ roffs,
                                                      const int32_t* __restrict__ rcols, u64* mark, int32_t* qout,
                                                      u64* ctr) {
  u64 arcs = cc_push_rows<false>(qin, nin, (int64_t)blockIdx.x * kCcBlock, (int64_t)gridDim.x * kCcBlock, label, offs,
                                 cols, roffs, rcols, mark, qout, ctr + kCtrCount);
  arcs = cc_block_reduce(arcs, CcSum());
  if (threadIdx.x == 0 && arcs) atomicAdd(ctr + kCtrArcs, arcs);
}

// Pull: every remaining vertex takes the smallest label among itself and its
// neighbours; the ones whose label fell form the next active list.  Only a
// vertex's own lane writes its label in a pull iteration.
// emit(take, v), by every thread, collects them.
template <bool kOne, class Emit>
__device__ __forceinline__ u64 cc_pull_rows(const int32_t* rest, int64_t nrest, int64_t base0, int64_t step,
                                            int32_t* label, const int64_t* __restrict__ offs,
                                            const int32_t* __restrict__ cols, const int64_t* __restrict__ roffs,
                                            const int32_t* __restrict__ rcols, Emit emit) {
  const int lane = cc_lane();
  u64 arcs = 0ull;
  const int nrows = roffs ? 2 : 1;
  for (int64_t base = base0; base < nrest; base += step) {
    const int64_t i = base + threadIdx.x;
    const bool mine = i < nrest;
    const int32_t v = mine ? rest[i] : 0;
    const int32_t lv = mine ? cc_label<kOne>(label + v) : 0;
    int32_t m = lv;
    for (int r = 0; r < nrows; ++r) {
      const int64_t* ro = r == 0 ? offs : roffs;
      const int32_t* co = r == 0 ? cols : rcols;
      int64_t beg = 0, end = 0;
      if (mine) {
        beg = ro[v];
        end = ro[v + 1];
      }
      const bool own = end - beg <= kCcLane;
      for (int64_t k = 0; __any(own && beg + k < end); k += kCcBatch) {
        if (own && beg + k < end) {
          int32_t u[kCcBatch];
#pragma unroll
          for (int q = 0; q < kCcBatch; ++q) u[q] = beg + k + q < end ? co[beg + k + q] : -1;
#pragma unroll
          for (int q = 0; q < kCcBatch; ++q)
            if (u[q] >= 0) m = min(m, cc_label<kOne>(label + u[q]));
        }
      }
      u64 longs = __ballot(!own);
      while (longs != 0ull) {
        const int owner = __ffsll((long long)longs) - 1;
        longs &= longs - 1ull;
        const int64_t lo = __shfl(beg, owner), hi = __shfl(end, owner);
        int32_t w = 0x7fffffff;
        for (int64_t c = lo + lane; c < hi; c += 64 * 4) {
          int32_t u[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) u[q] = c + 64 * q < hi ? co[c + 64 * q] : -1;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (u[q] >= 0) w = min(w, cc_label<kOne>(label + u[q]));
        }
        w = wave_min(w);
        if (lane == owner) m = min(m, w);
      }
    }
    const bool take = mine && m < lv;
    if (take) {
      cc_set_label<kOne>(label + v, m);
      arcs += (u64)cc_degree(offs, roffs, v);
    }
    emit(take, v);
  }
  return arcs;
}

__global__ void __launch_bounds__(kCcBlock) k_cc_pull(const int32_t* __restrict__ rest, int64_t nrest,
                                                      int32_t* label, const int64_t* __restrict__ offs,
                                                      const int32_t* __restrict__ cols,
                                                      const int64_t* __restrict__ roffs,
                                                      const int32_t* __restrict__ rcols, int32_t* qout, u64* ctr) {
  __shared__ CcStage S;
  cc_stage_init(S);
  u64 arcs = cc_pull_rows<false>(rest, nrest, (int64_t)blockIdx.x * kCcBlock, (int64_t)gridDim.x * kCcBlock, label,
                                 offs, cols, roffs, rcols, [&](bool take, int32_t v) {
                                   cc_stage_add(S, take, v, qout, ctr + kCtrCount);
                                 });
  cc_stage_flush(S, qout, ctr + kCtrCount);
  arcs = cc_block_reduce(arcs, CcSum());
  if (threadIdx.x == 0 && arcs) atomicAdd(ctr + kCtrArcs, arcs);
}

// Clears the list's bits of the mark bitmap (the only bits set after a push).
__global__ void __launch_bounds__(kCcBlock) k_cc_unmark(const int32_t* __restrict__ list, const u64* count,
                                                        u64* mark) {
  const int64_t cnt = (int64_t)*count;
  for (int64_t i = (int64_t)blockIdx.x * kCcBlock + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * kCcBlock)
    mark[list[i] >> 6] = 0ull;
}

// Components among the remaining vertices: those that are their own label.
__global__ void __launch_bounds__(kCcBlock) k_cc_roots(const int32_t* __restrict__ rest, int64_t nrest,
                                                       const int32_t* __restrict__ label, u64* roots) {
  u64 c = 0ull;
  for (int64_t i = (int64_t)blockIdx.x * kCcBlock + threadIdx.x; i < nrest; i += (int64_t)gridDim.x * kCcBlock)
    c += label[rest[i]] == rest[i] ? 1ull : 0ull;
  c = cc_block_reduce(c, CcSum());
  if (threadIdx.x == 0 && c) atomicAdd(roots, c);
}

// Phase 2 in one workgroup, where little is left of the graph (kCcSmall): the
// iterations of the host's loop, with the same choice between push and pull,
// up to kCcRows of them, and the components at the end; what it found goes to
// the host in one go.  A launch per iteration with the host in between cost
// 35 us each; three here take 25 in all (R-MAT scale 22, 1326 vertices; 42 with
// fences of the whole device, which write the L2 back).
__global__ void __launch_bounds__(kCcWide) k_cc_small(const int32_t* rest, int32_t* label,
                                                      const int64_t* __restrict__ offs,
                                                      const int32_t* __restrict__ cols,
                                                      const int64_t* __restrict__ roffs,
                                                      const int32_t* __restrict__ rcols, u64* mark, int32_t* q0,
                                                      int32_t* q1, int policy, double pull_above, u64* ctr, u64* res) {
  __shared__ u64 s_cnt, s_arcs, s_roots;
  const int tid = threadIdx.x;
  const u64 began = (u64)wall_clock64();
  const int64_t n_rest = (int64_t)ctr[kCtrCount], e_rest = (int64_t)ctr[kCtrArcs];
  const bool small = n_rest <= kCcSmall && e_rest <= kCcSmallArcs;
  int64_t n_act = n_rest, e_act = e_rest;
  int cur = -1;
  if (ctr[kCtrState]) {
    n_act = (int64_t)ctr[kCtrState + 1];
    e_act = (int64_t)ctr[kCtrState + 2];
    cur = (int)ctr[kCtrState + 3];
  }
  if (tid == 0) s_roots = 0ull;
  __syncthreads();  // (the state is rewritten at the end)
  int rows = 0;
  while (small && n_act > 0 && rows < kCcRows) {
    const u64 t0 = (u64)wall_clock64();
    const bool pull = policy == GSW_CC_PULL ||
                      (policy != GSW_CC_PUSH && (double)e_act > pull_above * (double)e_rest);
    const int32_t* act = cur < 0 ? rest : cur == 0 ? q0 : q1;
    int32_t* out = cur == 0 ? q1 : q0;
    if (tid == 0) s_cnt = s_arcs = 0ull;
    __syncthreads();
    u64 arcs;
    if (pull)
      arcs = cc_pull_rows<true>(rest, n_rest, 0, kCcWide, label, offs, cols, roffs, rcols,
                                [&](bool take, int32_t v) { cc_append(take, v, out, &s_cnt); });
    else
      arcs = cc_push_rows<true>(act, n_act, 0, kCcWide, label, offs, cols, roffs, rcols, mark, out, &s_cnt);
    arcs = wave_sum(arcs);
    if (cc_lane() == 0 && arcs) atomicAdd(&s_arcs, arcs);
    __builtin_amdgcn_s_waitcnt(0);  // labels are in place before the next iteration reads them
    __syncthreads();
    const int64_t changed = (int64_t)s_cnt, e_next = (int64_t)s_arcs;
    if (!pull)
      for (int64_t i = tid; i < changed; i += kCcWide)
        __hip_atomic_store(mark + (out[i] >> 6), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) {
      const u64 t1 = (u64)wall_clock64();
      const u64 row[kCcRow] = {pull ? (u64)GSW_CC_K_PULL : (u64)GSW_CC_K_PUSH, (u64)n_act, (u64)e_act, (u64)changed,
                               t1 > t0 ? t1 - t0 : 0ull};
      for (int i = 0; i < kCcRow; ++i)
        __hip_atomic_store(res + kResRow + rows * kCcRow + i, row[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __builtin_amdgcn_s_waitcnt(0);  // marks are clear before the next push
    __syncthreads();
    n_act = changed;
    e_act = e_next;
    cur = cur == 0 ? 1 : 0;
    ++rows;
  }
  if (small && n_act == 0) {
    u64 c = 0ull;
    for (int64_t i = tid; i < n_rest; i += kCcWide) c += cc_label<true>(label + rest[i]) == rest[i] ? 1ull : 0ull;
    c = wave_sum(c);
    if (cc_lane() == 0 && c) atomicAdd(&s_roots, c);
    __syncthreads();
  }
  if (tid == 0) {
    const bool done = small && n_act == 0;
    const u64 out[kResRow] = {done ? 1ull : 0ull, (u64)n_rest, (u64)e_rest, ctr[kCtrReached], ctr[kCtrIso], s_roots,
                              (u64)rows, began > ctr[kCtrClock] ? began - ctr[kCtrClock] : 0ull};
    for (int i = 0; i < kResRow; ++i)
      __hip_atomic_store(res + i, out[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    ctr[kCtrState] = 1ull;
    ctr[kCtrState + 1] = (u64)n_act;
    ctr[kCtrState + 2] = (u64)e_act;
    ctr[kCtrState + 3] = (u64)cur;
  }
}

// Counters to zero, the smallest reached id to n, the call's clock to now.
__global__ void k_cc_zero(u64* ctr, int64_t n) {
  for (int i = threadIdx.x; i < kCcCtr; i += blockDim.x)
    ctr[i] = i == kCtrKey ? (u64)n : i == kCtrClock ? (u64)wall_clock64() : 0ull;
}

void cc_free(CcWorkspace* w) {
  if (!w) return;
  void* p[] = {w->tmp, w->rest, w->q[0], w->q[1], w->mark, w->ctr};
  for (void* x : p)
    if (x) (void)hipFree(x);
  if (w->h_ctr) (void)hipHostFree(w->h_ctr);
  if (w->res) (void)hipHostFree(w->res);
  for (hipEvent_t e : w->ev)
    if (e) (void)hipEventDestroy(e);
  delete w;
}

size_t cc_bytes_for(int64_t n) {
  const size_t nw = (size_t)cdiv(n, 64);
  return 4 * (size_t)n * sizeof(int32_t) + nw * sizeof(u64) + kCcCtr * sizeof(u64);
}

gsw_status ensure_cc(gsw_graph* g) {
  if (g->cc) return GSW_OK;
  CcWorkspace* w = new (std::nothrow) CcWorkspace();
  if (!w) return fail(GSW_ENOMEM, "host allocation failed");
  w->n = g->n;
  const size_t nb = (size_t)g->n * sizeof(int32_t);
  struct Item {
    void** p;
    size_t bytes;
  } items[] = {{(void**)&w->tmp, nb},
               {(void**)&w->rest, nb},
               {(void**)&w->q[0], nb},
               {(void**)&w->q[1], nb},
               {(void**)&w->mark, (size_t)cdiv(g->n, 64) * sizeof(u64)},
               {(void**)&w->ctr, kCcCtr * sizeof(u64)}};
  for (auto& it : items) {
    if (hipMalloc(it.p, it.bytes) != hipSuccess) {
      (void)hipGetLastError();
      cc_free(w);
      return fail(GSW_ENOMEM, "hipMalloc(%zu) for connected components failed", it.bytes);
    }
    w->bytes += it.bytes;
  }
  // (the mark bitmap is cleared by every call, on its stream)
  int khz = 0;
  if (hipHostMalloc((void**)&w->h_ctr, kCcCtr * sizeof(u64), hipHostMallocDefault) != hipSuccess ||
      hipHostMalloc((void**)&w->res, kCcRes * sizeof(u64), hipHostMallocMapped | hipHostMallocCoherent) !=
          hipSuccess ||
      hipHostGetDevicePointer((void**)&w->d_res, w->res, 0) != hipSuccess ||
      hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, g->device) != hipSuccess ||
      hipEventCreate(&w->ev[0]) != hipSuccess || hipEventCreate(&w->ev[1]) != hipSuccess) {
    (void)hipGetLastError();
    cc_free(w);
    return fail(GSW_EHIP, "connected-components staging memory or events");
  }
  w->tick_ms = khz > 0 ? 1.0 / (double)khz : 0.0;
  g->cc = w;
  return GSW_OK;
}

// Reads the counters back (waits for the stream).
gsw_status cc_read(CcWorkspace& w, hipStream_t s) {
  GSW_HIP(hipMemcpyAsync(w.h_ctr, w.ctr, kCcCtr * sizeof(u64), hipMemcpyDeviceToHost, s));
  GSW_HIP(hipStreamSynchronize(s));
  return GSW_OK;
}

void cc_row(gsw_cc_trace* t, int32_t it, int32_t kernel, int64_t n_active, int64_t e_active, int64_t changed,
            float ms) {
  t->iteration = it;
  t->kernel = kernel;
  t->n_active = n_active;
  t->e_active = e_active;
  t->changed = changed;
  t->ms = ms;
}

}  // namespace

void cc_release(gsw_graph* g) {
  cc_free(g->cc);
  g->cc = nullptr;
}

size_t cc_workspace_bytes(const gsw_graph* g) { return g->cc ? g->cc->bytes : 0; }

}  // namespace gsw

using namespace gsw;

extern "C" {

void gsw_cc_opts_default(gsw_cc_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof *o);
  o->policy = GSW_CC_SWITCH;
  o->bfs_first = 1;
  o->pull_above = 0.05f;
}

gsw_status gsw_cc(const gsw_graph* cg, int32_t* labels, int64_t* n_components, gsw_cc_trace* trace,
                  int32_t trace_cap, int32_t* trace_len, const gsw_cc_opts* opts) {
  clear_error();
  if (trace_len) *trace_len = 0;
  if (n_components) *n_components = 0;
  if (!cg || !labels) return fail(GSW_EINVAL, "null graph or labels");
  if (trace_cap < 0 || (trace_cap > 0 && !trace)) return fail(GSW_EINVAL, "trace_cap > 0 without a trace");
  gsw_cc_opts def;
  gsw_cc_opts_default(&def);
  const gsw_cc_opts* o = opts ? opts : &def;
  if (o->policy != GSW_CC_SWITCH && o->policy != GSW_CC_PUSH && o->policy != GSW_CC_PULL)
    return fail(GSW_EINVAL, "unknown components policy %d", o->policy);
  if (!(o->pull_above >= 0.0f)) return fail(GSW_EINVAL, "pull_above must be >= 0");
  gsw_graph* g = const_cast<gsw_graph*>(cg);
  std::lock_guard<std::mutex> lock(g->mu);
  GSW_HIP(hipSetDevice(g->device));
  GSW_TRY(ensure_cc(g));
  CcWorkspace& w = *g->cc;
  const hipStream_t s = pick_stream(g, o->stream);
  const int64_t n = g->n;
  const int64_t* roffs = g->symmetric ? nullptr : g->roffs;
  const int32_t* rcols = g->symmetric ? nullptr : g->rcols;
  int32_t* lab = o->device_ptrs ? labels : w.tmp;
  int32_t rows = 0;
  auto add_row = [&](int32_t it, int32_t k, int64_t na, int64_t ea, int64_t ch, float ms) {
    if (trace && rows < trace_cap) cc_row(&trace[rows], it, k, na, ea, ch, ms);
    ++rows;
  };
  auto zero = [&]() { hipLaunchKernelGGL(k_cc_zero, dim3(1), dim3(kCcCtr), 0, s, w.ctr, n); };
  auto elapsed = [&]() -> float {
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, w.ev[0], w.ev[1]);
    return ms;
  };

  zero();
  const bool bfs = o->bfs_first && g->symmetric && g->nnz > 0;
  if (bfs) {
    if (w.seed < 0) {
      hipLaunchKernelGGL(k_cc_argmax, dim3(cc_grid(n)), dim3(kCcBlock), 0, s, g->offs, n, w.ctr + kCtrKey);
      GSW_HIP(hipGetLastError());
      GSW_TRY(cc_read(w, s));
      w.seed = (int32_t)(0x7fffffffu - (uint32_t)(w.h_ctr[kCtrKey] & 0xffffffffull));
      zero();
    }
    const int32_t seed = w.seed;
    GSW_TRY(bfs_rows_locked(g, &seed, 1, lab, o->tree, s, false, true));
    const int64_t nw = g->ws.nw;
    const int64_t steps = cdiv(nw, 4 * kCcBlock), seeds = cdiv(nw, 4 * (kCcWide / 64));
    hipLaunchKernelGGL(k_cc_first, dim3((unsigned)(steps < 256 ? steps : 256)), dim3(kCcBlock), 0, s,
                       (const u64*)g->ws.vis, (const u64*)g->iso, n, nw, w.ctr + kCtrKey);
    hipLaunchKernelGGL(k_cc_seed_bits, dim3((unsigned)(seeds < 256 ? seeds : 256)), dim3(kCcWide), 0, s,
                       (const u64*)g->ws.vis, (const u64*)g->iso, g->offs, n, nw, lab, w.rest, w.mark, w.ctr);
  } else {
    hipLaunchKernelGGL(k_cc_seed, dim3(cc_grid(n)), dim3(kCcBlock), 0, s, g->offs, roffs, n, lab, w.rest, w.mark,
                       w.ctr);
  }
  int32_t it = 0;
  bool done = false;
  int64_t n_rest = 0, e_rest = 0, found = 0;  // found: components but for the remaining vertices'
  for (bool again = true; again;) {
    hipLaunchKernelGGL(k_cc_small, dim3(1), dim3(kCcWide), 0, s, (const int32_t*)w.rest, lab, g->offs, g->cols, roffs,
                       rcols, w.mark, w.q[0], w.q[1], (int)o->policy, (double)o->pull_above, w.ctr, w.d_res);
    GSW_HIP(hipGetLastError());
    GSW_HIP(hipStreamSynchronize(s));
    const volatile u64* r = w.res;
    done = r[kResDone] != 0;
    n_rest = (int64_t)r[kResRest];
    e_rest = (int64_t)r[kResArcs];
    if (bfs && it == 0)
      add_row(it++, GSW_CC_K_BFS, 1, -1, (int64_t)r[kResReached], (float)((double)r[kResTicks] * w.tick_ms));
    const int n_rows = (int)r[kResRows];
    for (int i = 0; i < n_rows; ++i) {
      const volatile u64* x = r + kResRow + i * kCcRow;
      add_row(it++, (int32_t)x[0], (int64_t)x[1], (int64_t)x[2], (int64_t)x[3], (float)((double)x[4] * w.tick_ms));
    }
    found = (int64_t)r[kResIso] + (bfs ? 1 : 0) + (done ? (int64_t)r[kResRoots] : 0);
    again = !done && n_rows > 0;  // (none: more is left than one workgroup takes)
  }

  const int32_t* act = w.rest;
  int64_t n_act = done ? 0 : n_rest, e_act = e_rest;
  int cur = 0;
  for (; n_act > 0; ++it) {
    int k;
    if (o->policy == GSW_CC_PUSH) k = GSW_CC_K_PUSH;
    else if (o->policy == GSW_CC_PULL) k = GSW_CC_K_PULL;
    else k = (double)e_act > (double)o->pull_above * (double)e_rest ? GSW_CC_K_PULL : GSW_CC_K_PUSH;
    int32_t* out = w.q[cur];
    zero();
    GSW_HIP(hipEventRecord(w.ev[0], s));
    if (k == GSW_CC_K_PUSH) {
      hipLaunchKernelGGL(k_cc_push, dim3(cc_grid(n_act)), dim3(kCcBlock), 0, s, act, n_act, lab, g->offs, g->cols,
                         roffs, rcols, w.mark, out, w.ctr);
      GSW_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_cc_unmark, dim3(cc_grid(n_act)), dim3(kCcBlock), 0, s, (const int32_t*)out,
                         (const u64*)(w.ctr + kCtrCount), w.mark);
    } else {
      hipLaunchKernelGGL(k_cc_pull, dim3(cc_grid(n_rest)), dim3(kCcBlock), 0, s, (const int32_t*)w.rest, n_rest,
                         lab, g->offs, g->cols, roffs, rcols, out, w.ctr);
    }
    GSW_HIP(hipGetLastError());
    GSW_HIP(hipEventRecord(w.ev[1], s));
    GSW_TRY(cc_read(w, s));
    const int64_t changed = (int64_t)w.h_ctr[kCtrCount];
    add_row(it, k, n_act, e_act, changed, elapsed());
    act = out;
    n_act = changed;
    e_act = (int64_t)w.h_ctr[kCtrArcs];
    cur ^= 1;
  }
  if (!done) {
    zero();
    hipLaunchKernelGGL(k_cc_roots, dim3(cc_grid(n_rest)), dim3(kCcBlock), 0, s, (const int32_t*)w.rest, n_rest,
                       (const int32_t*)lab, w.ctr + kCtrRoots);
    GSW_HIP(hipGetLastError());
  }
  if (!o->device_ptrs)
    GSW_HIP(hipMemcpyAsync(labels, lab, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  if (!done) {
    GSW_TRY(cc_read(w, s));
    found += (int64_t)w.h_ctr[kCtrRoots];
  } else if (!o->device_ptrs) {
    GSW_HIP(hipStreamSynchronize(s));
  }
  if (n_components) *n_components = found;
  if (trace_len) *trace_len = rows;
  return GSW_OK;
}

}  // extern "C"
