// The library's host code without a GPU: the HIP calls it makes and the
// kernel launchers, by host memory and a replay of the level kernels' control
// protocol.  A search is a script -- frontier sizes and arcs by depth -- and a
// launch does at once what the kernel would do with its control slot: complete
// one level or half of one, run several, or pass the slot on.
#pragma once

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "../../paper_1708_01159_amd/csrc/gsw_internal.h"

namespace fake {

struct Script {
  std::vector<int32_t> nf;    // frontier of every depth
  std::vector<int64_t> arcs;  // ... and its arcs
};

struct Device {
  Script script;
  const int32_t* rows = nullptr;  // records that the host has read
  bool overrun = false;           // a record was overwritten before it was read
  bool stalled = false;           // the host waits for a record that no queued launch posts
  int64_t launches = 0, solo_levels = 0, handed_back = 0;
};
Device dev;

size_t pinned = 0, pinned_room = (size_t)1 << 40;  // bytes of host memory held, and left
std::map<void*, size_t> pinned_size;

inline int next_kernel(const gsw::BfsPolicy& p, int32_t d) {
  if (p.policy == GSW_POLICY_FIXED) return p.fixed;
  return p.sched[d < p.sched_len ? d : p.sched_len - 1];
}

inline int32_t size_at(int32_t d) { return d < (int32_t)dev.script.nf.size() ? dev.script.nf[(size_t)d] : 0; }

// The record of level d, run by kernel k in launch j.
inline void post(const gsw::BfsBase& b, int32_t d, int k, int32_t flags, long long disc, int next, int32_t j) {
  using namespace gsw;
  if (dev.rows && d - *dev.rows >= kBfsRing) dev.overrun = true;
  unsigned long long v[kBfsRec] = {};
  v[kRecKernel] = (unsigned long long)k;
  v[kRecFlags] = (unsigned long long)flags;
  v[kRecNf] = (unsigned long long)size_at(d);
  v[kRecDisc] = (unsigned long long)disc;
  v[kRecNext] = (unsigned long long)size_at(d + 1);
  v[kRecNextKernel] = (unsigned long long)(next + 1);
  v[kRecEf] = b.count_arcs ? (unsigned long long)dev.script.arcs[(size_t)d] + 1ull : 0ull;
  v[kRecLaunch] = (unsigned long long)j;
  for (int i = 0; i < kBfsRec; ++i) b.ring[(size_t)(d % kBfsRing) * kBfsRec + i] = rec_tag(d) | v[i];
}

// The slot of depth d, with `disc` vertices discovered through it.
inline void enter(gsw::BfsCtl* c, int32_t d, int k, long long disc) {
  c->d = d;
  c->kernel = size_at(d) > 0 ? k : gsw::kCtlDone;
  c->nf = size_at(d);
  c->disc = disc;
  c->phase = gsw::level_first_phase(c->kernel, c->nf);
}

}  // namespace fake

namespace gsw {

gsw_status launch_init(const gsw_graph*, const BfsBase& b, const unsigned long long*, int32_t, int32_t k0, int32_t,
                       hipStream_t) {
  fake::enter(b.ctl, 0, k0, 1);
  return GSW_OK;
}

gsw_status launch_level_auto(const gsw_graph*, const BfsBase& b, const BfsPolicy& p, int32_t j, int32_t, hipStream_t) {
  ++fake::dev.launches;
  const BfsCtl c = b.ctl[j & 1];
  BfsCtl* cn = b.ctl + ((j + 1) & 1);
  if (c.kernel < 0) {
    cn->kernel = kCtlDone;
    return GSW_OK;
  }
  if (kernel_base(c.kernel) == GSW_K_PUSH_EDGE && c.phase == 0) {  // the prefix; the expansion is the next launch's
    *cn = c;
    cn->phase = 1;
    return GSW_OK;
  }
  const long long disc = c.disc + fake::size_at(c.d + 1);
  fake::enter(cn, c.d + 1, fake::next_kernel(p, c.d + 1), disc);
  fake::post(b, c.d, c.kernel, 0, c.disc, cn->kernel, j);
  return GSW_OK;
}

gsw_status launch_level_solo(const gsw_graph*, const BfsBase& b, const BfsPolicy& p, int32_t j, bool, hipStream_t) {
  ++fake::dev.launches;
  BfsCtl c = b.ctl[j & 1];
  BfsCtl* cn = b.ctl + ((j + 1) & 1);
  const bool whole = solo_whole(b.n, b.nnz);
  const int last = whole ? GSW_K_PULL_BITMAP : GSW_K_PUSH_EDGE;
  *cn = c;
  if (b.solo <= 0 || c.kernel < 0 || kernel_base(c.kernel) > last || c.nf < 1 || c.nf > b.solo_max) return GSW_OK;
  const bool head_only = !whole && b.head_rows && b.deg_max <= kHeadArcs && !b.count_arcs;
  const int64_t bound = b.deg_max > 0 ? kSoloMaxArcs / b.deg_max : kSoloMax;
  for (int lv = 0;; ++lv) {
    if (!head_only && !whole && c.nf > bound &&
        !solo_takes(c.kernel, (int32_t)c.nf, fake::dev.script.arcs[(size_t)c.d],
                    std::min<int64_t>(b.deg_max, fake::dev.script.arcs[(size_t)c.d]))) {
      ++fake::dev.handed_back;
      if (lv > 0) *cn = c;  // (untouched on the first level)
      return GSW_OK;
    }
    const int32_t d = c.d;
    const int k = c.kernel;
    const long long nf = c.nf, disc = c.disc;
    fake::enter(&c, d + 1, fake::next_kernel(p, d + 1), disc + fake::size_at(d + 1));
    fake::post(b, d, k, kFlagSolo, disc, c.kernel, j);
    ++fake::dev.solo_levels;
    const bool go = lv + 1 < b.solo && c.nf > 0 && kernel_base(c.kernel) <= last && c.nf <= b.solo_max &&
                    (whole || c.nf <= b.solo_nf || (c.nf <= nf && c.disc * 100 >= b.n));
    if (go) continue;
    *cn = c;
    return GSW_OK;
  }
}

int32_t level_kernel_grid(int64_t, int64_t) { return 1536; }
int32_t level_participants(int, int64_t, const BfsBase&) { return 1; }
gsw_status launch_isolated(const gsw_graph*, unsigned long long*, hipStream_t) { return GSW_OK; }
gsw_status launch_canonical_parents(const gsw_graph*, const Workspace&, const int32_t*, int32_t*, hipStream_t) {
  return GSW_OK;
}
gsw_status launch_build_origin(const int64_t*, int64_t, int32_t*, hipStream_t) { return GSW_OK; }
gsw_status launch_build_head(const gsw_graph*, int32_t*, int32_t*, hipStream_t) { return GSW_OK; }
void ms_release(gsw_graph*) {}
void cc_release(gsw_graph*) {}
size_t cc_workspace_bytes(const gsw_graph*) { return 0; }

}  // namespace gsw

extern "C" {

hipError_t hipMalloc(void** p, size_t bytes) {
  *p = std::calloc(1, bytes ? bytes : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = nullptr;
  if (bytes > fake::pinned_room) return hipErrorOutOfMemory;
  fake::pinned_room -= bytes;
  fake::pinned += bytes;
  hipMalloc(p, bytes);
  fake::pinned_size[*p] = bytes;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  fake::pinned -= fake::pinned_size[p];
  fake::pinned_room += fake::pinned_size[p];
  fake::pinned_size.erase(p);
  return hipFree(p);
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
// (the one device array: the scratch memory of gsw_bfs_noalloc)
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static unsigned char* array = static_cast<unsigned char*>(std::calloc(1, GSW_NOALLOC_SCRATCH_BYTES));
  *p = array;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
// Everything queued has run: a host that still waits for a record waits for good.
hipError_t hipStreamQuery(hipStream_t) {
  fake::dev.stalled = true;
  return hipErrorUnknown;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 100000;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "no record"; }

}  // extern "C"
