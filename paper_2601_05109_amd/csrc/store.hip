// Device-resident graph store: the global view kept in HBM across passes and
// updated by deltas (futures appended with their dependencies, futures
// completed, deadlines and instances replaced), so that a pass needs no
// upload or rebuild of the snapshot.  The arrays are the snapshot's own struct
// of arrays (ids in append order), grown geometrically.  A pass over the
// store gives the results of nalar_policy_pass over them: after a successful
// pass the store keeps every future's remaining critical path, and the next
// pass recomputes it only for the futures appended or completed since and
// their ancestors (incremental.hip), falling back to a full pass when it
// cannot (no earlier pass, no splitters, a bin overflow).
#include <cstring>

#include "internal.hpp"
#include "nalar_store.h"

using namespace nalar;

struct nalar_store {
  nalar_policy* h = nullptr;
  int64_t N = 0, E = 0, W = 0, M = 0;
  int64_t capN = 0, capE = 0, capW = 0, capM = 0;
  bool contiguous = true;
  int32_t* wf = nullptr;
  int32_t* type = nullptr;
  int64_t* est = nullptr;
  uint8_t* done = nullptr;
  int32_t* loc = nullptr;
  uint4* att = nullptr;         // [capN] att_pack, for the incremental passes
  int32_t* dep_off = nullptr;   // [capN + 1]
  int32_t* dep_idx = nullptr;   // [capE]
  int64_t* deadline = nullptr;  // [capW]
  int32_t* inst_type = nullptr; // [capM]
  int64_t* inst_load = nullptr;
  int32_t* inst_speed = nullptr;
  uint32_t* bad = nullptr;      // pinned: count of completion calls with an id out of range,
                                //   and of appends whose offsets are malformed
  uint32_t bad_seen = 0;        // the count when last reported (only the device writes *bad)
  // incremental passes
  bool incremental = true;      // nalar_store_set_incremental
  bool rem_valid = false;       // rem holds [0, n_prev) from the last successful pass
  int last_incremental = 0;     // the last pass was an incremental one
  int last_fallback = 0;        // why the last pass was a full one (NALAR_STORE_FULL_*)
  int64_t n_prev = 0;
  int64_t W_prev = 0, M_prev = 0; // workflows and instances at the last pass (fewer now: the
                                //   stored futures must be validated again, in a full pass)
  int64_t capI = 0;             // futures the incremental buffers hold
  int64_t* rem = nullptr;       // [capI]
  uint2* fl = nullptr;          // [capI / 32 + 1] membership and done bits (pass scratch)
  int64_t* mxA = nullptr;
  int32_t* cntA = nullptr;
  int32_t* light = nullptr;
  int32_t* heavy = nullptr;
  uint64_t* rbits = nullptr;    // [capI / 64 + 1]
  int32_t* hv = nullptr;        // [capH] futures with more than kIncHeavy dependencies
  int32_t* rheavy = nullptr;    // [capH]
  uint32_t* hv_n = nullptr;     // their number (device memory; the appends count)
  int64_t capH = 0;
  bool hv_stale = false;        // a malformed append may be missing from hv
  IncCtrl* ic = nullptr;
  uint32_t rounds = kIncRoundsAll;  // depth of the last incremental pass (the next one's launch plan)
  int32_t* log = nullptr;       // ids completed since the last pass
  int64_t n_log = 0, capLog = 0;
};

namespace {

constexpr int kStoreThreads = 256;

// One append: every array of the call copied to the end of the store, and the
// offsets, given relative to the call, rebased by the store's edge count
// (off[0], the previous end, is kept).  Offsets that do not start at 0, end at
// the call's edge count and never decrease are counted in *bad, so the next
// pass reports NALAR_EINVAL.
//
// One launch instead of a copy per array: a control tick appends little (tens
// to thousands of futures between passes), and what it costs is the enqueuing.
// A tick of completions, an append and the pass over 1.3M futures took 326 us
// with six copies and a kernel, 308 us with this one.  A large append (millions
// of futures at once) streams through the same loop, coalesced at each array's
// own width.
struct AppendArgs {
  int32_t* wf;
  int32_t* type;
  int64_t* est;
  uint8_t* done;
  int32_t* loc;
  int32_t* off;
  int32_t* idx;
  const int32_t* swf;
  const int32_t* stype;
  const int64_t* sest;
  const uint8_t* sdone;
  const int32_t* sloc;
  const int32_t* soff;
  const int32_t* sidx;
  int64_t n, n_edges;
  int32_t base;
  uint32_t* bad;
  uint4* att;
  int32_t id0;                  // id of the first appended future
  int32_t* hv;                  // futures with more than kIncHeavy dependencies
  uint32_t* hv_n;
  int64_t hv_cap;
};

// Lists future v; false when the list is full.  The count stays at the entries
// written (a full list's count only rises above its capacity for a moment, and
// no entry is freed), so every counted entry is a stored future's id.
__device__ inline bool list_heavy(int32_t* hv, uint32_t* hv_n, int64_t cap, int32_t v) {
  const uint32_t at = atomicAdd(hv_n, 1u);
  if (int64_t(at) < cap) {
    hv[at] = v;
    return true;
  }
  atomicSub(hv_n, 1u);
  return false;
}

__global__ __launch_bounds__(kStoreThreads) void k_store_append(AppendArgs a) {
  bool b = false;
  const int64_t step = int64_t(gridDim.x) * kStoreThreads;
  const int64_t g0 = int64_t(blockIdx.x) * kStoreThreads + threadIdx.x;
  for (int64_t i = g0; i < a.n; i += step) {
    const int32_t wf = a.swf[i], type = a.stype[i], loc = a.sloc[i];
    const int64_t est = a.sest[i];
    a.wf[i] = wf;
    a.type[i] = type;
    a.est[i] = est;
    a.done[i] = a.sdone[i];
    a.loc[i] = loc;
    a.att[i] = att_pack(wf, type, est, loc);
    const int32_t x0 = a.soff[i], x1 = a.soff[i + 1];
    b |= x1 < x0 || (i == 0 && x0 != 0) || (i == a.n - 1 && int64_t(x1) != a.n_edges);
    a.off[i + 1] = a.base + x1;
    // (the degree as stored: off[0] was written by the append before)
    const int64_t deg = int64_t(a.base) + x1 - (i == 0 ? int64_t(a.off[0]) : int64_t(a.base) + x0);
    if (deg > kIncHeavy) {
      // more than the edges allow: malformed offsets
      b |= !list_heavy(a.hv, a.hv_n, a.hv_cap, a.id0 + int32_t(i));
    }
  }
  for (int64_t e = g0; e < a.n_edges; e += step) a.idx[e] = a.sidx[e];
  if (ballot(b) != 0 && lane_id() == 0)
    __hip_atomic_fetch_add(a.bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The list of futures with more than kIncHeavy dependencies made again from
// validated offsets (a malformed append may have left futures out of it).
__global__ __launch_bounds__(kStoreThreads) void k_store_heavy(const int32_t* off, int64_t N, int32_t* hv,
                                                               uint32_t* hv_n, int64_t cap) {
  for (int64_t i = int64_t(blockIdx.x) * kStoreThreads + threadIdx.x; i < N; i += int64_t(gridDim.x) * kStoreThreads)
    if (off[i + 1] - off[i] > kIncHeavy) list_heavy(hv, hv_n, cap, int32_t(i));
}

// Completed ids: their done flags set, and the ids kept for the next pass (log).
__global__ __launch_bounds__(kStoreThreads) void k_store_complete(uint8_t* done, int32_t* log, const int32_t* ids,
                                                                  int64_t n, int64_t N, uint32_t* bad) {
  bool b = false;
  for (int64_t i = int64_t(blockIdx.x) * kStoreThreads + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kStoreThreads) {
    const int32_t v = ids[i];
    if (log) log[i] = v;
    if (v >= 0 && int64_t(v) < N) done[v] = 1;
    else b = true;
  }
  if (ballot(b) != 0 && lane_id() == 0)
    __hip_atomic_fetch_add(bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

int grid_for(int64_t n) {
  int64_t g = (n + kStoreThreads - 1) / kStoreThreads;
  return int(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

// Grow one array to hold `need` elements (geometric), keeping `keep` of them.
template <typename T>
hipError_t grow(T*& p, int64_t& cap, int64_t need, int64_t keep, hipStream_t s) {
  if (need <= cap) return hipSuccess;
  int64_t nc = cap > 0 ? cap + cap / 2 : 1024;
  if (nc < need) nc = need;
  T* q = nullptr;
  hipError_t e = hipMalloc(&q, sizeof(T) * size_t(nc));
  if (e != hipSuccess) return e;
  if (p && keep > 0) {
    e = hipMemcpyAsync(q, p, sizeof(T) * size_t(keep), hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) { (void)hipFree(q); return e; }
  }
  if (p) (void)hipFree(p);
  p = q;
  cap = nc;
  return hipSuccess;
}

int store_fail(nalar_store* st, hipError_t e, const char* what) {
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  return policy_fail(st->h, e == hipErrorOutOfMemory ? NALAR_ENOMEM : NALAR_EDEVICE, m.c_str());
}

template <typename T>
hipError_t copy_in(T* dst, const T* src, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return hipMemcpyAsync(dst, src, sizeof(T) * size_t(n), hipMemcpyDeviceToDevice, s);
}

// The incremental buffers for every stored future (rem keeps what the last
// pass computed).
int ensure_incremental(nalar_store* st) {
  hipError_t e = hipSetDevice(policy_device(st->h));
  if (e != hipSuccess) return store_fail(st, e, "hipSetDevice");
  hipStream_t s = policy_stream(st->h);
  if (!st->ic) {
    e = hipMalloc(&st->ic, sizeof(IncCtrl));
    if (e != hipSuccess) return store_fail(st, e, "store incremental");
  }
  const int64_t need = st->N > 0 ? st->N : 1;
  if (need <= st->capI) return NALAR_OK;
  int64_t nc = st->capI > 0 ? st->capI + st->capI / 2 : 1024;
  if (nc < need) nc = need;
  int64_t c;
  c = st->capI; e = grow(st->rem, c, nc, st->rem_valid ? st->n_prev : 0, s);
  if (e == hipSuccess) { c = st->capI / 32 + 1; e = grow(st->fl, c, nc / 32 + 1, 0, s); }
  if (e == hipSuccess) { c = st->capI; e = grow(st->mxA, c, nc, 0, s); }
  if (e == hipSuccess) { c = st->capI; e = grow(st->cntA, c, nc + 32, 0, s); }  // whole words of 32
  if (e == hipSuccess) { c = st->capI; e = grow(st->light, c, nc, 0, s); }
  if (e == hipSuccess) { c = st->capI; e = grow(st->heavy, c, nc, 0, s); }
  if (e == hipSuccess) { c = st->capI / 64 + 1; e = grow(st->rbits, c, nc / 64 + 1, 0, s); }
  if (e != hipSuccess) {
    st->rem_valid = false;
    return store_fail(st, e, "store incremental");
  }
  st->capI = nc;
  return NALAR_OK;
}

}  // namespace

extern "C" {

int nalar_store_create(nalar_policy* h, nalar_store** out) {
  if (out) *out = nullptr;
  if (!h || !out) return NALAR_EINVAL;
  nalar_store* st = new (std::nothrow) nalar_store();
  if (!st) return NALAR_ENOMEM;
  st->h = h;
  hipError_t e = hipSetDevice(policy_device(h));
  if (e == hipSuccess)
    e = hipHostMalloc(reinterpret_cast<void**>(&st->bad), sizeof(uint32_t), hipHostMallocCoherent);
  if (e != hipSuccess) {
    delete st;
    return policy_fail(h, NALAR_ENOMEM, "hipHostMalloc(store flag)");
  }
  *st->bad = 0;
  *out = st;
  return NALAR_OK;
}

void nalar_store_destroy(nalar_store* st) {
  if (!st) return;
  (void)hipSetDevice(policy_device(st->h));
  (void)hipStreamSynchronize(policy_stream(st->h));
  for (void* p : {static_cast<void*>(st->wf), static_cast<void*>(st->type), static_cast<void*>(st->est),
                  static_cast<void*>(st->done), static_cast<void*>(st->loc), static_cast<void*>(st->att), static_cast<void*>(st->dep_off),
                  static_cast<void*>(st->dep_idx), static_cast<void*>(st->deadline),
                  static_cast<void*>(st->inst_type), static_cast<void*>(st->inst_load),
                  static_cast<void*>(st->inst_speed), static_cast<void*>(st->rem), static_cast<void*>(st->fl),
                  static_cast<void*>(st->mxA), static_cast<void*>(st->cntA), static_cast<void*>(st->light),
                  static_cast<void*>(st->heavy), static_cast<void*>(st->rbits), static_cast<void*>(st->ic),
                  static_cast<void*>(st->hv), static_cast<void*>(st->rheavy), static_cast<void*>(st->hv_n),
                  static_cast<void*>(st->log)})
    if (p) (void)hipFree(p);
  if (st->bad) (void)hipHostFree(st->bad);
  delete st;
}

int nalar_store_append(nalar_store* st, int64_t n_new, int64_t n_new_edges, const int32_t* wf,
                       const int32_t* type, const int64_t* est_us, const uint8_t* done,
                       const int32_t* loc, const int32_t* dep_off, const int32_t* dep_idx,
                       uint32_t flags) {
  if (!st) return NALAR_EINVAL;
  if (n_new < 0 || n_new_edges < 0 || (flags & ~NALAR_WF_CONTIGUOUS) != 0 ||
      st->N + n_new > NALAR_MAX_NODES || st->E + n_new_edges > NALAR_MAX_EDGES ||
      (n_new == 0 && n_new_edges != 0))
    return policy_fail(st->h, NALAR_EINVAL, "store append: sizes or flags out of range");
  if (n_new > 0 && (!wf || !type || !est_us || !done || !loc || !dep_off))
    return policy_fail(st->h, NALAR_EINVAL, "store append: NULL node array");
  if (n_new_edges > 0 && !dep_idx) return policy_fail(st->h, NALAR_EINVAL, "store append: NULL dep_idx");
  hipError_t e = hipSetDevice(policy_device(st->h));
  if (e != hipSuccess) return store_fail(st, e, "hipSetDevice");
  hipStream_t s = policy_stream(st->h);
  const int64_t N = st->N, E = st->E, need = N + n_new;
  if (need > st->capN) {  // every node array to the same new capacity
    int64_t nc = st->capN > 0 ? st->capN + st->capN / 2 : 1024;
    if (nc < need) nc = need;
    int64_t c0;
    c0 = st->capN; e = grow(st->wf, c0, nc, N, s);
    if (e == hipSuccess) { c0 = st->capN; e = grow(st->type, c0, nc, N, s); }
    if (e == hipSuccess) { c0 = st->capN; e = grow(st->est, c0, nc, N, s); }
    if (e == hipSuccess) { c0 = st->capN; e = grow(st->done, c0, nc, N, s); }
    if (e == hipSuccess) { c0 = st->capN; e = grow(st->loc, c0, nc, N, s); }
    if (e == hipSuccess) { c0 = st->capN; e = grow(st->att, c0, nc, N, s); }
    if (e == hipSuccess) { c0 = st->capN + 1; e = grow(st->dep_off, c0, nc + 1, N + 1, s); }
    if (e != hipSuccess) return store_fail(st, e, "store grow");
    st->capN = nc;
  }
  if (E + n_new_edges > st->capE) {
    e = grow(st->dep_idx, st->capE, E + n_new_edges, E, s);
    if (e != hipSuccess) return store_fail(st, e, "store grow");
  }
  if (N == 0) {  // dep_off[0] = 0
    const int32_t zero = 0;
    e = hipMemcpyAsync(st->dep_off, &zero, sizeof(int32_t), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return store_fail(st, e, "store init");
  }
  {  // room for every future of more than kIncHeavy dependencies
    const int64_t need_h = (E + n_new_edges) / (kIncHeavy + 1) + 1;
    if (!st->hv_n) {  // (kept only once its clearing is enqueued)
      uint32_t* count = nullptr;
      e = hipMalloc(&count, sizeof(uint32_t));
      if (e == hipSuccess) e = launch_inc_clear(s, count, 1);
      if (e != hipSuccess) {
        if (count) (void)hipFree(count);
        return store_fail(st, e, "store grow");
      }
      st->hv_n = count;
    }
    if (need_h > st->capH) {
      int64_t c0 = st->capH;
      e = grow(st->rheavy, c0, need_h, 0, s);
      if (e == hipSuccess) e = grow(st->hv, st->capH, need_h, st->capH, s);
      if (e != hipSuccess) return store_fail(st, e, "store grow");
    }
  }
  if (n_new > 0) {
    const AppendArgs aa{st->wf + N, st->type + N, st->est + N, st->done + N, st->loc + N, st->dep_off + N,
                        st->dep_idx + E, wf, type, est_us, done, loc, dep_off, dep_idx, n_new, n_new_edges,
                        int32_t(E), st->bad, st->att + N, int32_t(N), st->hv, st->hv_n, st->capH};
    hipLaunchKernelGGL(k_store_append, dim3(grid_for(n_new > n_new_edges ? n_new : n_new_edges)),
                       dim3(kStoreThreads), 0, s, aa);
    e = hipGetLastError();
    if (e != hipSuccess) return store_fail(st, e, "store append");
  }
  st->N = need;
  st->E = E + n_new_edges;
  st->contiguous = st->contiguous && (flags & NALAR_WF_CONTIGUOUS);
  // the per-future buffers of the next pass grow here, with the store, and
  // not inside the pass
  int rc = ensure_incremental(st);
  if (rc == NALAR_OK) rc = policy_reserve(st->h, st->N, st->E, st->W);
  return rc;
}

int nalar_store_complete(nalar_store* st, int64_t n, const int32_t* ids) {
  if (!st) return NALAR_EINVAL;
  if (n < 0 || (n > 0 && !ids)) return policy_fail(st->h, NALAR_EINVAL, "store complete: bad arguments");
  if (n == 0) return NALAR_OK;
  hipError_t e = hipSetDevice(policy_device(st->h));
  if (e != hipSuccess) return store_fail(st, e, "hipSetDevice");
  hipStream_t s = policy_stream(st->h);
  // the completed ids seed the next incremental pass (more completions than
  // futures: the next pass is a full one)
  const bool keep = st->n_log + n <= NALAR_MAX_NODES;
  if (!keep) {
    st->rem_valid = false;
    st->n_log = 0;
  } else {
    e = grow(st->log, st->capLog, st->n_log + n, st->n_log, s);
    if (e != hipSuccess) return store_fail(st, e, "store complete log");
  }
  hipLaunchKernelGGL(k_store_complete, dim3(grid_for(n)), dim3(kStoreThreads), 0, s, st->done,
                     keep ? st->log + st->n_log : nullptr, ids, n, st->N, st->bad);
  e = hipGetLastError();
  if (e != hipSuccess) return store_fail(st, e, "store complete");
  if (keep) st->n_log += n;
  return NALAR_OK;
}

int nalar_store_set_workflows(nalar_store* st, int64_t n_workflows, const int64_t* deadline_us) {
  if (!st) return NALAR_EINVAL;
  if (n_workflows < 0 || n_workflows > NALAR_MAX_WORKFLOWS || (n_workflows > 0 && !deadline_us))
    return policy_fail(st->h, NALAR_EINVAL, "store workflows: bad arguments");
  hipError_t e = hipSetDevice(policy_device(st->h));
  if (e == hipSuccess) e = grow(st->deadline, st->capW, n_workflows, 0, policy_stream(st->h));
  if (e == hipSuccess) e = copy_in(st->deadline, deadline_us, n_workflows, policy_stream(st->h));
  if (e != hipSuccess) return store_fail(st, e, "store workflows");
  st->W = n_workflows;
  return NALAR_OK;
}

int nalar_store_set_instances(nalar_store* st, int64_t n_instances, const int32_t* inst_type,
                              const int64_t* inst_load_us, const int32_t* inst_speed_permille) {
  if (!st) return NALAR_EINVAL;
  if (n_instances < 0 || n_instances > NALAR_MAX_INSTANCES ||
      (n_instances > 0 && (!inst_type || !inst_load_us || !inst_speed_permille)))
    return policy_fail(st->h, NALAR_EINVAL, "store instances: bad arguments");
  hipStream_t s = policy_stream(st->h);
  hipError_t e = hipSetDevice(policy_device(st->h));
  int64_t c1 = st->capM, c2 = st->capM;
  if (e == hipSuccess) e = grow(st->inst_type, st->capM, n_instances, 0, s);
  if (e == hipSuccess) e = grow(st->inst_load, c1, n_instances, 0, s);
  if (e == hipSuccess) e = grow(st->inst_speed, c2, n_instances, 0, s);
  if (e == hipSuccess) e = copy_in(st->inst_type, inst_type, n_instances, s);
  if (e == hipSuccess) e = copy_in(st->inst_load, inst_load_us, n_instances, s);
  if (e == hipSuccess) e = copy_in(st->inst_speed, inst_speed_permille, n_instances, s);
  if (e != hipSuccess) return store_fail(st, e, "store instances");
  st->M = n_instances;
  return NALAR_OK;
}

int64_t nalar_store_n_nodes(const nalar_store* st) { return st ? st->N : -1; }

int nalar_store_pass(nalar_store* st, int64_t now_us, int64_t migration_cost_us, uint32_t policy,
                     nalar_result* r) {
  if (!st) return NALAR_EINVAL;
  if ((policy & ~(NALAR_ORDER_LPT | NALAR_ORDER_SRTF | NALAR_ROUTE_STATEFUL | NALAR_ROUTE_GREEDY)) != 0)
    return policy_fail(st->h, NALAR_EINVAL, "store pass: unknown policy bits");
  nalar_problem p;
  std::memset(&p, 0, sizeof(p));
  p.n_nodes = st->N;
  p.n_edges = st->E;
  p.n_workflows = st->W;
  p.n_instances = st->M;
  p.now_us = now_us;
  p.migration_cost_us = migration_cost_us;
  p.flags = (st->contiguous ? NALAR_WF_CONTIGUOUS : 0u) | policy;
  p.wf = st->wf;
  p.type = st->type;
  p.est_us = st->est;
  p.done = st->done;
  p.loc = st->loc;
  p.dep_off = st->dep_off;
  p.dep_idx = st->dep_idx;
  p.deadline_us = st->deadline;
  p.inst_type = st->inst_type;
  p.inst_load_us = st->inst_load;
  p.inst_speed_permille = st->inst_speed;
  int rc = ensure_incremental(st);
  if (rc != NALAR_OK) return rc;
  st->last_incremental = 0;
  // a malformed append or completion since the last pass fails this one (the
  // pass has synchronised the stream, so every such call has been counted; the
  // host never writes the counter)
  auto bad_calls = [st]() {
    const uint32_t bad = __atomic_load_n(st->bad, __ATOMIC_ACQUIRE);
    const bool b = bad != st->bad_seen;
    st->bad_seen = bad;
    return b;
  };
  rc = kIncFallback;
  if (!st->incremental) st->last_fallback = NALAR_STORE_FULL_DISABLED;
  else if (!st->rem_valid || !r) st->last_fallback = NALAR_STORE_FULL_NO_STATE;
  else if (st->W < st->W_prev || st->M < st->M_prev) st->last_fallback = NALAR_STORE_FULL_SHRUNK;
  else {
    IncStore is{st->n_prev, st->log, st->n_log, st->rem, st->fl, st->mxA, st->cntA, st->light,
                      st->heavy, st->att, st->rbits, st->hv, st->hv_n, st->capH, st->rheavy, st->ic,
                st->rounds};
    rc = policy_pass_incremental(st->h, &p, r, is);
    st->rounds = is.rounds;
    if (!inc_fallback(rc)) st->last_incremental = 1;
    st->last_fallback = rc == kIncFallback ? NALAR_STORE_FULL_NO_SPLITTERS
                      : rc == kIncFallbackOverflow ? NALAR_STORE_FULL_OVERFLOW
                      : rc == kIncFallbackRounds ? NALAR_STORE_FULL_ROUNDS : 0;
  }
  if (inc_fallback(rc)) {  // a full pass, its rem kept for the next one
    nalar_result r2{};
    if (r) r2 = *r;
    r2.rem_us = st->rem;
    policy_split_any(st->h, true);
    rc = nalar_policy_pass(st->h, &p, r ? &r2 : nullptr);
    policy_split_any(st->h, false);
    if (r) r->n_ready = r2.n_ready;
    if (rc == NALAR_OK && r && r->rem_us && st->N > 0) {
      hipError_t e = hipMemcpyAsync(r->rem_us, st->rem, sizeof(int64_t) * size_t(st->N), hipMemcpyDeviceToDevice,
                                    policy_stream(st->h));
      if (e == hipSuccess) e = hipStreamSynchronize(policy_stream(st->h));
      if (e != hipSuccess) rc = store_fail(st, e, "store rem");
    }
  }
  const bool bad = bad_calls();
  st->hv_stale |= bad;
  if (rc == NALAR_OK && !bad && st->hv_stale && st->N > 0) {
    // (a full pass: the bad call's had no rem to leave)
    hipStream_t s = policy_stream(st->h);
    hipError_t e = launch_inc_clear(s, st->hv_n, 1);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_store_heavy, dim3(grid_for(st->N)), dim3(kStoreThreads), 0, s, st->dep_off, st->N, st->hv,
                         st->hv_n, st->capH);
      e = hipGetLastError();
    }
    if (e != hipSuccess) rc = store_fail(st, e, "store heavy list");
    else st->hv_stale = false;
  }
  st->rem_valid = rc == NALAR_OK && !bad;
  st->n_prev = st->N;
  st->W_prev = st->W;
  st->M_prev = st->M;
  st->n_log = 0;
  if (bad) return policy_fail(st->h, NALAR_EINVAL, "a completed id was out of range, or appended offsets malformed");
  return rc;
}

int nalar_store_set_incremental(nalar_store* st, int enable) {
  if (!st) return NALAR_EINVAL;
  st->incremental = enable != 0;
  return NALAR_OK;
}

int nalar_store_last_pass_incremental(const nalar_store* st) { return st ? st->last_incremental : -1; }

int nalar_store_last_fallback(const nalar_store* st) { return st ? st->last_fallback : -1; }

}  // extern "C"
