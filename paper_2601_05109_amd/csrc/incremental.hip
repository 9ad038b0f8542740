// Incremental pass over the graph store.  Between two passes the store only
// changes by deltas (Section 4.3.1: futures created with their dependencies,
// values materialising): futures appended, futures marked done.  A future's
// remaining critical path rem(v) = est'(v) + max over its consumers c of
// rem(c) (est' = 0 once done) depends only on v and its descendants, so after
// a delta it can change only for the changed futures (the seeds: appended or
// completed since the last pass) and their ancestors (every future a seed
// depends on, transitively): the closure.  Everything else keeps the rem of
// the last pass, persisted in the store.
//
// The pass, after validating the appended futures (k_nodes over the appended
// range):
//   1. closure: from every seed, its dependencies are marked (one bit per
//      future) and visited in turn;
//   2. scan (every future, O(N + E)): readiness (not done, every dependency
//      done) as one bit per future; for a closure member, one count per
//      dependency (its consumers inside the closure); for a future outside
//      the closure, its unchanged rem pushed to each dependency inside the
//      closure (max);
//   3. sweep of the closure: the members without closure consumers listed,
//      then a member whose closure consumers are all finalised takes rem =
//      est' + max, and pushes it to its dependencies;
//   4. the ready futures keyed, routed and dropped into the bins of the
//      partition sort (the splitters of the previous pass), which then orders
//      them by (key, wf, id).
// Steps 1 and 3 let a thread follow a chain of single dependencies itself (the
// common shape: a future created as the child of one future), so a chain of
// any length costs one launch; a future with several new dependencies hands
// all but one to its workgroup's LDS queue, and a future with more than
// kIncHeavy dependencies goes to a second LDS queue whose futures the whole
// workgroup expands together; the workgroup drains both before it ends.  A
// full queue spills into the next round's lists.  Of the kIncRounds rounds the
// first one to three get a launch each and one workgroup runs the others in one
// launch; work left after the last round makes the pass fall back to a full
// pass (kStIncomplete).
#include "internal.hpp"

namespace nalar {

namespace {

constexpr int kIncThreads = 256;
constexpr int kIncTail = 3;       // rounds from here on always run in one workgroup (k_inc_*_tail)
constexpr int kIncTailThreads = 1024;
constexpr int kScanPer = 8;       // futures per thread in the scan (kIncThreads apart)

// A future's flags: closure membership and done, one bit of each word of a pair.
__device__ inline bool bit_set_new(uint2* fl, int32_t v) {
  const uint32_t m = 1u << (uint32_t(v) & 31u);
  return (atomicOr(&fl[uint32_t(v) >> 5].x, m) & m) == 0u;
}

__device__ inline bool bit_of(uint32_t word, int32_t v) { return ((word >> (uint32_t(v) & 31u)) & 1u) != 0u; }
__device__ inline bool done_get(const uint2* fl, int32_t v) { return bit_of(fl[uint32_t(v) >> 5].y, v); }

// One atomic of a workgroup into one of the spread words of a counter.
__device__ inline void add_part(uint32_t* parts, uint32_t x) {
  if (x) atomicAdd(&parts[blockIdx.x & (kIncParts - 1)], x);
}

// A round's count, read where the atomics that wrote it are coherent (the
// tail kernel reads counts its own earlier rounds wrote).
__device__ inline uint32_t ld_count(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Start of round r's items in a list whose rounds are appended one after the
// other (counts of rounds 0 .. r-1, stable once round r runs).
__device__ inline uint32_t round_base(const uint32_t* cnt, int r) {
  uint32_t b = 0;
  for (int i = 0; i < r; ++i) b += ld_count(&cnt[i]);
  return b;
}

__device__ inline void push_round(int32_t* list, uint32_t* cnt, int r, int32_t v) {
  if (r > kIncRounds) return;  // cannot happen: rounds past the last are never appended to
  const uint32_t at = round_base(cnt, r) + atomicAdd(&cnt[r], 1u);
  list[at] = v;
}

// Appends the lanes' futures with one atomic per workgroup: thread t holds the
// futures first + j for the set bits j of mask (every thread of the workgroup
// calls).  s_tmp holds one word per wave and two more.
__device__ inline void push_block(uint64_t mask, int64_t first, int32_t* list, uint32_t* n, uint32_t base,
                                  uint32_t* s_tmp) {
  const int nw = int(blockDim.x) / kWave;
  const int wv = int(threadIdx.x) / kWave;
  const uint32_t k = uint32_t(__popcll(mask));
  const uint32_t inc = wave_incl_scan_u32(k);
  if (lane_id() == kWave - 1) s_tmp[wv] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    off += w < wv ? s_tmp[w] : 0u;
    tot += s_tmp[w];
  }
  if (threadIdx.x == 0) s_tmp[nw] = tot ? atomicAdd(n, tot) : 0u;
  __syncthreads();
  uint32_t at = base + s_tmp[nw] + off + inc - k;
  while (mask) {
    list[at++] = int32_t(first + __builtin_ctzll(mask));
    mask &= mask - 1;
  }
  __syncthreads();  // s_tmp is free again
}

// One future (or none) per thread, appended as push_block does.
__device__ inline void push_block1(bool in, int32_t v, int32_t* list, uint32_t* n, uint32_t base,
                                   uint32_t* s_tmp) {
  push_block(in ? 1u : 0u, v, list, n, base, s_tmp);
}

__device__ inline void flag(Ctrl* c, uint32_t bits) {
  __hip_atomic_fetch_or(&c->status_sweep, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A dependency d of closure member u, checked: in range and not u itself;
// for an appended future (u >= n_prev, never validated before) also of u's
// workflow.
__device__ inline bool dep_ok(const IncArgs& a, int32_t u, int32_t d) {
  if (d < 0 || int64_t(d) >= a.p.N) {
    flag(a.ctrl, kStInval);
    return false;
  }
  if (d == u) {
    flag(a.ctrl, kStCycle);
    return false;
  }
  if (int64_t(u) >= a.n_prev && a.p.wf[d] != a.p.wf[u]) {
    flag(a.ctrl, kStInval);
    return false;
  }
  return true;
}

__device__ inline void join(const IncArgs& a, int32_t d) {
  a.mxA[d] = 0;
  a.cntA[d] = 0;
}

// A workgroup's queues of futures to continue from (LDS): single ones and
// heavy ones; past a queue's capacity a future goes to the next round's list
// instead.
constexpr int kIncQueue = 2048;
constexpr int kIncHeavyQueue = 64;

struct WgQueue {
  int32_t* q;       // [kIncQueue]
  int* n;
  int32_t* hq;      // [kIncHeavyQueue]
  int* hn;
  uint32_t* tmp;    // [waves + 2] for push_block
  int* htaken;      // heavy futures this workgroup kept (at most kIncHeavyKeep)
  bool keep_all;    // one workgroup for every round left: keep every heavy future
};

__device__ inline void wg_push(const WgQueue& wq, int32_t* list, uint32_t* cnt, int round, int32_t v) {
  const int at = atomicAdd(wq.n, 1);
  if (at < kIncQueue) wq.q[at] = v;
  else push_round(list, cnt, round + 1, v);
}

// A workgroup expands heavy futures itself while its queue has room, but at
// most kIncHeavyKeep of those with more than kIncHugeDeps dependencies (a
// reduction over thousands of futures); the others go to the next round,
// whose workgroups expand them side by side.
constexpr int kIncHeavyKeep = 1;
constexpr int kIncHugeDeps = 1024;

__device__ inline void wg_push_heavy(const WgQueue& wq, int32_t* list, uint32_t* cnt, int round, int32_t v,
                                     int32_t deg) {
  if (wq.keep_all || deg <= kIncHugeDeps || atomicAdd(wq.htaken, 1) < kIncHeavyKeep) {
    const int at = atomicAdd(wq.hn, 1);
    if (at < kIncHeavyQueue) {
      wq.hq[at] = v;
      return;
    }
  }
  push_round(list, cnt, round + 1, v);
}

// ------------------------------------------------------------------ closure

// Marks the lanes' dependencies d (d < 0: none) with one atomic per group of
// lanes holding the same d (a fan-in: many consumers of one future walking
// at once), else one per lane; returns whether this lane made d a member
// (one lane per d).  Every lane of the wave calls.
__device__ inline bool wave_mark(uint2* bits, int32_t d) {
  uint64_t pend = ballot(d >= 0);
  bool fresh = false;
  for (int it = 0; it < 2 && pend != 0; ++it) {
    const int lead = __builtin_ctzll(pend);
    const int32_t t = readlane_i32(d, lead);
    const uint64_t grp = ballot(((pend >> lane_id()) & 1u) && d == t);
    if (__popcll(grp) < 2) break;
    if (lane_id() == lead) fresh = bit_set_new(bits, t);
    pend &= ~grp;
  }
  if ((pend >> lane_id()) & 1u) fresh = bit_set_new(bits, d);
  return fresh;
}

// u has just joined the closure: visit its dependencies, following the chain
// while exactly one of them is new.  Every lane of the wave calls (u = -1:
// nothing), so that the lanes whose single dependency is one future mark it
// together.
__device__ void close_walk(const IncArgs& a, int32_t u, int round, const WgQueue& wq) {
  while (ballot(u >= 0) != 0) {
    int32_t d1 = -1;  // the one dependency of a single-dependency future
    if (u >= 0) {
      const int32_t o0 = a.p.dep_off[u], o1 = a.p.dep_off[u + 1];
      if (o1 - o0 > kIncHeavy) {
        wg_push_heavy(wq, a.heavy, a.ic->ch, round, u, o1 - o0);
        u = -1;
      } else if (o1 - o0 == 1) {
        const int32_t d = a.p.dep_idx[o0];
        if (dep_ok(a, u, d)) d1 = d;
        u = -1;
      } else {
        int32_t next = -1;
        for (int32_t e = o0; e < o1; ++e) {
          const int32_t d = a.p.dep_idx[e];
          if (!dep_ok(a, u, d)) continue;
          if (bit_set_new(a.fl, d)) {
            join(a, d);
            if (next < 0) next = d;
            else wg_push(wq, a.light, a.ic->cl, round, d);
          }
        }
        u = next;
      }
    }
    if (wave_mark(a.fl, d1)) {
      join(a, d1);
      u = d1;
    }
  }
}

// Drains the workgroup's queues (every thread of the workgroup calls): a heavy
// future is expanded by the whole workgroup (expand(v) on every thread), else
// up to one single future per thread is taken from the top, until both are
// empty.
template <typename Walk, typename Expand>
__device__ void wg_drain(const WgQueue& wq, Walk walk, Expand expand) {
  for (;;) {
    __syncthreads();
    const int hc = *wq.hn, c = *wq.n;
    const int hn = hc < kIncHeavyQueue ? hc : kIncHeavyQueue;
    const int n = c < kIncQueue ? c : kIncQueue;
    if (hn == 0 && n == 0) break;  // the same on every thread
    if (hn > 0) {
      const int32_t h = wq.hq[hn - 1];
      __syncthreads();
      if (threadIdx.x == 0) *wq.hn = hn - 1;
      __syncthreads();
      expand(h);
      continue;
    }
    int32_t mine = -1;
    if (int(threadIdx.x) < n) mine = wq.q[n - 1 - int(threadIdx.x)];
    __syncthreads();
    if (threadIdx.x == 0) *wq.n = n > int(blockDim.x) ? n - int(blockDim.x) : 0;
    __syncthreads();
    walk(mine);  // every lane: the walks work wave by wave
  }
}

// A heavy member's dependencies visited by the whole workgroup; the new
// members go to the next round, where every workgroup shares their walks.
__device__ inline void close_expand(const IncArgs& a, int32_t u, int round, const WgQueue& wq) {
  const int32_t o0 = a.p.dep_off[u], o1 = a.p.dep_off[u + 1];
  for (int32_t e0 = o0; e0 < o1; e0 += int32_t(blockDim.x)) {
    const int32_t e = e0 + int32_t(threadIdx.x);
    bool fresh = false;
    int32_t d = -1;
    if (e < o1) {
      d = a.p.dep_idx[e];
      if (dep_ok(a, u, d) && bit_set_new(a.fl, d)) {
        join(a, d);
        fresh = true;
      }
    }
    const int rn = round + 1 <= kIncRounds ? round + 1 : kIncRounds;
    push_block1(fresh, d, a.light, &a.ic->cl[rn], round_base(a.ic->cl, rn), wq.tmp);
  }
}

// Every kernel leaves the snapshot alone once validation has failed (the
// dependency offsets of the appended futures are trusted only then).
__device__ inline bool invalid(const IncArgs& a) { return a.ctrl->status != 0; }

// Round 0 takes the seeds (completed ids of the log, then the appended
// range); round r >= 1 the futures handed on: heavy ones expanded one per
// workgroup, the others one per thread.  Then the workgroup drains its queue.
// One round of the closure, this workgroup's share of it (every thread of the
// workgroup calls; the workgroup's queues are empty on entry and on return).
__device__ void close_round(const IncArgs& a, int r, const WgQueue& wq) {
  const uint32_t nh = r ? ld_count(&a.ic->ch[r]) : 0u, nl = r ? ld_count(&a.ic->cl[r]) : 0u;
  const int64_t n_app = a.p.N - a.n_prev;
  const int64_t n_seed = r ? 0 : a.n_log + (n_app > 0 ? n_app : 0);
  if (nh == 0 && nl == 0 && n_seed == 0) return;  // the same on every thread
  if (threadIdx.x == 0) {
    *wq.n = 0;
    *wq.hn = 0;
    *wq.htaken = 0;
  }
  __syncthreads();
  // every lane of a wave runs each iteration (the walks work wave by wave)
  for (int64_t i0 = int64_t(blockIdx.x) * blockDim.x; i0 < n_seed; i0 += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    int32_t v = -1;
    if (i < n_seed) {
      if (i >= a.n_log) {  // appended: already members (the pack)
        v = int32_t(a.n_prev + (i - a.n_log));
        join(a, v);
      } else {
        const int32_t c = a.log[i];
        // an id out of range is counted by the completion kernel
        if (c >= 0 && int64_t(c) < a.p.N && bit_set_new(a.fl, c)) {
          join(a, c);
          v = c;
        }
      }
    }
    close_walk(a, v, r, wq);
  }
  const uint32_t bh = round_base(a.ic->ch, r), bl = round_base(a.ic->cl, r);
  for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) close_expand(a, a.heavy[bh + h], r, wq);
  for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < nl; i0 += gridDim.x * blockDim.x) {
    const uint32_t i = i0 + threadIdx.x;
    close_walk(a, i < nl ? a.light[bl + i] : -1, r, wq);
  }
  wg_drain(wq, [&](int32_t v) { close_walk(a, v, r, wq); }, [&](int32_t v) { close_expand(a, v, r, wq); });
}

// The workgroup's LDS queues.
#define NALAR_INC_QUEUES(threads, keep)                                         \
  __shared__ int32_t s_q[kIncQueue], s_hq[kIncHeavyQueue];                      \
  __shared__ int s_n, s_hn, s_htaken;                                           \
  __shared__ uint32_t s_tmp[(threads) / kWave + 2];                             \
  const WgQueue wq{s_q, &s_n, s_hq, &s_hn, s_tmp, &s_htaken, keep}

__global__ __launch_bounds__(kIncThreads) void k_inc_close(IncArgs a, int r) {
  if (invalid(a)) return;
  NALAR_INC_QUEUES(kIncThreads, false);
  close_round(a, r, wq);
}

// Rounds r0 .. kIncRounds - 1 by one workgroup (they are usually empty, and one
// launch costs less than one per round).  What a round hands on is read by the
// same workgroup in the next one.
__global__ __launch_bounds__(kIncTailThreads) void k_inc_close_tail(IncArgs a, int r0) {
  if (invalid(a)) return;
  NALAR_INC_QUEUES(kIncTailThreads, true);
  for (int r = r0; r < kIncRounds; ++r) {
    close_round(a, r, wq);
    __syncthreads();
  }
}

// --------------------------------------------------------------------- scan

// Pending pushes of one lane to one dependency: merged while the target
// repeats (children of one future are appended next to one another).
struct Pend {
  int32_t d = -1;
  int64_t v = 0;
};

__device__ inline void flush_max(int64_t* mx, Pend& p) {
  if (p.d >= 0) atomicMax(reinterpret_cast<long long*>(&mx[p.d]), (long long)p.v);
  p.d = -1;
}

__device__ inline void flush_cnt(int32_t* cnt, Pend& p) {
  if (p.d >= 0) atomicAdd(&cnt[p.d], int32_t(p.v));
  p.d = -1;
}

// The last pushes of a wave: one atomic when every lane holds the same target.
__device__ inline void flush_wave_max(int64_t* mx, Pend& p) {
  const uint64_t act = ballot(p.d >= 0);
  if (act == 0) return;
  const int lead = __builtin_ctzll(act);
  const int32_t first = readlane_i32(p.d, lead);
  if ((act & (act - 1)) != 0 && ballot(p.d >= 0 && p.d != first) == 0) {
    const int64_t m = wave_max_i64(p.d >= 0 ? p.v : INT64_MIN);
    if (lane_id() == lead) atomicMax(reinterpret_cast<long long*>(&mx[first]), (long long)m);
    p.d = -1;
    return;
  }
  flush_max(mx, p);
}

__device__ inline void flush_wave_cnt(int32_t* cnt, Pend& p) {
  const uint64_t act = ballot(p.d >= 0);
  if (act == 0) return;
  const int lead = __builtin_ctzll(act);
  const int32_t first = readlane_i32(p.d, lead);
  if ((act & (act - 1)) != 0 && ballot(p.d >= 0 && p.d != first) == 0) {
    const int64_t s = wave_sum_i64(p.d >= 0 ? p.v : 0);
    if (lane_id() == lead) atomicAdd(&cnt[first], int32_t(s));
    p.d = -1;
    return;
  }
  flush_cnt(cnt, p);
}

// The futures with more than kIncHeavy dependencies, one per workgroup at a
// time.
__device__ void scan_heavy(const IncArgs& a, uint32_t first, uint32_t step) {
  __shared__ int s_blocked;
  constexpr int U = 4;  // dependencies a thread keeps in flight
  const uint32_t nh = uint32_t(int64_t(*a.hv_n) < a.hv_cap ? *a.hv_n : uint32_t(a.hv_cap));
  for (uint32_t h = first; h < nh; h += step) {
    const int32_t v = a.hv[h];
    if (threadIdx.x == 0) s_blocked = 0;
    __syncthreads();
    const uint2 f = a.fl[uint32_t(v) >> 5];
    const bool in = bit_of(f.x, v);
    const int32_t o0 = a.p.dep_off[v], o1 = a.p.dep_off[v + 1];
    bool blocked = false;
    int64_t rv = 0;
    if (!in && int64_t(v) < a.n_prev) rv = a.rem[v];
    for (int32_t e0 = o0 + int32_t(threadIdx.x); e0 < o1; e0 += U * kIncThreads) {
      int32_t d[U];
      uint2 w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t e = e0 + u * kIncThreads;
        d[u] = e < o1 ? a.p.dep_idx[e] : -1;
        if (int64_t(d[u]) >= a.p.N) d[u] = -1;  // reported by the closure or an earlier pass
      }
#pragma unroll
      for (int u = 0; u < U; ++u) w[u] = a.fl[d[u] >= 0 ? uint32_t(d[u]) >> 5 : 0u];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (d[u] < 0) continue;
        blocked |= !bit_of(w[u].y, d[u]);
        if (in) atomicAdd(&a.cntA[d[u]], 1);
        else if (bit_of(w[u].x, d[u])) atomicMax(reinterpret_cast<long long*>(&a.mxA[d[u]]), (long long)rv);
      }
    }
    if (blocked) s_blocked = 1;
    __syncthreads();
    if (threadIdx.x == 0) {
      if (in) add_part(a.ic->a_n, 1u);
      if (!bit_of(f.y, v) && s_blocked == 0) a.rheavy[atomicAdd(&a.ic->r_heavy, 1u)] = v;
    }
    __syncthreads();
  }
}

// The first hb workgroups take the futures of many dependencies (a list the
// appends keep).  The others take kScanPer x kIncThreads consecutive futures
// at a time, thread t the futures t, t + kIncThreads, ... of them (so every
// load of a wave is coalesced), and issue the loads of all of them together,
// stage by stage (offsets and flags; the first dependency; its flags), so that
// the gathers of a thread overlap; further dependencies (rare in the graphs
// this serves) are visited one by one after.  A thread's futures lie
// kIncThreads apart, so a run of futures with one common dependency (the
// children of a hub) still merges its pushes per lane.
//
// What bounds it is the atomics: what every workgroup adds to must not be one
// word.  The ready futures leave as one bit each, written per wave (a list
// cost one returning atomic per workgroup on its length, all queued on that
// word), and the member count goes to spread words.  At 12.4M futures 191 us,
// and 17 us for the futures of many dependencies, became 70 us together; at
// 1.3M 39 + 13 became 21.
__global__ __launch_bounds__(kIncThreads) void k_inc_scan(IncArgs a, int hb) {
  if (invalid(a)) return;
  if (int(blockIdx.x) < hb) {
    scan_heavy(a, blockIdx.x, uint32_t(hb));
    return;
  }
  __shared__ uint32_t s_members[kIncThreads / kWave];
  const int64_t N = a.p.N;
  const int ln = lane_id();
  const int wv = int(threadIdx.x) / kWave;
  Pend pm, pc;
  uint32_t members = 0;
  const int64_t step = int64_t(gridDim.x - hb) * kIncThreads * kScanPer;
  for (int64_t g0 = int64_t(int(blockIdx.x) - hb) * kIncThreads * kScanPer; g0 < N; g0 += step) {
    const int64_t v0 = g0 + int64_t(threadIdx.x);
    int32_t o0[kScanPer], o1[kScanPer], d0[kScanPer];
    uint2 f[kScanPer], df[kScanPer];
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      const int64_t v = v0 + int64_t(j) * kIncThreads;
      const int64_t vs = v < N ? v : N - 1;
      o0[j] = a.p.dep_off[vs];
      o1[j] = a.p.dep_off[vs + 1];
      f[j] = a.fl[vs >> 5];
    }
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      const bool one = o1[j] > o0[j] && o1[j] - o0[j] <= kIncHeavy;
      d0[j] = one ? a.p.dep_idx[o0[j]] : -1;
      if (int64_t(d0[j]) >= N) d0[j] = -1;
    }
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) df[j] = a.fl[d0[j] >= 0 ? uint32_t(d0[j]) >> 5 : 0u];
    uint64_t rword = 0;  // lane j: the ready bits of the wave's futures of item j
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      const int64_t v = v0 + int64_t(j) * kIncThreads;
      bool ready = false;
      if (v < N && o1[j] - o0[j] <= kIncHeavy) {
        const bool in = bit_of(f[j].x, int32_t(v));
        members += in ? 1u : 0u;
        bool blocked = false;
        int64_t rv = 0;
        bool have_rv = false;
        auto visit = [&](int32_t d, const uint2& w) {
          blocked |= !bit_of(w.y, d);
          if (in) {
            if (d != pc.d) {
              flush_cnt(a.cntA, pc);
              pc.d = d;
              pc.v = 0;
            }
            pc.v += 1;
          } else if (bit_of(w.x, d)) {
            if (!have_rv) {
              rv = a.rem[v];
              have_rv = true;
            }
            if (d != pm.d) {
              flush_max(a.mxA, pm);
              pm.d = d;
              pm.v = rv;
            }
            pm.v = rv > pm.v ? rv : pm.v;
          }
        };
        // (out of range: reported by the closure or an earlier pass.  The first
        // dependency, loaded above, has a visit of its own: choosing between it
        // and the loaded one inside the loop made the compiler keep the loaded
        // ones in scratch memory and read either through one pointer.)
        if (d0[j] >= 0) visit(d0[j], df[j]);
        for (int32_t e = o0[j] + 1; e < o1[j]; ++e) {
          const int32_t d = a.p.dep_idx[e];
          if (d >= 0 && int64_t(d) < N) visit(d, a.fl[uint32_t(d) >> 5]);
        }
        ready = !bit_of(f[j].y, int32_t(v)) && !blocked;
      }
      const uint64_t m = ballot(ready);
      rword = ln == j ? m : rword;
    }
    // the wave's word of item j covers futures g0 + j * kIncThreads + 64 wv ..
    const int64_t rw = (g0 + int64_t(ln) * kIncThreads + int64_t(wv) * kWave) / kWave;
    if (ln < kScanPer && rw * kWave < N) a.rbits[rw] = rword;
    // pushes still pending go out per wave, before the next tile's would push
    // them out lane by lane (a hub's children: 64 atomics queueing on one word)
    flush_wave_cnt(a.cntA, pc);
    flush_wave_max(a.mxA, pm);
  }
  const uint32_t mt = uint32_t(wave_sum_i64(int64_t(members)));
  if (ln == 0) s_members[wv] = mt;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int x = 0; x < kIncThreads / kWave; ++x) t += s_members[x];
    add_part(a.ic->a_n, t);
  }
}

// -------------------------------------------------------------------- sweep

// A device-scope max that is skipped when a plain read of the location
// already shows a value at least as large.  Within the sweep a member's max
// only grows (the closure zeroed it, the scan and the sweep only raise it),
// so a stale read is never above the true value and skipping stays exact; it
// saves a memory-side atomic whenever an earlier push was larger.  (In the
// scan the extra reads cost more than the atomics they save.)
__device__ inline void max_if_larger(int64_t* p, int64_t v) {
  if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
    __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One push of a finalised member: its rem into d's max, then d's count down
// by k; returns the count before.  Every access to the maxima and counts in
// the sweep is a device-scope atomic, so their values meet where such
// atomics are coherent, and the only order needed is the max before the
// count: the wait makes the max complete there before the count is touched,
// so the member that sees the count reach zero (and then loads the max
// atomically) sees every push.  No cache write-back or invalidation is
// needed: the only other access is the read that lets max_if_larger skip a
// max, and a stale value there is never above the true one.
__device__ inline int32_t push_count(const IncArgs& a, int32_t d, int64_t r, int32_t k) {
  max_if_larger(&a.mxA[d], r);
  __asm__ __volatile__("s_waitcnt vmcnt(0)" ::: "memory");
  return __hip_atomic_fetch_add(&a.cntA[d], -k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Pushes the lanes' rem r to their dependencies d (d < 0: none) with one
// pair of atomics per group of lanes holding the same d (a fan-in), else one
// pair per lane; returns whether this lane brought d's count to zero (one
// lane per d).  Every lane of the wave calls.
__device__ inline bool wave_push(const IncArgs& a, int32_t d, int64_t r) {
  uint64_t pend = ballot(d >= 0);
  bool zero = false;
  for (int it = 0; it < 2 && pend != 0; ++it) {
    const int lead = __builtin_ctzll(pend);
    const int32_t t = readlane_i32(d, lead);
    const bool in = ((pend >> lane_id()) & 1u) && d == t;
    const uint64_t grp = ballot(in);
    const int n = __popcll(grp);
    if (n < 2) break;
    const int64_t m = wave_max_i64(in ? r : INT64_MIN);
    if (lane_id() == lead) zero = push_count(a, t, m, n) == n;
    pend &= ~grp;
  }
  if ((pend >> lane_id()) & 1u) zero = push_count(a, d, r, 1) == 1;
  return zero;
}

// u's closure consumers are all finalised: rem(u) = est' + max, pushed to its
// dependencies; a dependency whose count reaches zero is finalised next (by
// this lane if it is the first, else through the workgroup's queue).  Every
// lane of the wave calls (u = -1: nothing).
__device__ void sweep_walk(const IncArgs& a, int32_t u, int round, uint32_t& fin, const WgQueue& wq) {
  while (ballot(u >= 0) != 0) {
    int32_t d1 = -1;  // the one dependency of a single-dependency future
    int64_t r = 0;
    if (u >= 0) {
      const int64_t est = done_get(a.fl, u) ? 0 : a.p.est[u];
      const int64_t m = __hip_atomic_load(&a.mxA[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      r = est + m;
      if (r > NALAR_REM_MAX) {
        r = NALAR_REM_MAX + 1;
        flag(a.ctrl, kStRange);
      }
      a.rem[u] = r;
      ++fin;
      const int32_t o0 = a.p.dep_off[u], o1 = a.p.dep_off[u + 1];
      if (o1 - o0 > kIncHeavy) {
        wg_push_heavy(wq, a.heavy, a.ic->sh, round, u, o1 - o0);
        u = -1;
      } else if (o1 - o0 == 1) {
        const int32_t d = a.p.dep_idx[o0];
        if (d >= 0 && int64_t(d) < a.p.N && d != u) d1 = d;
        u = -1;
      } else {
        int32_t next = -1;
        for (int32_t e = o0; e < o1; ++e) {
          const int32_t d = a.p.dep_idx[e];
          if (d < 0 || int64_t(d) >= a.p.N || d == u) continue;
          if (push_count(a, d, r, 1) == 1) {
            if (next < 0) next = d;
            else wg_push(wq, a.light, a.ic->sl, round, d);
          }
        }
        u = next;
      }
    }
    if (wave_push(a, d1, r)) u = d1;
  }
}

__device__ inline void add_fin(const IncArgs& a, uint32_t fin) {
  const int64_t t = wave_sum_i64(int64_t(fin));
  if (lane_id() == 0) add_part(a.ic->fin, uint32_t(t));
}

// The sweep's first round: every closure member without closure consumers,
// listed before any member is finalised (a walk may bring another member's
// count to zero while this list is taken, and that member is then the
// walker's).  A thread takes kFrontWords words of the membership bits and, where a
// word has members, loads all its 32 counts at once (one 128-byte line, in
// flight together; one member after another, a stretch of appended ids, every
// bit set, took 32 round trips).  A workgroup appends once, with one returning
// atomic on the list's length: they queue on that word, so it covers 64K futures.
//
// Measured and dropped: no list, but a count of one extra that the first round
// itself takes off each member.  Spread over all waves the members no longer
// share their pushes to a common dependency (a session's root), and those
// atomics, queueing on one word, took the round from 48 to 145 us at 12M futures.
constexpr int kFrontThreads = 1024;
constexpr int kFrontWords = 2;

__global__ __launch_bounds__(kFrontThreads) void k_inc_front0(IncArgs a) {
  if (invalid(a)) return;
  __shared__ uint32_t s_tmp[kFrontThreads / kWave + 2];
  const int64_t words = (a.p.N + 31) / 32;
  const int64_t step = int64_t(gridDim.x) * kFrontThreads * kFrontWords;
  // the loop runs the same number of times on every thread of the workgroup
  for (int64_t w0 = int64_t(blockIdx.x) * kFrontThreads * kFrontWords; w0 < words; w0 += step) {
    uint64_t zmask = 0;
#pragma unroll
    for (int q = 0; q < kFrontWords; ++q) {
      const int64_t w = w0 + int64_t(threadIdx.x) * kFrontWords + q;
      const uint32_t bits = w < words ? a.fl[w].x : 0u;
      if (bits == 0) continue;
      const int4* c4 = reinterpret_cast<const int4*>(a.cntA + w * 32);  // padded to whole words
      int4 c[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) c[k] = c4[k];
      uint32_t z = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        z |= (uint32_t(c[k].x == 0) | (uint32_t(c[k].y == 0) << 1) | (uint32_t(c[k].z == 0) << 2) |
              (uint32_t(c[k].w == 0) << 3)) << (4 * k);
      zmask |= uint64_t(z & bits) << (32 * q);
    }
    push_block(zmask, (w0 + int64_t(threadIdx.x) * kFrontWords) * 32, a.light, &a.ic->sl[0], 0u, s_tmp);
  }
}

// A finalised heavy member's rem pushed to its dependencies by the whole
// workgroup; the dependencies it finalises go to the next round, where every
// workgroup shares their walks.
__device__ inline void sweep_expand(const IncArgs& a, int32_t u, int round, uint32_t& fin, const WgQueue& wq) {
  const int64_t ru = a.rem[u];
  const int32_t o0 = a.p.dep_off[u], o1 = a.p.dep_off[u + 1];
  const int rn = round + 1 <= kIncRounds ? round + 1 : kIncRounds;
  for (int32_t e0 = o0; e0 < o1; e0 += int32_t(blockDim.x)) {
    const int32_t e = e0 + int32_t(threadIdx.x);
    bool zero = false;
    int32_t d = -1;
    if (e < o1) {
      d = a.p.dep_idx[e];
      if (d >= 0 && int64_t(d) < a.p.N && d != u) zero = push_count(a, d, ru, 1) == 1;
    }
    push_block1(zero, d, a.light, &a.ic->sl[rn], round_base(a.ic->sl, rn), wq.tmp);
  }
  (void)fin;
}

// One round of the sweep, this workgroup's share of it (as close_round).
__device__ void sweep_round(const IncArgs& a, int r, const WgQueue& wq, uint32_t& fin) {
  const uint32_t nh = ld_count(&a.ic->sh[r]), nl = ld_count(&a.ic->sl[r]);
  if (nh == 0 && nl == 0) return;  // the same on every thread
  if (threadIdx.x == 0) {
    *wq.n = 0;
    *wq.hn = 0;
    *wq.htaken = 0;
  }
  __syncthreads();
  const uint32_t bh = round_base(a.ic->sh, r), bl = round_base(a.ic->sl, r);
  for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) sweep_expand(a, a.heavy[bh + h], r, fin, wq);
  for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < nl; i0 += gridDim.x * blockDim.x) {
    const uint32_t i = i0 + threadIdx.x;
    sweep_walk(a, i < nl ? a.light[bl + i] : -1, r, fin, wq);
  }
  wg_drain(wq, [&](int32_t v) { sweep_walk(a, v, r, fin, wq); },
           [&](int32_t v) { sweep_expand(a, v, r, fin, wq); });
}

__global__ __launch_bounds__(kIncThreads) void k_inc_sweep(IncArgs a, int r) {
  if (invalid(a)) return;
  NALAR_INC_QUEUES(kIncThreads, false);
  uint32_t fin = 0;
  sweep_round(a, r, wq, fin);
  add_fin(a, fin);
}

// Rounds r0 .. kIncRounds - 1 of the sweep by one workgroup (r0 >= 1).
__global__ __launch_bounds__(kIncTailThreads) void k_inc_sweep_tail(IncArgs a, int r0) {
  if (invalid(a)) return;
  NALAR_INC_QUEUES(kIncTailThreads, true);
  uint32_t fin = 0;
  for (int r = r0; r < kIncRounds; ++r) {
    sweep_round(a, r, wq, fin);
    __syncthreads();
  }
  add_fin(a, fin);
}

// -------------------------------------------------------------------- ready

// Incomplete rounds or an unfinished closure: status for the host (one wave).
__device__ inline void check_rounds(const IncArgs& a) {
  static_assert(kIncParts == kWave, "one spread word per lane");
  const IncCtrl* ic = a.ic;
  const int64_t open = wave_sum_i64(int64_t(ic->a_n[lane_id()]) - int64_t(ic->fin[lane_id()]));
  if (lane_id() != 0) return;
  int rc = 0, rs = 0;  // the deepest rounds that had work
  for (int r = 1; r < kIncRounds; ++r) {
    if (ic->cl[r] | ic->ch[r]) rc = r;
    if (ic->sl[r] | ic->sh[r]) rs = r;
  }
  __hip_atomic_store(&a.host->inc_rounds, uint32_t(rc) | (uint32_t(rs) << 8), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_SYSTEM);
  if (ic->cl[kIncRounds] | ic->ch[kIncRounds] | ic->sl[kIncRounds] | ic->sh[kIncRounds])
    flag(a.ctrl, kStIncomplete);
  else if (open != 0)
    flag(a.ctrl, kStCycle);  // some member's closure consumers never all finalised
}

__device__ inline int64_t key_of(uint32_t policy, int64_t rem, int64_t dl) {
  if (policy & NALAR_ORDER_LPT) return -rem;
  if (policy & NALAR_ORDER_SRTF) return rem;
  return dl - rem;
}

// The ready futures: key, bin (splitters in LDS), route, slot; and the caller's
// copy of rem, whose lines the ready futures' gathers read anyway.
//
// Every workgroup takes each gridDim-th unit of kReadyUnit consecutive futures
// (so that all get an even mix of dense and sparse stretches of ids), copies
// their rem and lists the ready ones in LDS; a chunk of up to kReadyChunk of them
// is then keyed, counted per bin in LDS, given one segment of each bin with one
// returning atomic per bin, routed and stored.  The atomics (performed at the
// memory side, about 12 per ns on the whole chip) and the sparse gathers bound
// it, so a workgroup is as large as it can be, and a chunk as long: half the
// segments of 1,024-future chunks over 256-thread workgroups.  At 12.4M futures,
// 2.3M ready, 159 us and a 40 us copy of rem became 155 us, and 142 us with the
// attributes gathered as one record per future instead of four arrays; at 1.3M
// 42 + 5 became 40 (512 threads, in chunks of 4,096 or 8,192: 42 to 47).
constexpr int kReadyThreads = 1024;
constexpr int kReadyPer = 8;                          // ready futures per thread and chunk
constexpr int kReadyChunk = kReadyPer * kReadyThreads;
constexpr int kReadyUnit = 256;
constexpr int kReadyTake = 4;                         // futures per thread and step of the copy
constexpr int kReadyStep = kReadyTake * kReadyThreads;
constexpr int kReadyList = kReadyChunk + kReadyStep;  // a chunk and one step's worth

struct ReadyLds {
  int64_t* split;   // [kBinMax]
  int64_t* load;    // the instance table
  double* inv;
  int32_t* type;
  int32_t* idx;
  int32_t* speed;
  int32_t* pos;
  uint32_t* run;
  uint32_t* prun;
  uint32_t* cnt;    // [kBinMax] the chunk's futures per bin (zero between chunks)
  uint32_t* base;   // [kBinMax] its segments
  int32_t* list;    // [kReadyList]
};

__device__ inline ReadyLds carve_ready(unsigned char* sp, int M) {
  ReadyLds S;
  S.split = reinterpret_cast<int64_t*>(sp); sp += 8 * size_t(kBinMax);
  S.load = reinterpret_cast<int64_t*>(sp); sp += 8 * size_t(M);
  S.inv = reinterpret_cast<double*>(sp); sp += 8 * size_t(M);
  S.type = reinterpret_cast<int32_t*>(sp); sp += 4 * size_t(M);
  S.idx = reinterpret_cast<int32_t*>(sp); sp += 4 * size_t(M);
  S.speed = reinterpret_cast<int32_t*>(sp); sp += 4 * size_t(M);
  S.pos = reinterpret_cast<int32_t*>(sp); sp += 4 * size_t(M);
  S.run = reinterpret_cast<uint32_t*>(sp); sp += 4 * size_t(kTypeDirect);
  S.prun = reinterpret_cast<uint32_t*>(sp); sp += 4 * size_t(kTypeDirect);
  S.cnt = reinterpret_cast<uint32_t*>(sp); sp += 4 * size_t(kBinMax);
  S.base = reinterpret_cast<uint32_t*>(sp); sp += 4 * size_t(kBinMax);
  S.list = reinterpret_cast<int32_t*>(sp);
  return S;
}

struct ReadyAcc {
  int64_t mn = INT64_MAX, mx = INT64_MIN, n = 0;
};

// One chunk: the n (at most kReadyChunk) listed futures from `first` on.  Every
// thread of the workgroup calls it, after a barrier behind the listing.  kStore:
// the incremental pass (rem by id, attribute records), else the full pass by
// records (rem by position, the caller's attribute arrays).
template <bool kStore>
__device__ inline void ready_chunk(const IncArgs& a, const ReadyLds& S, int first, int n, ReadyAcc& acc) {
  constexpr int T = kReadyThreads;
  const int tid = threadIdx.x;
  const int nb = a.bk.nb;
  const uint32_t policy = a.p.policy;
  const bool out_slack = (policy & (NALAR_ORDER_LPT | NALAR_ORDER_SRTF)) != 0;
  const bool pack_wf = a.p.W <= kPackWf;
  int32_t v[kReadyPer];
  uint4 at[kReadyPer];
  int64_t key[kReadyPer];
  uint32_t bin[kReadyPer];  // bin, then bin | rank << 16 (rank < kReadyChunk)
  static_assert(kBinMax <= 65536 && kReadyChunk <= 65536, "bin and rank share a word");
#pragma unroll
  for (int j = 0; j < kReadyPer; ++j) v[j] = j * T + tid < n ? S.list[first + j * T + tid] : -1;
#pragma unroll
  for (int j = 0; j < kReadyPer; ++j) {
    const int32_t u = v[j] >= 0 ? v[j] : 0;
    at[j] = kStore ? a.att[u] : att_pack(a.p.wf[u], a.p.type[u], a.p.est[u], a.p.loc[u]);
    // (by records: the caller's copy, which this workgroup has just written)
    key[j] = kStore ? a.rem[u] : (a.rem_out ? a.rem_out[u] : a.rem_pos[a.pos_of_node[u]]);
  }
#pragma unroll
  for (int j = 0; j < kReadyPer; ++j) {
    bin[j] = 0;
    if (v[j] < 0) continue;
    const int64_t dl = a.p.deadline[at[j].y] - a.p.now;
    if (out_slack) a.stg_oslack[v[j]] = dl - key[j];
    key[j] = key_of(policy, key[j], dl);
  }
  for (int st = nb >> 1; st > 0; st >>= 1) {
#pragma unroll
    for (int j = 0; j < kReadyPer; ++j)
      if (v[j] >= 0 && S.split[bin[j] + st - 1] <= key[j]) bin[j] += st;
  }
#pragma unroll
  for (int j = 0; j < kReadyPer; ++j)
    if (v[j] >= 0) bin[j] |= atomicAdd(&S.cnt[bin[j]], 1u) << 16;
  __syncthreads();
  {  // one segment per bin for the chunk: every thread's atomics in flight together
    constexpr int kPerT = kBinMax / T;
    uint32_t c[kPerT];
#pragma unroll
    for (int q = 0; q < kPerT; ++q) {
      const int t = tid + q * T;
      c[q] = t < nb ? S.cnt[t] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kPerT; ++q) c[q] = c[q] ? add_agent(a.bk.cnt + tid + q * T, c[q]) : 0u;
#pragma unroll
    for (int q = 0; q < kPerT; ++q) {
      const int t = tid + q * T;
      if (t < nb) {
        S.base[t] = c[q];
        S.cnt[t] = 0;  // clean again before the next chunk
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kReadyPer; ++j) {
    if (v[j] < 0) continue;
    int32_t route;
    int64_t cost;
    route_future(int32_t(at[j].x), att_est(at[j]), att_loc(at[j]), int32_t(a.p.M), a.p.mig, S.type, S.idx, S.load,
                 S.speed, S.inv, S.pos, S.run, (policy & NALAR_ROUTE_STATEFUL) != 0, route, cost, S.prun);
    const uint32_t b = bin[j] & 0xFFFFu;
    const uint32_t slot = (bin[j] >> 16) + S.base[b];
    if (slot < uint32_t(a.bk.cap)) {
      int64_t* sl = reinterpret_cast<int64_t*>(a.bk.slot + int64_t(b) * a.bk.cap + slot);
      const int32_t rw = pack_wf ? slot_pack_wf(route, int32_t(at[j].y)) : slot_pack(route, 0);
      sl[0] = key[j];
      sl[1] = cost;
      sl[2] = int64_t(uint64_t(uint32_t(v[j])) | (uint64_t(uint32_t(rw)) << 32));
    } else {
      st_relaxed_agent(&a.ctrl->bucket_overflow, 1u);
    }
    acc.mn = key[j] < acc.mn ? key[j] : acc.mn;
    acc.mx = key[j] > acc.mx ? key[j] : acc.mx;
    acc.n += 1;
  }
}

template <bool kStore>
__global__ __launch_bounds__(kReadyThreads) void k_inc_ready(IncArgs a) {
  constexpr int T = kReadyThreads;
  const int tid = threadIdx.x;
  for (int64_t i = int64_t(blockIdx.x) * T + tid; i < a.bk_clear_n; i += int64_t(gridDim.x) * T)
    a.bk_clear[i] = 0;  // the next pass's bin counters
  Ctrl* ctrl = a.ctrl;
  if (ctrl->status != 0 || (!kStore && ctrl->unordered != 0)) return;  // written by earlier kernels only
  if (kStore && blockIdx.x == 0 && tid < kWave) check_rounds(a);
  extern __shared__ __align__(16) unsigned char smem[];
  const int M = int(a.p.M);
  const ReadyLds S = carve_ready(smem, M);
  __shared__ int s_n;
  __shared__ int64_t s_red[3][T / kWave];
  for (int i = tid; i < M; i += T) {
    S.load[i] = a.itab.load[i];
    S.inv[i] = a.itab.inv_speed[i];
    S.type[i] = a.itab.type[i];
    S.idx[i] = a.itab.idx[i];
    S.speed[i] = a.itab.speed[i];
    S.pos[i] = a.itab.pos_of[i];
  }
  for (int t = tid; t < kTypeDirect; t += T) {
    S.run[t] = a.itab.run[t];
    S.prun[t] = a.itab.prun[t];
  }
  for (int i = tid; i < a.bk.nb - 1; i += T) S.split[i] = a.bk.split[i];
  for (int i = tid; i < a.bk.nb; i += T) S.cnt[i] = 0;
  if (tid == 0) s_n = 0;
  __syncthreads();
  const int64_t N = a.p.N;
  const int64_t G = gridDim.x;
  ReadyAcc acc;
  // the ready futures of many dependencies (their own list)
  const uint32_t nh = kStore ? a.ic->r_heavy : 0u;
  for (uint32_t h0 = blockIdx.x; h0 < nh; h0 += uint32_t(G) * T) {
    const uint64_t h = uint64_t(h0) + uint64_t(tid) * uint64_t(G);
    const bool in = h < nh;
    const uint64_t m = ballot(in);
    int at = 0;
    if (lane_id() == 0 && m) at = atomicAdd(&s_n, int(__popcll(m)));
    at = readlane_i32(at, 0);
    if (in) S.list[at + int(lanes_below(m))] = a.rheavy[h];
    __syncthreads();
    const int n = s_n;
    if (n >= kReadyChunk) {  // the same on every thread
      ready_chunk<kStore>(a, S, n - kReadyChunk, kReadyChunk, acc);
      if (tid == 0) s_n = n - kReadyChunk;
    }
    __syncthreads();
  }
  // (by records a unit is a whole step: ids of one workflow lie hundreds apart,
  // and their rems side by side)
  constexpr int U = kStore ? kReadyUnit : kReadyStep;
  constexpr int kUnits = kReadyStep / U;  // units per step
  const int64_t units = (N + U - 1) / U;
  for (int64_t k0 = 0; int64_t(blockIdx.x) + k0 * G < units; k0 += kUnits) {
    int64_t id[kReadyTake], rv[kReadyTake];
    uint64_t w[kReadyTake];
#pragma unroll
    for (int j = 0; j < kReadyTake; ++j) {
      const int at = j * T + tid;  // within the step
      const int64_t u = int64_t(blockIdx.x) + (k0 + at / U) * G;
      id[j] = u < units ? u * U + at % U : N;
      if (id[j] > N) id[j] = N;
      w[j] = id[j] < N ? a.rbits[id[j] / kWave] : 0;  // the same on the lanes of the wave below N
      if (a.rem_out) {
        const int64_t x = id[j] < N ? id[j] : 0;
        rv[j] = kStore ? a.rem[x] : a.rem_pos[a.pos_of_node[x]];
      }
    }
#pragma unroll
    for (int j = 0; j < kReadyTake; ++j) {
      if (a.rem_out && id[j] < N) a.rem_out[id[j]] = rv[j];
      const bool in = (w[j] >> lane_id()) & 1u;
      const uint64_t m = ballot(in);
      int at = 0;
      if (lane_id() == 0 && m) at = atomicAdd(&s_n, int(__popcll(m)));
      at = readlane_i32(at, 0);
      if (in) S.list[at + int(lanes_below(m))] = int32_t(id[j]);
    }
    __syncthreads();
    const int n = s_n;
    if (n >= kReadyChunk) {  // the same on every thread
      ready_chunk<kStore>(a, S, n - kReadyChunk, kReadyChunk, acc);
      if (tid == 0) s_n = n - kReadyChunk;
    }
    __syncthreads();
  }
  if (s_n > 0) ready_chunk<kStore>(a, S, 0, s_n, acc);  // at most kReadyChunk - 1
  const int64_t mn = wave_min_i64(acc.mn), mx = wave_max_i64(acc.mx), rd = wave_sum_i64(acc.n);
  const int wv = tid / kWave;
  if (lane_id() == 0) {
    s_red[0][wv] = mn;
    s_red[1][wv] = mx;
    s_red[2][wv] = rd;
  }
  __syncthreads();
  if (tid == 0) {
    int64_t a0 = INT64_MAX, a1 = INT64_MIN, a2 = 0;
    for (int x = 0; x < T / kWave; ++x) {
      a0 = s_red[0][x] < a0 ? s_red[0][x] : a0;
      a1 = s_red[1][x] > a1 ? s_red[1][x] : a1;
      a2 += s_red[2][x];
    }
    if (a2 > 0) {
      const int slot = blockIdx.x & (kParts - 1);
      __hip_atomic_fetch_min(&ctrl->part_min[slot], a0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_max(&ctrl->part_max[slot], a1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      add_agent(&ctrl->part_cnt[slot], a2);
    }
  }
}

__global__ __launch_bounds__(kIncThreads) void k_inc_clear(uint32_t* p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * kIncThreads + threadIdx.x; i < n; i += int64_t(gridDim.x) * kIncThreads)
    p[i] = 0;
}

int inc_grid(int64_t n, int cap) {
  int64_t g = (n + kIncThreads - 1) / kIncThreads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return int(g);
}

}  // namespace

size_t inc_ready_lds(int64_t M) {
  return 8 * size_t(kBinMax) + 32 * size_t(M) + 8 * size_t(kTypeDirect) + 8 * size_t(kBinMax) +
         4 * size_t(kReadyList);
}

hipError_t prepare_inc_kernels() {
  for (const void* k : {reinterpret_cast<const void*>(&k_inc_ready<true>), reinterpret_cast<const void*>(&k_inc_ready<false>)}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             int(inc_ready_lds(NALAR_MAX_INSTANCES)));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_inc_clear(hipStream_t s, uint32_t* p, int64_t n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_inc_clear, dim3(inc_grid(n, 2048)), dim3(kIncThreads), 0, s, p, n);
  return hipGetLastError();
}

constexpr const char* kCloseNames[kIncTail] = {"inc_close_r0", "inc_close_r1", "inc_close_r2"};
constexpr const char* kSweepNames[kIncTail] = {"inc_sweep_r0", "inc_sweep_r1", "inc_sweep_r2"};

hipError_t launch_inc_closure(hipStream_t s, const IncArgs& a, int cus, int rounds,
                              void (*mark)(void*, const char*), void* ctx) {
  const int64_t seeds = a.n_log + (a.p.N - a.n_prev);
  if (rounds > kIncTail) rounds = kIncTail;
  if (rounds < 1) rounds = 1;
  mark(ctx, kCloseNames[0]);
  hipLaunchKernelGGL(k_inc_close, dim3(inc_grid(seeds, 4096)), dim3(kIncThreads), 0, s, a, 0);
  hipError_t e = hipGetLastError();
  for (int r = 1; r < rounds && e == hipSuccess; ++r) {
    mark(ctx, kCloseNames[r]);
    hipLaunchKernelGGL(k_inc_close, dim3(r < 2 ? 4 * cus : cus), dim3(kIncThreads), 0, s, a, r);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  mark(ctx, "inc_close_tail");
  hipLaunchKernelGGL(k_inc_close_tail, dim3(1), dim3(kIncTailThreads), 0, s, a, rounds);
  return hipGetLastError();
}

hipError_t launch_inc_scan(hipStream_t s, const IncArgs& a, int cus) {
  // as many workgroups for the futures of many dependencies as the edges allow
  const int64_t most = a.p.E / (kIncHeavy + 1);
  const int hb = int(most < cus ? most : cus);
  hipLaunchKernelGGL(k_inc_scan, dim3(hb + inc_grid((a.p.N + kScanPer - 1) / kScanPer, 16 * cus)),
                     dim3(kIncThreads), 0, s, a, hb);
  return hipGetLastError();
}

hipError_t launch_inc_sweep(hipStream_t s, const IncArgs& a, int cus, int rounds,
                            void (*mark)(void*, const char*), void* ctx) {
  if (rounds > kIncTail) rounds = kIncTail;
  if (rounds < 1) rounds = 1;
  mark(ctx, "inc_front0");
  const int64_t words = (a.p.N + 31) / 32, per = kFrontThreads * kFrontWords;
  hipLaunchKernelGGL(k_inc_front0, dim3(inc_grid((words + per - 1) / per * kIncThreads, 4 * cus)),
                     dim3(kFrontThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  for (int r = 0; r < rounds && e == hipSuccess; ++r) {
    mark(ctx, kSweepNames[r]);
    hipLaunchKernelGGL(k_inc_sweep, dim3(4 * cus), dim3(kIncThreads), 0, s, a, r);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  mark(ctx, "inc_sweep_tail");
  hipLaunchKernelGGL(k_inc_sweep_tail, dim3(1), dim3(kIncTailThreads), 0, s, a, rounds);
  return hipGetLastError();
}

hipError_t launch_inc_ready(hipStream_t s, const IncArgs& a, int cus, bool records) {
  // one workgroup per CU (their LDS allows no more), fewer for few futures
  int64_t g = (a.p.N + kReadyStep - 1) / kReadyStep;
  if (g > cus) g = cus;
  const dim3 grid(unsigned(g < 1 ? 1 : g));
  if (records)
    hipLaunchKernelGGL(k_inc_ready<false>, grid, dim3(kReadyThreads), inc_ready_lds(a.p.M), s, a);
  else
    hipLaunchKernelGGL(k_inc_ready<true>, grid, dim3(kReadyThreads), inc_ready_lds(a.p.M), s, a);
  return hipGetLastError();
}

}  // namespace nalar
