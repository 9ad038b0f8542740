// Remaining critical paths of a large snapshot whose ids are not grouped by
// workflow (ids by age, workflows beyond what one wave sweeps), when every
// dependency lies at a lower id than its consumer inside its workflow.
//
// Everything about a future is read where it lies together: by id.  Sweeping
// workflow by workflow, as the block sweep does, reads each attribute of each
// future through the position maps, a 64-byte line at a time (6.6M futures over
// 256 workflows moved 1.2 GB, against 0.3 GB needed, and every ready future
// claimed its bin slot with an atomic of its own).  So:
//   k_rec        by id: dependencies checked, readiness (one bit per future), and
//                one 16-byte record per future written at its position (est',
//                the position of its only dependency, its id); a tile of ids
//                writes runs of neighbouring positions, which the L2 joins;
//   k_sweep_rec  by position: one workgroup per workflow, chunks of positions
//                from the last to the first, rem written by position; it also
//                checks the dependencies of futures with more than kRecLight,
//                whose lists it reads anyway, and decides their readiness;
// and the ready kernel of the incremental pass (by id again) brings rem into the
// caller's order while it keys, routes and bins the ready futures.
//
// A snapshot with a dependency that does not lie lower sets Ctrl::unordered: the
// pass is then done again by the block sweep.  Done twice, that pass costs up to
// 1.5 times one by the block sweep alone (348 us, so 525, for 1.3M futures of
// 1,000 workflows; 1,360 and 1,860 for 4.6M of 256), so k_order_probe looks for
// such a dependency behind the block sweeps: on a handle's first pass, which has no
// bins for this path yet, and after a snapshot out of order.
//
// Per future k_rec moves about 45 bytes (6.6M: 84 us, 3.5 TB/s, with one line
// written per run of records) and k_sweep_rec 24 (83 us: 26 chunks of about 3 us,
// three to five barriers and LDS trips each).  The whole pass over 6.6M futures of
// 256 workflows went from 607 to 430 us: the block sweep took 424 us of it, these
// two and the ready kernel take 276, and the bin sort 38 for 58, its futures
// having been appended a workgroup's worth at a time.
//
// The fan-ins of sessions started together are created together: with their
// lists taken where their ids lie, in k_rec, one workgroup read 64 of them one
// after another and single threads the rest (1.05M futures of 256 map/reduce
// sessions in creation order: k_rec 4,600 us, now 17, the pass 4,734, now 162; the
// block sweep's pass 181).
#include "internal.hpp"

namespace nalar {

namespace {

constexpr int kRecThreads = 256;
constexpr int kRecPer = 8;                       // futures per thread, kRecThreads apart
constexpr int kRecTile = kRecThreads * kRecPer;
constexpr int kRecLight = 32;                    // more dependencies: left to the sweep's workgroups
constexpr int kRecList = 64;                     // such futures a chunk of the sweep lists

// A record's third word: the position (inside the workflow) of the future's only
// dependency, or one of these.
constexpr int32_t kRecNone = -1;  // no (valid) dependency
constexpr int32_t kRecMany = -2;  // several: gathered from the list

__device__ inline bool done_of(const uint32_t* bits, int32_t v) {
  return ((bits[uint32_t(v) >> 5] >> (uint32_t(v) & 31u)) & 1u) != 0u;
}

// The workflow-local position of dependency d at position q (its future at
// local position k of the workflow at [b, b + n)), or -1 with the problem
// reported; up: it does not lie lower.
__device__ inline int32_t rec_dep(const RecArgs& a, bool in_range, int32_t q, int32_t b, int32_t n, int32_t k,
                                  bool& up) {
  const int32_t lp = q - b;
  if (!in_range || lp < 0 || lp >= n) {
    flag_sweep(a.ctrl, kStInval);
    return -1;
  }
  if (lp == k) {
    flag_sweep(a.ctrl, kStCycle);
    return -1;
  }
  up |= lp > k;
  return lp;
}

// Not this path: the host does the pass again.
__device__ inline void flag_unordered(Ctrl* c) {
  st_relaxed_agent(&c->unordered, 1u);
  st_relaxed_agent(&c->bucket_overflow, 1u);
}

__global__ __launch_bounds__(kRecThreads) void k_rec(RecArgs a) {
  if (a.ctrl->status) return;
  __shared__ int s_up;
  const int64_t N = a.p.N;
  const int tid = threadIdx.x, wv = tid / kWave, ln = lane_id();
  const int64_t t0 = int64_t(blockIdx.x) * kRecTile;
  if (tid == 0) s_up = 0;
  __syncthreads();
  int32_t o0[kRecPer], o1[kRecPer], w[kRecPer], q[kRecPer], d0[kRecPer], dq[kRecPer], b[kRecPer], n[kRecPer];
  int64_t est[kRecPer];
  uint8_t dn[kRecPer];
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    const int64_t v = t0 + j * kRecThreads + tid;
    const int64_t vs = v < N ? v : N - 1;
    w[j] = a.p.wf[vs];
    o0[j] = a.p.dep_off[vs];
    o1[j] = a.p.dep_off[vs + 1];
    q[j] = a.pos_of_node[vs];
    est[j] = a.p.est[vs];
    dn[j] = a.p.done[vs];
  }
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    d0[j] = o1[j] > o0[j] ? a.p.dep_idx[o0[j]] : -1;
    b[j] = a.wf_off[w[j]];
    n[j] = a.wf_off[w[j] + 1];
  }
  bool dd[kRecPer];
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    const bool ok = d0[j] >= 0 && int64_t(d0[j]) < N;
    dq[j] = a.pos_of_node[ok ? d0[j] : 0];
    dd[j] = done_of(a.done_bits, ok ? d0[j] : 0);
  }
  bool up = false;
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    const int64_t v = t0 + j * kRecThreads + tid;
    const int32_t deg = o1[j] - o0[j];
    const int32_t k = q[j] - b[j], nn = n[j] - b[j];
    bool ready = v < N && dn[j] == 0;
    int32_t one = kRecNone;
    if (v < N && deg > kRecLight) {
      one = kRecMany;
      ready = false;  // the sweep decides
    } else if (v < N && deg > 0) {
      const int32_t lp = rec_dep(a, d0[j] >= 0 && int64_t(d0[j]) < N, dq[j], b[j], nn, k, up);
      if (lp >= 0 && !dd[j]) ready = false;
      one = deg == 1 ? lp : kRecMany;
      for (int32_t e = o0[j] + 1; e < o1[j]; ++e) {
        const int32_t d = a.p.dep_idx[e];
        const bool ok = d >= 0 && int64_t(d) < N;
        const int32_t x = rec_dep(a, ok, ok ? a.pos_of_node[d] : 0, b[j], nn, k, up);
        if (x >= 0 && !done_of(a.done_bits, d)) ready = false;
      }
    }
    const uint64_t m = ballot(ready);
    const int64_t v0 = t0 + j * kRecThreads + wv * kWave;
    if (ln == 0 && v0 < N) a.rbits[v0 / kWave] = m;
    if (v < N) {
      const int64_t e = dn[j] ? 0 : est[j];
      a.rec[q[j]] = make_uint4(uint32_t(uint64_t(e)), uint32_t(uint64_t(e) >> 32), uint32_t(one), uint32_t(v));
    }
  }
  if (up) s_up = 1;
  __syncthreads();
  if (tid == 0 && s_up) flag_unordered(a.ctrl);
}

// Ids ascend with the position inside a workflow, so a dependency lies higher
// exactly if its id does.  Of a longer list only the first kRecLight entries are
// looked at: a miss costs the host one pass done twice.
__global__ __launch_bounds__(kRecThreads) void k_order_probe(ProblemDev p, Ctrl* ctrl, HostStatus* host) {
  if (ctrl->status) return;
  const int64_t t0 = int64_t(blockIdx.x) * kRecTile + threadIdx.x;
  int32_t o0[kRecPer], o1[kRecPer], d0[kRecPer];
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    const int64_t v = t0 + j * kRecThreads;
    o0[j] = v < p.N ? p.dep_off[v] : 0;
    o1[j] = v < p.N ? p.dep_off[v + 1] : 0;
  }
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) d0[j] = o1[j] > o0[j] ? p.dep_idx[o0[j]] : -1;
  bool up = false;
#pragma unroll
  for (int j = 0; j < kRecPer; ++j) {
    const int64_t v = t0 + j * kRecThreads;
    up |= d0[j] > v;
    const int32_t e1 = o1[j] - o0[j] < kRecLight ? o1[j] : o0[j] + kRecLight;
    for (int32_t e = o0[j] + 1; e < e1; ++e) up |= p.dep_idx[e] > v;
  }
  if (ballot(up) == 0 || lane_id() != 0 || ld_relaxed_agent(&ctrl->higher) != 0) return;
  if (__hip_atomic_exchange(&ctrl->higher, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)  // the first wave tells
    __hip_atomic_store(&host->higher, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------------- sweep

constexpr int kRecT = 1024;           // positions per chunk, one per thread
// Chunks whose maxima are in LDS: as many as fit when the chip holds every
// workflow at once with one workgroup per CU, else as many as fit twice.  19 and 9
// chunks, in us of this kernel: 24 workflows of 23K futures 63 and 70, 100 of 23K
// 65 and 75, 64 of 20K 69 and 75, 128 of 10K 43 and 43; 500 of 2.5K 32 and 31,
// 1,000 of 5K 92 and 89, 4,000 of 1.3K 160 and 152, but 300 of 14K 86 and 92.
constexpr int kRecWinOne = 19, kRecWinTwo = 9;

__device__ inline void lds_max(int64_t* p, int64_t v) {
  atomicMax(reinterpret_cast<long long*>(p), (long long)v);
}

// One workgroup per workflow; every consumer of a future lies at a higher
// position, so its positions are taken in chunks from the last to the first.  A
// push into the chunk in work or one of the next win - 1 goes to their maxima in
// LDS.  One further down goes to rem_pos, which holds a running maximum (zero at
// first) until the chunk is done, by an atomic of the workgroup's own: nobody
// else reads or writes the workflow's positions, so it is done in this XCD's L2
// and nothing waits for it.  The next chunk's maxima and the records of the one
// after are loaded while this chunk is worked on: the atomics they may depend on
// were issued win - 1 chunks earlier, and every wave has waited for its own
// before a barrier since.  (With the maxima of two chunks in LDS and the other
// pushes in a log per chunk, counted beforehand, the kernel took 169 us over 6.6M
// futures, 62 of them the count; with those pushes as atomics, 200 us: they miss
// the L2.  In 19 chunks of 26 LDS takes more than nine pushes of ten: 78 us.)
// Inside a chunk every future whose rem has grown pushes into its dependencies in
// the chunk until none grows (the maxima only grow: the longest path exactly).
__global__ __launch_bounds__(kRecT) void k_sweep_rec(RecArgs a, int win) {
  constexpr int T = kRecT;
  extern __shared__ __align__(16) unsigned char smem[];
  int64_t* const s_mx = reinterpret_cast<int64_t*>(smem);  // [win][T], the chunks in turn
  __shared__ int s_stop, s_hn;
  __shared__ int32_t s_hk[kRecList], s_hv[kRecList];  // listed futures of many dependencies: position, id
  __shared__ int64_t s_hr[kRecList];                  // their rem so far
  __shared__ int s_hg[kRecList];                      // grown this round
  __shared__ int s_hb[kRecList];                      // some dependency is open
  __shared__ int s_any[3];                            // some push inside the chunk, by round
  const int tid = threadIdx.x;
  Ctrl* ctrl = a.ctrl;
  if (tid == 0) s_stop = (ctrl->status | ctrl->unordered) != 0 ? 1 : 0;
  __syncthreads();
  if (s_stop) return;
  const int64_t N = a.p.N;
  bool up = false;

  for (int64_t w = blockIdx.x; w < a.p.W; w += gridDim.x) {
    const int32_t b = a.wf_off[w];
    const int n = a.wf_off[w + 1] - b;
    if (n <= 0) continue;  // the same on every thread
    const int nc = (n + T - 1) / T;
    const uint4* rec = a.rec + b;
    int64_t* rem = a.rem_pos + b;
    // local position of dependency entry e (checked when the records were made)
    auto dep_pos = [&](int32_t e) -> int32_t {
      const int32_t d = a.p.dep_idx[e];
      const int32_t lp = d >= 0 && int64_t(d) < N ? a.pos_of_node[d] - b : -1;
      return lp < n ? lp : -1;
    };
    // the same, checked, for the future of many dependencies at position hk
    auto check_pos = [&](int32_t e, int32_t hk, bool& blocked) -> int32_t {
      const int32_t d = a.p.dep_idx[e];
      const bool ok = d >= 0 && int64_t(d) < N;
      const int32_t q = a.pos_of_node[ok ? d : 0];
      const bool dd = done_of(a.done_bits, ok ? d : 0);
      const int32_t lp = rec_dep(a, ok, q, b, n, hk, up);
      blocked |= lp >= 0 && !dd;
      return lp;
    };
    auto set_ready = [&](int32_t hv) {  // no dependency of hv is open
      if (!done_of(a.done_bits, hv))
        atomicOr(reinterpret_cast<unsigned long long*>(&a.rbits[uint32_t(hv) / kWave]), 1ull << (uint32_t(hv) % kWave));
    };
    bool overflow = false;
    // (behind the barrier the last workflow ended with)
    for (int u = 0; u < win; ++u) s_mx[u * T + tid] = 0;
    for (int i = tid; i < (nc - win) * T; i += T) rem[i] = 0;
    __syncthreads();
    const int kl = (nc - 1) * T + tid;
    uint4 cur = kl < n ? rec[kl] : make_uint4(0, 0, uint32_t(kRecNone), 0);
    uint4 next = nc > 1 ? rec[kl - T] : make_uint4(0, 0, uint32_t(kRecNone), 0);
    int64_t far = 0;  // the chunk's maximum from further up
    int slot0 = 0;    // the chunk's maxima; those of the chunk i after it: slot0 + i, modulo win
    for (int c = nc - 1; c >= 0; --c, slot0 = slot0 + 1 < win ? slot0 + 1 : 0) {
      const int c0 = c * T;
      int64_t* mx = s_mx + slot0 * T;
      s_mx[(slot0 > 0 ? slot0 - 1 : win - 1) * T + tid] = 0;  // the last chunk's, done with
      if (tid == 0) {
        s_hn = 0;
        s_any[0] = 0;
      }
      // the next chunk's maxima and the records of the one after, in flight
      // through this chunk
      uint4 after = make_uint4(0, 0, uint32_t(kRecNone), 0);
      int64_t far1 = 0;
      if (c > 1) after = rec[c0 - 2 * T + tid];
      if (c > 0 && c - 1 + win < nc)
        far1 = __hip_atomic_load(rem + c0 - T + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const int k = c0 + tid;
      const bool own = k < n;
      const int64_t est = int64_t((uint64_t(cur.y) << 32) | cur.x);
      const int32_t one = own ? int32_t(cur.z) : kRecNone;
      const int32_t v = int32_t(cur.w);
      int32_t o0 = 0, o1 = 0;
      int slot = -1;  // in the list of futures of many dependencies
      if (one == kRecMany) {
        o0 = a.p.dep_off[v];
        o1 = a.p.dep_off[v + 1];
      }
      // These barriers order LDS only: the loads above stay in flight.
      lds_barrier();
      if (o1 - o0 > kRecLight) {
        slot = atomicAdd(&s_hn, 1);
        if (slot < kRecList) {
          s_hk[slot] = k;
          s_hv[slot] = v;
          s_hb[slot] = 0;
        } else {
          slot = -1;  // the list is full: its thread pushes alone
        }
      }
      lds_barrier();
      const int nh = __builtin_amdgcn_readfirstlane(s_hn < kRecList ? s_hn : kRecList);
      // 1: inside the chunk
      int64_t r = -1;
      for (int round = 0;; ++round) {
        int64_t x = r;
        if (own) {
          const int64_t m = mx[tid];
          x = est + (m > far ? m : far);
          if (x > NALAR_REM_MAX) {
            overflow = true;
            x = NALAR_REM_MAX + 1;
          }
        }
        const bool grew = x != r;
        r = x;
        bool pushed = false;
        if (tid == 0) s_any[(round + 1) % 3] = 0;
        lds_barrier();  // every maximum is read before this round's pushes
        if (slot >= 0) {
          s_hr[slot] = r;
          s_hg[slot] = grew ? 1 : 0;
        } else if (grew) {
          if (one >= c0) {
            lds_max(&mx[one - c0], r);
            pushed = true;
          } else if (one == kRecMany) {
            for (int32_t e = o0; e < o1; ++e) {
              const int32_t lp = dep_pos(e);
              if (lp >= c0 && lp < k) {
                lds_max(&mx[lp - c0], r);
                pushed = true;
              }
            }
          }
        }
        if (nh > 0) {  // the same on every thread
          lds_barrier();
          for (int h = 0; h < nh; ++h) {
            if (!s_hg[h]) continue;
            const int64_t hr = s_hr[h];
            const int32_t hv = s_hv[h], hk = s_hk[h], e1 = a.p.dep_off[hv + 1];
            for (int32_t e = a.p.dep_off[hv] + tid; e < e1; e += T) {
              const int32_t lp = dep_pos(e);
              if (lp >= c0 && lp < hk) {
                lds_max(&mx[lp - c0], hr);
                pushed = true;
              }
            }
          }
        }
        if (ballot(pushed) != 0 && lane_id() == 0) s_any[round % 3] = 1;
        lds_barrier();
        if (s_any[round % 3] == 0) break;  // the same on every thread
      }
      // 2: rem is final; out of the chunk (every lane of a wave calls)
      auto push_out = [&](int32_t lp, int64_t rr) {
        bool mine = lp >= 0 && lp < c0;
        const uint64_t act = ballot(mine);
        if (act == 0) return;
        const int lead = __builtin_ctzll(act);
        const int32_t first = readlane_i32(lp, lead);
        if ((act & (act - 1)) != 0 && ballot(mine && lp != first) == 0) {  // a fan-in: one push
          const int64_t m = wave_max_i64(mine ? rr : INT64_MIN);
          mine = lane_id() == lead;
          rr = m;
        }
        if (!mine) return;
        const int off = c - lp / T;
        if (off < win) {
          const int at = slot0 + off < win ? slot0 + off : slot0 + off - win;
          lds_max(&s_mx[at * T + lp % T], rr);
        } else {
          __hip_atomic_fetch_max(rem + lp, rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      };
      // The last chunk's atomics are done (and this chunk's loads have arrived).
      __asm__ __volatile__("s_waitcnt vmcnt(0)" ::: "memory");
      if (own) rem[k] = r;
      push_out(one, r);
      {
        const bool alone = one == kRecMany && slot < 0, open = alone && o1 - o0 > kRecLight;
        const int32_t e1 = open ? o0 : o1;
        for (int32_t e = o0; ballot(alone && e < e1) != 0; ++e) push_out(alone && e < e1 ? dep_pos(e) : -1, r);
        if (ballot(open) != 0) {
          bool blocked = false;
          for (int32_t e = o0; ballot(open && e < o1) != 0; ++e)
            push_out(open && e < o1 ? check_pos(e, k, blocked) : -1, r);
          if (open && !blocked) set_ready(v);
        }
      }
      for (int h = 0; h < nh; ++h) {
        const int64_t hr = s_hr[h];
        const int32_t hv = s_hv[h], hk = s_hk[h], e1 = a.p.dep_off[hv + 1];
        bool blocked = false;
        for (int32_t e0 = a.p.dep_off[hv]; e0 < e1; e0 += T) {
          const int32_t e = e0 + tid;
          push_out(e < e1 ? check_pos(e, hk, blocked) : -1, hr);
        }
        if (blocked) s_hb[h] = 1;
      }
      cur = next;
      next = after;
      far = far1;
      lds_barrier();
      if (nh > 0 && tid < nh && s_hb[tid] == 0) set_ready(s_hv[tid]);
    }
    if (overflow) flag_sweep(ctrl, kStRange);
  }
  if (ballot(up) != 0 && lane_id() == 0 && ld_relaxed_agent(&ctrl->unordered) == 0) flag_unordered(ctrl);
}

size_t sweep_rec_lds(int win) { return 8 * size_t(kRecT) * size_t(win); }

}  // namespace

hipError_t prepare_rec_kernels() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sweep_rec), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(sweep_rec_lds(kRecWinOne)));
}

hipError_t launch_order_probe(hipStream_t s, const ProblemDev& p, Ctrl* ctrl, HostStatus* host) {
  hipLaunchKernelGGL(k_order_probe, dim3(unsigned((p.N + kRecTile - 1) / kRecTile)), dim3(kRecThreads), 0, s, p, ctrl, host);
  return hipGetLastError();
}

hipError_t launch_rec(hipStream_t s, const RecArgs& a) {
  hipLaunchKernelGGL(k_rec, dim3(unsigned((a.p.N + kRecTile - 1) / kRecTile)), dim3(kRecThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_sweep_rec(hipStream_t s, const RecArgs& a, int cus) {
  const int64_t g = a.p.W < 2 * int64_t(cus) ? a.p.W : 2 * int64_t(cus);
  const int win = a.p.W <= cus ? kRecWinOne : kRecWinTwo;
  hipLaunchKernelGGL(k_sweep_rec, dim3(unsigned(g)), dim3(kRecT), sweep_rec_lds(win), s, a, win);
  return hipGetLastError();
}

}  // namespace nalar
