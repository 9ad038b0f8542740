// Load-aware routing (NALAR_ROUTE_GREEDY): the ready futures, already in
// output order, are routed one at a time; each takes the cheapest candidate of
// its type under the loads left by the futures before it and adds its service
// time on the chosen instance to that instance's load (routing that balances
// load across instances, Section 6.1).
//
// Futures of different types never share a candidate, so each type is an
// independent sequence: one workgroup of four waves per type.  What bounds it
// is the chain from one future to the next (the chosen instance's load decides
// the next choice), so with at most 64 candidates everything else is taken off
// the wave that runs the chain, in steps of one batch of 64 futures:
//   wave 1      walks the output order and queues the type's futures in LDS;
//   waves 2, 3  turn a queued batch into a table of each future's cost on each
//               candidate, less the running load;
//   wave 0      routes the batch tabulated in the step before.
// The chain itself runs on 32-bit words.  A batch's loads are taken relative to
// the lowest one, and a cost is packed as (relative cost << bits) | candidate,
// so that one unsigned minimum yields the cheapest candidate with the lowest
// index: per future a saturating add, a minimum over the candidates' lanes
// (fused DPP minima inside a row of 16; the groups of lanes hold copies of the
// same candidates, so every lane knows the winner) and the winner's add.  A
// word that does not hold its value saturates and then loses against every
// word that does, so the result is exact unless a saturated word wins or a load
// saturates on the way; such a batch is routed again in 64 bits (relative
// costs of 2^29 us with 8 candidates, 2^26 us with 64: minutes of queued work
// beyond the least loaded instance).  More than 64 candidates stay in LDS and
// each future scans them lane-parallel.
//
// Measured, the whole pass over 131,072 futures, 15.7K of them ready, 8 types
// of about 8 instances: 563 us with one wave per type and a 64-bit chain (497 us
// in this kernel, about 240 ns per future of the longest type), 168 us in this
// form, 159 us launched behind the sort without a wait of the host.
#include "internal.hpp"

namespace nalar {

namespace {

constexpr int kGreedyThreads = 4 * kWave;   // router, scanner, two table builders
constexpr int kBuilders = 2;
constexpr int kWalk = 16;                   // chunks of the output order loaded at once
constexpr int kWalkBlock = kWalk * kWave;
constexpr int kGreedyRing = 2048;           // queued futures of the type
static_assert(kGreedyRing >= 2 * kWave + kWalkBlock, "room for the batches in work and one walk block");
constexpr uint32_t kSat = 0xFFFFFFFFu;      // a packed word that does not hold its value

// DPP controls that stay inside a row of 16 lanes.
constexpr int kDppHalfMirror = 0x141;       // lane i <- lane 7 - i within each 8 lanes
constexpr int kDppMirror = 0x140;           // lane i <- lane 15 - i within each 16 lanes

template <int kCtrl>
__device__ inline uint32_t row_min_u32(uint32_t x) {
  // every pattern used reads a lane of the same row, so bound_ctrl changes
  // nothing, but with it the move folds into the minimum
  const uint32_t y = uint32_t(__builtin_amdgcn_mov_dpp(int(x), kCtrl, 0xF, 0xF, true));
  return y < x ? y : x;
}

// Minimum over each group of W lanes, on every lane of it (W = 8, 16 or 64).
template <int W>
__device__ inline uint32_t lanes_min_u32(uint32_t x) {
  x = row_min_u32<kDppXor1>(x);
  x = row_min_u32<kDppXor2>(x);
  x = row_min_u32<kDppHalfMirror>(x);
  if constexpr (W > 8) x = row_min_u32<kDppMirror>(x);
  if constexpr (W > 16) {
    const uint32_t a = uint32_t(readlane_i32(int(x), 0)), b = uint32_t(readlane_i32(int(x), 16));
    const uint32_t c = uint32_t(readlane_i32(int(x), 32)), d = uint32_t(readlane_i32(int(x), 48));
    const uint32_t ab = a < b ? a : b, cd = c < d ? c : d;
    x = ab < cd ? ab : cd;
  }
  return x;
}

struct Cand {  // the type's candidates in LDS (candidate q = the q-th instance of the type)
  int64_t* load;
  double* inv;
  int32_t* speed;
  int32_t* idx;
  int32_t* q_of;   // candidate of an instance of the type
  int32_t* itype;  // type of every instance
};

// A future's packed cost on a candidate less its load, and the packed service
// time that choosing the candidate adds to the load.
struct Entry {
  uint32_t cost;
  uint32_t svc;
};

struct Queue {  // LDS: the queued futures, two batches' tables, and the walk's progress
  int32_t out[kGreedyRing];
  int64_t est[kGreedyRing];
  int32_t loc[kGreedyRing];
  Entry tab[2][kWave * kWave];
  int tail[2];   // futures queued so far, by the parity of the step that reads it
  int done[2];   // the walk has reached the end of the order
};

// A queued future pinned to candidate >= 0 (a future whose state lives on an
// instance of its own type runs there), or -1.
__device__ inline int pin_of(const GreedyArgs& g, const Cand& cd, int32_t t, int32_t l) {
  return (g.stateful && l >= 0 && cd.itype[l] == t) ? cd.q_of[l] : -1;
}

// The table of the batch [head, head + B), one builder's share: 64 / W futures
// per step, lane (f, q) taking future f and candidate q.
template <int W, int IB>
__device__ inline void build_table(const GreedyArgs& g, const Cand& cd, int32_t t, int nc, int builder, int head,
                                   int B, const Queue& Q, Entry* tab) {
  const int ln = lane_id();
  const int q = ln & (W - 1);
  const bool cand = q < nc;
  const int32_t sp = cand ? cd.speed[q] : 1;
  const double inv = cand ? cd.inv[q] : 1.0;
  const int32_t idx = cand ? cd.idx[q] : -1;
  constexpr int F = kWave / W;
  for (int j0 = builder * F; j0 < B; j0 += kBuilders * F) {
    const int j = j0 + ln / W;
    const int slot = (head + (j < B ? j : 0)) & (kGreedyRing - 1);
    const int32_t l = Q.loc[slot];
    const int pin = pin_of(g, cd, t, l);
    const int64_t svc = floordiv_exact(double(Q.est[slot] * 1000), sp, inv);
    const uint64_t c = uint64_t(svc) + uint64_t((pin < 0 && l >= 0 && l != idx) ? g.mig : 0);
    const bool out = !cand || (pin >= 0 && pin != q);
    Entry e;
    e.cost = (out || (c >> (32 - IB)) != 0) ? kSat : (uint32_t(c) << IB) | uint32_t(q);
    e.svc = (uint64_t(svc) >> (32 - IB)) != 0 ? kSat : uint32_t(svc) << IB;
    if (j < B) tab[j * W + q] = e;
  }
}

// Routes the batch in 64 bits (lane q, q + W, ... hold copies of candidate q's
// running load).
template <int W>
__device__ void route_batch_wide(const GreedyArgs& g, const Cand& cd, int32_t t, int nc, int head, int B,
                                 const Queue& Q, int64_t& my_load, int& qv, int64_t& cv) {
  const int ln = lane_id();
  const int q = ln & (W - 1);
  const int32_t sp = q < nc ? cd.speed[q] : 1;
  const double inv = q < nc ? cd.inv[q] : 1.0;
  const int32_t idx = q < nc ? cd.idx[q] : -1;
  for (int j = 0; j < B; ++j) {
    const int slot = (head + j) & (kGreedyRing - 1);
    const int32_t l = Q.loc[slot];
    const int pin = pin_of(g, cd, t, l);
    const int64_t svc = floordiv_exact(double(Q.est[slot] * 1000), sp, inv);
    const int64_t c = ln < nc ? my_load + svc + ((pin < 0 && l >= 0 && l != idx) ? g.mig : 0) : INT64_MAX;
    int qb = __builtin_amdgcn_readfirstlane(pin);
    int64_t cb;
    if (qb >= 0) {
      cb = readlane_i64(c, qb);
    } else {
      cb = wave_min_i64(c);
      qb = __builtin_ctzll(ballot(c == cb));  // lanes ascend with the index: lowest wins
    }
    my_load += q == qb ? svc : 0;
    qv = ln == j ? qb : qv;
    cv = ln == j ? cb : cv;
  }
}

// Routes the batch [head, head + B) from its table.
template <int W, int IB>
__device__ inline void route_batch(const GreedyArgs& g, const Cand& cd, int32_t t, int nc, int head, int B,
                                   const Queue& Q, const Entry* tab, int64_t& my_load, bool& bad) {
  const int ln = lane_id();
  const int q = ln & (W - 1);
  const int64_t base = wave_min_i64(my_load);  // lanes past the candidates hold INT64_MAX
  const uint64_t rel = uint64_t(my_load) - uint64_t(base);
  const uint32_t l0 = (q >= nc || (rel >> (32 - IB)) != 0) ? kSat : uint32_t(rel) << IB;
  uint32_t l = l0, mv = 0;
  constexpr int U = 8;  // entries read ahead
  Entry nx[U];
#pragma unroll
  for (int u = 0; u < U; ++u) nx[u] = tab[u * W + q];
  auto route = [&](const Entry& e, int j) {
    const uint32_t c = __builtin_elementwise_add_sat(l, e.cost);
    const uint32_t m = lanes_min_u32<W>(c);
    l = c == m ? __builtin_elementwise_add_sat(l, e.svc) : l;
    mv = ln == j ? m : mv;
  };
  int j0 = 0;
  for (; j0 + U <= B; j0 += U) {
    Entry e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      e[u] = nx[u];
      const int jn = j0 + U + u;
      nx[u] = tab[(jn < kWave ? jn : 0) * W + q];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) route(e[u], j0 + u);
  }
  for (; j0 < B; ++j0) route(tab[j0 * W + q], j0);
  const bool act = ln < B;
  int qv = int(mv & uint32_t((1 << IB) - 1));
  int64_t cv = base + int64_t(mv >> IB);
  if (ballot((act && mv == kSat) || (l == kSat && l0 != kSat)) == 0) {
    if (l0 != kSat) my_load = base + int64_t(l >> IB);
  } else {
    route_batch_wide<W>(g, cd, t, nc, head, B, Q, my_load, qv, cv);
  }
  if (act) {
    const int32_t out = Q.out[(head + ln) & (kGreedyRing - 1)];
    g.route[out] = cd.idx[qv];
    if (g.cost) g.cost[out] = cv;
  }
  // loads only grow, and a batch adds at most 64 service times (each below
  // 2^50), so one check per batch sees every load that passes the limit
  bad |= q < nc && my_load > NALAR_REM_MAX;
}

// The walk over the output order (one wave): blocks of kWalkBlock positions,
// every attribute load of a block issued before any is used, the next block's
// ids loaded while this block is queued.
struct Walk {
  int64_t k0;
  int32_t vn[kWalk];
};

__device__ inline void walk_ids(const GreedyArgs& g, int64_t R, Walk& w, int64_t k0) {
  const int ln = lane_id();
#pragma unroll
  for (int u = 0; u < kWalk; ++u) {
    const int64_t k = k0 + u * kWave + ln;
    w.vn[u] = k < R ? g.order[k] : 0;
  }
}

// Queues the type's futures of the next block; returns the new tail.
__device__ inline int walk_block(const GreedyArgs& g, int64_t R, int32_t t, Walk& w, Queue& Q, int tail) {
  const int ln = lane_id();
  int32_t tt[kWalk], ll[kWalk];
  int64_t ee[kWalk];
#pragma unroll
  for (int u = 0; u < kWalk; ++u) {
    const bool in = w.k0 + u * kWave + ln < R;
    tt[u] = in ? g.type[w.vn[u]] : -1;
    ee[u] = in ? g.est[w.vn[u]] : 0;
    ll[u] = in ? g.loc[w.vn[u]] : -1;
  }
  walk_ids(g, R, w, w.k0 + kWalkBlock);
#pragma unroll
  for (int u = 0; u < kWalk; ++u) {
    const uint64_t mk = ballot(tt[u] == t);
    if (tt[u] == t) {
      const int s = (tail + int(lanes_below(mk))) & (kGreedyRing - 1);
      Q.out[s] = int32_t(w.k0 + u * kWave + ln);
      Q.est[s] = ee[u];
      Q.loc[s] = ll[u];
    }
    tail += int(__popcll(mk));
  }
  w.k0 += kWalkBlock;
  return tail;
}

// The type's futures in output order (nc <= W <= 64 candidates).  Every wave
// follows the same counts: the batch tabulated in a step is the one routed in
// the next, and the walk never overwrites a batch still in work.
template <int W, int IB>
__device__ void route_type_batches(const GreedyArgs& g, int64_t R, const Cand& cd, int32_t t, int nc, Queue& Q,
                                   bool& bad) {
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  const int q = lane_id() & (W - 1);
  int64_t my_load = q < nc ? cd.load[q] : INT64_MAX;
  Walk w;
  if (wv == 1) {
    w.k0 = 0;
    walk_ids(g, R, w, 0);
  }
  if (threadIdx.x == 0) {
    Q.tail[0] = 0;
    Q.done[0] = 0;
  }
  lds_barrier();
  int head = 0, routing = 0;  // the batch being routed: [head, head + routing)
  for (int step = 0;; ++step) {
    const int tail = Q.tail[step & 1];
    const bool done = Q.done[step & 1] != 0;
    const int next = head + routing;
    int build = tail - next;
    build = build >= kWave ? kWave : (done ? build : 0);
    if (done && build == 0 && routing == 0) break;  // the same on every wave
    if (wv == 0) {
      if (routing > 0) route_batch<W, IB>(g, cd, t, nc, head, routing, Q, Q.tab[(step + 1) & 1], my_load, bad);
    } else if (wv == 1) {
      int nt = tail;
      if (!done && tail - head + kWalkBlock <= kGreedyRing) nt = walk_block(g, R, t, w, Q, tail);
      if (lane_id() == 0) {
        Q.tail[(step + 1) & 1] = nt;
        Q.done[(step + 1) & 1] = w.k0 >= R ? 1 : 0;
      }
    } else if (build > 0) {
      build_table<W, IB>(g, cd, t, nc, wv - 2, next, build, Q, Q.tab[step & 1]);
    }
    head = next;
    routing = build;
    lds_barrier();
  }
}

// More than 64 candidates: every future scans them lane-parallel in LDS.
__device__ void route_type_lds(const GreedyArgs& g, int64_t R, const Cand& cd, int32_t t, int nc, bool& bad) {
  const int ln = lane_id();
  for (int64_t k0 = 0; k0 < R; k0 += kWave) {
    const int64_t k = k0 + ln;
    int32_t tk = -1, lk = -1;
    int64_t ek = 0;
    if (k < R) {
      const int32_t v = g.order[k];
      tk = g.type[v];
      ek = g.est[v];
      lk = g.loc[v];
    }
    uint64_t mk = ballot(tk == t);
    while (mk != 0) {  // this chunk's futures of type t, in order
      const int src = __builtin_ctzll(mk);
      mk &= mk - 1;
      const int64_t e = readlane_i64(ek, src);
      const int32_t l = readlane_i32(lk, src);
      const double a = double(e * 1000);
      const bool pinned = g.stateful && l >= 0 && cd.itype[l] == t;
      int qb;
      int64_t cb;
      if (pinned) {
        qb = cd.q_of[l];
        cb = cd.load[qb] + floordiv_exact(a, cd.speed[qb], cd.inv[qb]);
      } else {
        int64_t bc = INT64_MAX;
        int bq = INT32_MAX;
        for (int q = ln; q < nc; q += kWave) {  // ascending q per lane: strict < keeps the lowest
          int64_t c = cd.load[q] + floordiv_exact(a, cd.speed[q], cd.inv[q]);
          if (l >= 0 && l != cd.idx[q]) c += g.mig;
          if (c < bc) { bc = c; bq = q; }
        }
        cb = wave_min_i64(bc);
        qb = int(wave_min_i64(bc == cb ? int64_t(bq) : int64_t(INT32_MAX)));
      }
      if (ln == 0) {
        g.route[k0 + src] = cd.idx[qb];
        if (g.cost) g.cost[k0 + src] = cb;
        const int64_t nl = cd.load[qb] + floordiv_exact(a, cd.speed[qb], cd.inv[qb]);
        cd.load[qb] = nl;
        bad |= nl > NALAR_REM_MAX;
      }
      // One wavefront: its LDS accesses complete in program order, so the
      // next future's reads see this update; only the compiler must not
      // move them (a barrier would also wait for the stores above).
      __asm__ __volatile__("" ::: "memory");
    }
  }
}

__global__ __launch_bounds__(kGreedyThreads) void k_route_greedy(GreedyArgs g) {
  __shared__ int64_t s_load[NALAR_MAX_INSTANCES];   // running load of candidate q
  __shared__ double s_inv[NALAR_MAX_INSTANCES];
  __shared__ int32_t s_speed[NALAR_MAX_INSTANCES];
  __shared__ int32_t s_idx[NALAR_MAX_INSTANCES];    // instance id of candidate q
  __shared__ int32_t s_q[NALAR_MAX_INSTANCES];      // candidate of instance i (type t only)
  __shared__ int32_t s_itype[NALAR_MAX_INSTANCES];  // type of every instance
  __shared__ Queue Q;
  const int w = blockIdx.x;
  const int ln = lane_id();
  const int M = g.M;
  const int32_t t = g.inst_type[w];
  const bool finished = sort_finished(g.ctrl, g.passes_launched);
  const int64_t R = g.ctrl->n_ready;
  if (!finished) return;
  for (int j = threadIdx.x; j < M; j += kGreedyThreads) s_itype[j] = g.inst_type[j];
  __syncthreads();
  // only the lowest-index instance of each type runs its type's sequence
  for (int j0 = 0; j0 < w; j0 += kWave) {
    const int j = j0 + ln;
    if (ballot(j < w && s_itype[j] == t) != 0) return;  // the same on every wave
  }
  // every wave finds the candidates; the first writes them
  int nc = 0;
  for (int j0 = 0; j0 < M; j0 += kWave) {
    const int j = j0 + ln;
    const bool m = j < M && s_itype[j] == t;
    const uint64_t mk = ballot(m);
    if (m && threadIdx.x < kWave) {
      const int q = nc + int(lanes_below(mk));
      const int32_t sp = g.inst_speed[j];
      s_idx[q] = j;
      s_load[q] = g.inst_load[j];
      s_speed[q] = sp;
      s_inv[q] = sp >= 1 ? 1.0 / double(sp) : 0.0;
      s_q[j] = q;
    }
    nc += int(__popcll(mk));
  }
  __syncthreads();

  const Cand cd{s_load, s_inv, s_speed, s_idx, s_q, s_itype};
  bool bad = false;
  if (nc <= 8)
    route_type_batches<8, 3>(g, R, cd, t, nc, Q, bad);
  else if (nc <= 16)
    route_type_batches<16, 4>(g, R, cd, t, nc, Q, bad);
  else if (nc <= kWave)
    route_type_batches<kWave, 6>(g, R, cd, t, nc, Q, bad);
  else if (threadIdx.x < kWave)
    route_type_lds(g, R, cd, t, nc, bad);
  bad = ballot(bad) != 0;
  if (ln == 0 && bad)
    __hip_atomic_fetch_or(&g.host->aux_status, kStRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

hipError_t launch_route_greedy(hipStream_t s, const GreedyArgs& g) {
  if (g.M <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_route_greedy, dim3(g.M), dim3(kGreedyThreads), 0, s, g);
  return hipGetLastError();
}

}  // namespace nalar
