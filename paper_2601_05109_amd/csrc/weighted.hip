// Weighted routing (NALAR_ROUTE_WEIGHTED): route with a list of instances and
// weights (Table 2).  After ordering, the ready futures of each type that has
// instances of positive weight are dealt to those instances in proportion to
// their weights: the futures of type t, in output order, take sequence numbers
// j = 0, 1, 2, ...; with the weighted instances of t listed by ascending index,
// w[i] their weights and S their total, future j goes to the instance whose run
// of w[i] consecutive numbers in 0 .. S-1 holds j mod S.
//
// A future's sequence number is its rank among the futures of its type before
// it in the output order, which is a per-type prefix count over the order:
//   k_weighted_table   (one workgroup, before the sweep) the weighted instances
//                      sorted by (type, index) with the weight before each entry
//                      inside its type, the type's total and its first entry
//                      (the type's slot, which names it in the counts below);
//   k_weighted_count   one workgroup per tile of kWTile output positions counts
//                      the tile's futures per slot;
//   k_weighted_scan    (more than kWDirectTiles tiles) one workgroup per slot
//                      turns the tile counts into exclusive prefixes;
//   k_weighted_assign  each tile again: every future's rank inside the tile (in
//                      order: each wave's rows of 64 positions, lanes of equal
//                      slot ranked by ballots, behind the counts of the waves
//                      before) plus the tile prefix is its sequence number; the
//                      instance whose weight run holds it is found by a binary
//                      search, and route and cost are written.
// Futures pinned by NALAR_ROUTE_STATEFUL and futures of types with no weighted
// instance keep the route the pass gave them.
//
// All of it is latency: a few dependent loads and LDS searches per future.  So
// a tile is spread over a workgroup with four positions per thread (a tile per
// wave with sixteen left 15 tiles of a 15.3K ready set on 4 CUs: count 20.5 us,
// assign 36 us), every position's loads are issued together, the slot of a
// small type is one LDS read, the table is built from vector LDS reads (one entry
// at a time it took 24 us), and the kernels read the ready count on the device (no
// wait of the host between the sort and the routing).  With few tiles the assign
// kernel adds up the earlier tiles' counts itself instead of a scan launch.  Measured, the whole pass over 240K futures of ragged workflows, 15.3K of
// them ready, 200 instances: 170 -> 100 us.
#include "internal.hpp"

namespace nalar {

namespace {

constexpr int kWThreads = 256;
constexpr int kWWaves = kWThreads / kWave;
constexpr int kWItems = 4;
constexpr int kWTile = kWThreads * kWItems;   // positions per workgroup tile
// Up to this many tiles of the whole id space the assign kernel sums the
// earlier tiles' counts itself: one load per slot and tile, in flight together,
// against a launch of its own for the scan (about 4 us); beyond, the sum's
// length would show.  The line is drawn by the id space, since the host launches
// these kernels before the ready count is known: a large snapshot with few ready
// futures pays for the scan launch as well.
constexpr int64_t kWDirectTiles = 256;
constexpr int kWTableThreads = 1024;
constexpr int kSlotBits = 10;             // slots < NALAR_MAX_INSTANCES = 2^10
static_assert((1 << kSlotBits) == NALAR_MAX_INSTANCES, "slot bits");

// Within one wavefront LDS operations complete in program order; this only
// keeps the compiler from moving LDS accesses across it.
__device__ inline void wave_barrier() { __asm__ __volatile__("" ::: "memory"); }

__global__ __launch_bounds__(kWTableThreads) void k_weighted_table(WeightedArgs g) {
  // four entries per LDS read; the padding is of weight 0 and counts nowhere
  __shared__ __align__(16) int32_t s_type[NALAR_MAX_INSTANCES];
  __shared__ __align__(16) uint32_t s_w[NALAR_MAX_INSTANCES];
  const int M = g.M;
  const int i = int(threadIdx.x);
  int32_t t = INT32_MAX;
  uint32_t w = 0;
  if (i < M) {
    t = g.inst_type[i];
    w = g.inst_weight[i];
  }
  const bool bad = w > NALAR_WEIGHT_MAX;
  if (bad) w = 0;
  s_type[i] = t;
  s_w[i] = w;
  if (ballot(bad) != 0 && lane_id() == 0) flag_status(g.ctrl, kStInval);
  __syncthreads();
  int n = 0;
  if (i < M && w != 0) {
    const int4* t4 = reinterpret_cast<const int4*>(s_type);
    const uint4* w4 = reinterpret_cast<const uint4*>(s_w);
    int rank = 0, before_type = 0, in_type = 0;
    uint32_t cum = 0, tot = 0;
#pragma unroll 4
    for (int q = 0; q < (M + 3) / 4; ++q) {
      const int4 u = t4[q];
      const uint4 x = w4[q];
      const int32_t uu[4] = {u.x, u.y, u.z, u.w};
      const uint32_t ww[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int pos = ww[d] != 0 ? 1 : 0;
        const int lt = uu[d] < t ? pos : 0, eq = uu[d] == t ? pos : 0, lo = 4 * q + d < i ? eq : 0;
        before_type += lt;
        in_type += eq;
        rank += lt + lo;
        tot += eq ? ww[d] : 0u;
        cum += lo ? ww[d] : 0u;
      }
    }
    g.wt_type[rank] = t;
    g.wt_idx[rank] = i;
    g.wt_cum[rank] = cum;
    g.wt_tot[rank] = tot;
    g.wt_first[rank] = before_type;
    g.wt_cnt[rank] = in_type;
    n = 1;
  }
  // the number of entries: the weighted instances
  const int nw = int(__popcll(ballot(n != 0)));
  __shared__ int s_n[kWTableThreads / kWave];
  if (lane_id() == 0) s_n[threadIdx.x / kWave] = nw;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int q = 0; q < kWTableThreads / kWave; ++q) tot += s_n[q];
    *g.n_wt = tot;
  }
}

// Types and slots of the weighted instances in LDS (n entries), and the slot of
// every type below kTypeDirect (-1: no weighted instance).
struct WSlots {
  int32_t type[NALAR_MAX_INSTANCES];
  int32_t direct[kTypeDirect];
};

// Every thread of the workgroup calls; the caller's barrier follows.
__device__ inline void load_slots(const WeightedArgs& g, WSlots& S, int n) {
  for (int t = int(threadIdx.x); t < kTypeDirect; t += kWThreads) S.direct[t] = -1;
  __syncthreads();
  for (int i = int(threadIdx.x); i < n; i += kWThreads) {
    const int32_t t = g.wt_type[i];
    S.type[i] = t;
    if (g.wt_first[i] == i && uint32_t(t) < uint32_t(kTypeDirect)) S.direct[t] = i;
  }
}

// Slot of type t (its first weighted entry), or -1 without weighted instances.
__device__ inline int slot_of(const WSlots& S, int n, int32_t t) {
  if (uint32_t(t) < uint32_t(kTypeDirect)) return S.direct[t];
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (S.type[mid] < t) lo = mid + 1; else hi = mid;
  }
  return (lo < n && S.type[lo] == t) ? lo : -1;
}

// The futures at this thread's positions of a tile (wave w's rows follow those
// of the waves before it; row j of lane l at j * 64 + l): type (-1 past the
// end), id and state location, every load in flight together.
struct WItems {
  int32_t v[kWItems], t[kWItems], l[kWItems];
};

__device__ inline int64_t item_pos(int64_t tile, int j) {
  return tile * kWTile + int64_t(threadIdx.x / kWave) * (kWave * kWItems) + j * kWave + lane_id();
}

__device__ inline void load_items(const WeightedArgs& g, int64_t R, int64_t tile, WItems& it) {
#pragma unroll
  for (int j = 0; j < kWItems; ++j) {
    const int64_t k = item_pos(tile, j);
    it.v[j] = g.order[k < R ? k : 0];
  }
#pragma unroll
  for (int j = 0; j < kWItems; ++j) {
    it.t[j] = g.type[it.v[j]];
    it.l[j] = g.loc[it.v[j]];
  }
#pragma unroll
  for (int j = 0; j < kWItems; ++j)
    if (item_pos(tile, j) >= R) it.t[j] = -1;
}

// Slots of the positions, -1 for a future that keeps its route.
__device__ inline void item_slots(const WeightedArgs& g, const WSlots& S, int n, const WItems& it, int* sl) {
#pragma unroll
  for (int j = 0; j < kWItems; ++j) {
    sl[j] = it.t[j] >= 0 ? slot_of(S, n, it.t[j]) : -1;
    if (g.stateful && it.t[j] >= 0 && it.l[j] >= 0 && g.inst_type[it.l[j]] == it.t[j]) sl[j] = -1;
  }
}

__global__ __launch_bounds__(kWThreads) void k_weighted_count(WeightedArgs g) {
  __shared__ WSlots S;
  __shared__ uint32_t hist[NALAR_MAX_INSTANCES];
  const int64_t R = g.ctrl->n_ready;
  const int64_t tile = blockIdx.x;
  if (!sort_finished(g.ctrl, g.passes_launched) || tile * kWTile >= R) return;
  const int n = *g.n_wt;
  WItems it;
  load_items(g, R, tile, it);
  load_slots(g, S, n);
  for (int i = int(threadIdx.x); i < n; i += kWThreads) hist[i] = 0;
  __syncthreads();
  int sl[kWItems];
  item_slots(g, S, n, it, sl);
#pragma unroll
  for (int j = 0; j < kWItems; ++j)
    if (sl[j] >= 0) atomicAdd(&hist[sl[j]], 1u);
  __syncthreads();
  uint32_t* row = g.counts + tile * NALAR_MAX_INSTANCES;
  for (int i = int(threadIdx.x); i < n; i += kWThreads) row[i] = hist[i];
}

// Exclusive prefix over the tiles of one slot (one workgroup per slot; slots
// that are no type's first entry have no futures and return).
__global__ __launch_bounds__(kWThreads) void k_weighted_scan(WeightedArgs g) {
  __shared__ uint32_t s_part[kWWaves];
  const int s = blockIdx.x;
  if (!sort_finished(g.ctrl, g.passes_launched) || s >= *g.n_wt || g.wt_first[s] != s) return;
  const int64_t tiles = (g.ctrl->n_ready + kWTile - 1) / kWTile;
  uint32_t carry = 0;
  for (int64_t t0 = 0; t0 < tiles; t0 += kWThreads) {
    const int64_t t = t0 + threadIdx.x;
    const uint32_t c = t < tiles ? g.counts[t * NALAR_MAX_INSTANCES + s] : 0u;
    const uint32_t inc = wave_incl_scan_u32(c);
    if (lane_id() == kWave - 1) s_part[threadIdx.x / kWave] = inc;
    __syncthreads();
    uint32_t before = carry;
    uint32_t total = 0;
    for (int w = 0; w < kWWaves; ++w) {
      before += w < int(threadIdx.x / kWave) ? s_part[w] : 0u;
      total += s_part[w];
    }
    if (t < tiles) g.counts[t * NALAR_MAX_INSTANCES + s] = before + inc - c;
    carry += total;
    __syncthreads();
  }
}

// direct: the counts are per tile (summed here), else already prefixes.
__global__ __launch_bounds__(kWThreads) void k_weighted_assign(WeightedArgs g, int direct) {
  __shared__ WSlots S;
  __shared__ int32_t s_idx[NALAR_MAX_INSTANCES];
  __shared__ uint32_t s_cum[NALAR_MAX_INSTANCES];
  __shared__ uint32_t s_tot[NALAR_MAX_INSTANCES];
  __shared__ int32_t s_cnt[NALAR_MAX_INSTANCES];
  __shared__ uint32_t run[kWWaves][NALAR_MAX_INSTANCES];  // per wave: counts, then the next sequence number
  const int wv = int(threadIdx.x) / kWave;
  const int64_t R = g.ctrl->n_ready;
  const int64_t tile = blockIdx.x;
  if (!sort_finished(g.ctrl, g.passes_launched) || tile * kWTile >= R) return;
  const int n = *g.n_wt;
  WItems it;
  load_items(g, R, tile, it);
  int64_t est[kWItems];
#pragma unroll
  for (int j = 0; j < kWItems; ++j) est[j] = g.est[it.v[j]];
  load_slots(g, S, n);
  for (int i = int(threadIdx.x); i < n; i += kWThreads) {
    s_idx[i] = g.wt_idx[i];
    s_cum[i] = g.wt_cum[i];
    s_tot[i] = g.wt_tot[i];
    s_cnt[i] = g.wt_cnt[i];
#pragma unroll
    for (int w = 0; w < kWWaves; ++w) run[w][i] = 0;
  }
  __syncthreads();
  int sl[kWItems];
  item_slots(g, S, n, it, sl);
#pragma unroll
  for (int j = 0; j < kWItems; ++j)
    if (sl[j] >= 0) atomicAdd(&run[wv][sl[j]], 1u);
  __syncthreads();
  // each wave's first sequence number per slot: the futures of earlier tiles
  // and of the waves before it in this one
  for (int i = int(threadIdx.x); i < n; i += kWThreads) {
    uint32_t base = 0;
    if (direct) {
#pragma unroll 8
      for (int64_t q = 0; q < tile; ++q) base += g.counts[q * NALAR_MAX_INSTANCES + i];
    } else {
      base = g.counts[tile * NALAR_MAX_INSTANCES + i];
    }
#pragma unroll
    for (int w = 0; w < kWWaves; ++w) {
      const uint32_t c = run[w][i];
      run[w][i] = base;
      base += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kWItems; ++j) {
    // lanes of equal slot, ranked by lane (positions ascend with the lane)
    const bool valid = sl[j] >= 0;
    const uint32_t s = valid ? uint32_t(sl[j]) : 0u;
    uint64_t peers = ballot(valid);
    if (peers == 0) continue;
#pragma unroll
    for (int b = 0; b < kSlotBits; ++b) {
      const bool bit = (s >> b) & 1u;
      const uint64_t m = ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint64_t below = peers & lanemask_lt();
    uint32_t seq = 0;
    if (valid) seq = run[wv][s] + uint32_t(__popcll(below));
    wave_barrier();
    if (valid && below == 0) run[wv][s] += uint32_t(__popcll(peers));
    wave_barrier();
    if (!valid) continue;
    // the entry whose weight run holds seq mod S
    const uint32_t r = seq % s_tot[s];
    int lo = int(s), hi = int(s) + s_cnt[s] - 1;  // last entry with cum <= r
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_cum[mid] <= r) lo = mid; else hi = mid - 1;
    }
    const int32_t inst = s_idx[lo];
    const int64_t k = item_pos(tile, j);
    const int32_t l = it.l[j];
    g.route[k] = inst;
    if (g.cost) {
      const int32_t sp = g.inst_speed[inst];
      g.cost[k] = g.inst_load[inst] + floordiv_exact(double(est[j] * 1000), sp, 1.0 / double(sp)) +
                  ((l >= 0 && l != inst) ? g.mig : 0);
    }
  }
}

}  // namespace

int64_t weighted_tiles(int64_t N) { return (N + kWTile - 1) / kWTile; }

hipError_t launch_weighted_table(hipStream_t s, const WeightedArgs& g) {
  if (g.M <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_weighted_table, dim3(1), dim3(kWTableThreads), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_route_weighted(hipStream_t s, const WeightedArgs& g, void (*mark)(void*, const char*),
                                 void* ctx) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  hipError_t e;
  const int64_t tiles = weighted_tiles(g.N);  // at most: the ready futures' tiles return early past R
  const bool direct = tiles <= kWDirectTiles;
  mark(ctx, "weighted_count");
  hipLaunchKernelGGL(k_weighted_count, dim3(unsigned(tiles)), dim3(kWThreads), 0, s, g);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!direct) {
    mark(ctx, "weighted_scan");
    hipLaunchKernelGGL(k_weighted_scan, dim3(unsigned(g.M)), dim3(kWThreads), 0, s, g);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  mark(ctx, "weighted_assign");
  hipLaunchKernelGGL(k_weighted_assign, dim3(unsigned(tiles)), dim3(kWThreads), 0, s, g, direct ? 1 : 0);
  return hipGetLastError();
}

}  // namespace nalar
