"""GPU parity at the edges of the dispatch rules: sizes and values at which a
pass moves from one kernel or number format to another, each against the CPU
oracle, bit-exact."""
import numpy as np
import pytest

from paper_2601_05109_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts too
    pytest.skip("no GPU", allow_module_level=True)

from paper_2601_05109_amd import nalar  # noqa: E402
import oracle  # noqa: E402
from test_gpu_parity import _one_type, assert_parity, check, policy, say  # noqa: E402,F401
from test_gpu_store_incremental import feed, store_pass  # noqa: E402


# ---------------------------------------------------------------- greedy routing

@pytest.mark.parametrize("n_inst", [1, 2, 8, 9, 16, 17, 64])
@pytest.mark.parametrize("spread", ["near", "limit", "far", "huge-estimates", "huge-penalty"])
def test_greedy_relative_costs(policy, n_inst, spread):  # noqa: F811
    """The greedy chain's 32-bit relative costs: loads close together; loads at
    the distance where a relative load stops fitting (2^29 us with 8 candidates,
    2^28 with 16, 2^26 with 64); loads up to 2^60 apart; service times and a
    migration penalty that never fit.  5,000 futures wrap the queue and leave a
    partial batch."""
    rng = np.random.default_rng(n_inst * 31 + len(spread))
    n = 5000
    loads = rng.integers(0, 10**6, n_inst)
    est = rng.integers(0, 10**6, n)
    mig = 200_000
    if spread == "limit":
        loads = loads + rng.choice([0, 1 << 26, (1 << 26) - 1, 1 << 28, 1 << 29, (1 << 29) - 1], n_inst)
    elif spread == "far":
        loads = loads + rng.choice([0, 1 << 31, 1 << 40, (1 << 60) - 10**6], n_inst)
    elif spread == "huge-estimates":
        est[rng.random(n) < 0.01] = 1 << 36
    elif spread == "huge-penalty":
        mig = 1 << 60
    loc = np.where(rng.random(n) < 0.4, rng.integers(0, n_inst, n), -1)
    p = _one_type(n_inst, np.minimum(loads, 1 << 60), rng.integers(300, 3000, n_inst), est, loc=loc, mig=mig)
    G = nalar.NALAR_ROUTE_GREEDY
    check(policy, p, f"greedy {n_inst} {spread}", policy=G)
    check(policy, p, f"greedy {n_inst} {spread} stateful", policy=G | nalar.NALAR_ROUTE_STATEFUL)


# ---------------------------------------------------------------- weighted routing

def _independent(n, m, n_types, seed, done_share=0.0):
    """n one-future workflows of n_types types over m instances (some types
    without one), with state on an instance for half the futures."""
    rng = np.random.default_rng(seed)
    now = 10_000
    return wl.Problem(f"independent-{n}", now, 150_000, np.arange(n, dtype=np.int32),
                      rng.integers(0, n_types, n).astype(np.int32), rng.integers(0, 10**6, n).astype(np.int64),
                      (rng.random(n) < done_share).astype(np.uint8),
                      np.where(rng.random(n) < 0.5, rng.integers(0, m, n), -1).astype(np.int32),
                      np.zeros(n + 1, np.int32), np.zeros(0, np.int32),
                      (now + rng.integers(0, 10**7, n)).astype(np.int64),
                      rng.integers(0, n_types, m).astype(np.int32), rng.integers(0, 10**6, m).astype(np.int64),
                      rng.integers(300, 3000, m).astype(np.int32), wf_contiguous=True)


@pytest.mark.parametrize("n,m,n_types", [(1, 1, 1), (64, 5, 2), (1023, 40, 63), (1024, 40, 64), (1025, 40, 65),
                                         (4097, 1024, 130), (262_144, 64, 8), (262_145, 64, 8), (300_001, 200, 70)])
def test_weighted_tiles(policy, n, m, n_types):  # noqa: F811
    """Weighted routing around its tile of 1,024 positions, the types with and
    without a direct slot (64), and 256 tiles, where the scan launch begins."""
    p = _independent(n, m, n_types, n + m)
    W = nalar.NALAR_ROUTE_WEIGHTED
    w = np.random.default_rng(n).integers(0, 4, m).astype(np.uint32)
    for rep in range(2):  # a first pass (tiled sort) and a planned one
        check(policy, p, f"weighted n={n} pass {rep}", policy=W, weights=w)
    check(policy, p, f"weighted stateful n={n}", policy=W | nalar.NALAR_ROUTE_STATEFUL | nalar.NALAR_ORDER_LPT,
          weights=w)


# ---------------------------------------------------------------- incremental store passes

def _fan_in_store(n, W, seed):
    """Workflow 0: up to 300 futures, the last depending on all others (more than
    64: expanded by a workgroup); then one-future workflows with few distinct
    keys, so that ties are broken by (workflow, id)."""
    rng = np.random.default_rng(seed)
    k = min(n, 300)
    wf = np.zeros(n, np.int32)
    wf[k:] = rng.integers(0, W, n - k)
    counts = np.zeros(n, np.int64)
    counts[k - 1] = k - 1
    dep_off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dep_idx = np.arange(k - 1, dtype=np.int32)
    now, M, K = 10_000, 12, 3
    return wl.Problem(f"fan-in-{n}", now, 150_000, wf, rng.integers(0, K, n).astype(np.int32),
                      rng.integers(1, 4 + n // 300, n).astype(np.int64) * 100, np.zeros(n, np.uint8),
                      np.where(rng.random(n) < 0.5, rng.integers(0, M, n), -1).astype(np.int32), dep_off, dep_idx,
                      (now + rng.integers(1, 4 + n // 300, W) * 1000).astype(np.int64), (np.arange(M) % K).astype(np.int32),
                      rng.integers(0, 10**6, M).astype(np.int64), rng.integers(300, 3000, M).astype(np.int32),
                      wf_contiguous=False)


def _extended(p, done_ids, parents, seed):
    """p with the ids done and one child appended per parent."""
    rng = np.random.default_rng(seed)
    t = len(parents)
    done = p.done.copy()
    done[done_ids] = 1
    cat = lambda a, b: np.concatenate([a, np.asarray(b, a.dtype)])  # noqa: E731
    return wl.Problem(p.name, p.now_us, p.migration_cost_us, cat(p.wf, p.wf[parents]),
                      cat(p.type, rng.integers(0, 3, t)), cat(p.est_us, rng.integers(1, 500, t)), cat(done, np.zeros(t)),
                      cat(p.loc, np.full(t, -1)), cat(p.dep_off, p.dep_off[-1] + np.arange(1, t + 1)),
                      cat(p.dep_idx, parents), p.deadline_us, p.inst_type, p.inst_load_us, p.inst_speed_permille,
                      wf_contiguous=False)


@pytest.mark.parametrize("order", [0, nalar.NALAR_ORDER_LPT, nalar.NALAR_ORDER_SRTF])
@pytest.mark.parametrize("W", [3, 65_536, 65_537])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 65, 66, 255, 257, 2049, 4097, 70_001])
def test_store_incremental_sizes(n, W, order):
    """Incremental passes around the sizes their kernels work in (words of 32 and
    64 futures, units of 256, steps of 2,048 and 4,096), and around 65,536
    workflows, up to which the records carry the workflow of a tie; under each order,
    with splitters cut for it."""
    p = _fan_in_store(n, W, n + W)
    with nalar.Policy() as pol, nalar.Store(pol) as st:
        prev = feed(st, p, 0, None)
        g, _ = store_pass(pol, st, p, policy=order)
        assert_parity(g, oracle.run(p, policy=order), "full")
        rng = np.random.default_rng(n)
        for tick in range(3):
            every = np.arange(min(n, 300) - 1, dtype=np.int64)
            ids = every[tick::2] if tick < 2 else rng.choice(p.n_nodes, min(p.n_nodes, 40), replace=False)
            p = _extended(p, ids, rng.integers(0, p.n_nodes, 1 + tick * 40), tick)
            prev = feed(st, p, *prev)
            g, inc = store_pass(pol, st, p, policy=order)
            assert_parity(g, oracle.run(p, policy=order), f"n={n} W={W} order={order} tick {tick}")
            say(f"n={n} W={W} order={order} tick {tick}: incremental {inc}, reason {st.last_fallback}")
            assert inc


# ---------------------------------------------------------------- wave sweep

def _chained(W, n, seed, heavy):
    """W contiguous workflows of n futures, each on the one before it in a window
    of 70 (mostly the last one: as deep as it is long) and up to two more."""
    rng = np.random.default_rng(seed)
    counts, flat = [], []
    for w in range(W):
        for i in range(n):
            par = set()
            if i:
                par.add(i - 1 if rng.random() < 0.8 else int(rng.integers(max(0, i - 70), i)))
                for _ in range(int(rng.integers(0, 3))):
                    par.add(int(rng.integers(max(0, i - 70), i)))
                if heavy and i % 17 == 16:
                    par |= set(int(x) for x in rng.integers(0, i, 6))
            counts.append(len(par))
            flat += [w * n + q for q in sorted(par)]
    N, M, K, now = W * n, 9, 3, 5_000
    return wl.Problem(f"chained-{W}x{n}", now, 150_000, np.repeat(np.arange(W, dtype=np.int32), n),
                      rng.integers(0, K, N).astype(np.int32), rng.integers(0, 10**5, N).astype(np.int64),
                      (np.tile(np.arange(n), W) < 3 * n // 10).astype(np.uint8),
                      np.where(rng.random(N) < 0.5, rng.integers(0, M, N), -1).astype(np.int32),
                      np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), np.asarray(flat, np.int32),
                      (now + rng.integers(0, 10**7, W)).astype(np.int64), (np.arange(M) % K).astype(np.int32),
                      rng.integers(0, 10**6, M).astype(np.int64), rng.integers(300, 3000, M).astype(np.int32),
                      wf_contiguous=True)


@pytest.mark.parametrize("heavy", [False, True])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 128, 129, 255, 257, 512])
def test_wave_sweep_orders(policy, n, heavy):  # noqa: F811
    """One wave per workflow (or pair) around its groups of 64 positions, with
    ids in topological order (no counters), reversed and shuffled inside each
    workflow, and with one workflow of several out of order."""
    W = 11
    p = _chained(W, n, n, heavy)
    local = np.tile(np.arange(n), W)
    base = np.repeat(np.arange(W) * n, n)
    rng = np.random.default_rng(n)
    shuffled = np.concatenate([w * n + rng.permutation(n) for w in range(W)])
    one = np.concatenate([w * n + (rng.permutation(n) if w == 3 else np.arange(n)) for w in range(W)])
    for name, perm in (("topological", np.arange(W * n)), ("reversed", base + n - 1 - local),
                       ("shuffled", shuffled), ("one-shuffled", one)):
        check(policy, wl.relabel(p, perm), f"{name} n={n} heavy={heavy}")


# ---------------------------------------------------------------- grouping by workflow

@pytest.mark.parametrize("W,n", [(1, 5000), (3, 700), (255, 30), (256, 9), (257, 9), (1023, 3), (1024, 5), (2048, 1), (2049, 2), (4097, 3),
                                 (16_384, 2), (16_385, 2), (300, 700)])
def test_grouping_by_many_workflows(policy, W, n):  # noqa: F811
    """Ids of W workflows in random order, around the counts at which the
    grouping changes (256 and 16,384 workflows, and few of them) and its tile grows (2,048, 4,096
    ...), with workflows left empty and one larger than the others."""
    rng = np.random.default_rng(W + n)
    p = _chained(W, n, W, False)
    keep = np.flatnonzero((p.wf % 7 != 3) | (p.wf == W - 1))  # some workflows without futures
    new = np.full(p.n_nodes, -1)
    new[keep] = np.arange(keep.size)
    cnt = np.diff(p.dep_off)[keep]
    idx = np.concatenate([p.dep_idx[p.dep_off[v]:p.dep_off[v + 1]] for v in keep]) if cnt.sum() else p.dep_idx[:0]
    q = wl.Problem(p.name, p.now_us, p.migration_cost_us, *[np.ascontiguousarray(getattr(p, f)[keep])
                                                            for f in wl.Problem.NODE_FIELDS],
                   np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32), new[idx].astype(np.int32), p.deadline_us,
                   p.inst_type, p.inst_load_us, p.inst_speed_permille)
    perm = rng.permutation(q.n_nodes)
    r = wl.relabel(q, perm)
    for rep in range(2):
        check(policy, r, f"grouped W={W} n={n} pass {rep}", flags=0)


@pytest.mark.parametrize("W,n,counted", [(8192, 3, True), (8193, 3, False), (8193, 23, False), (8193, 24, True),
                                         (16_384, 23, False), (16_384, 24, True), (16_385, 24, False)])
def test_grouping_of_small_workflows(policy, W, n, counted):  # noqa: F811
    """Many small workflows with ids in random order: the radix passes group what
    the counting kernels' tiles of 8,192 ids would leave to a few workgroups."""
    p = _independent(W * n, 24, 5, W + n)
    rng = np.random.default_rng(n)
    p = p.copy(wf=rng.permutation(np.repeat(np.arange(W, dtype=np.int32), n)),
               deadline_us=(p.now_us + rng.integers(0, 10**7, W)).astype(np.int64), wf_contiguous=False)
    policy.set_timing(True)
    try:
        for rep in range(2):
            check(policy, p, f"{W} workflows of {n} pass {rep}")
            assert ("group_count" in [k for k, _ in policy.timing()]) == counted
    finally:
        policy.set_timing(False)


# ---------------------------------------------------------------- bin sort

@pytest.mark.parametrize("equal", [1, 31, 33, 127, 128, 129, 300])
def test_bin_sort_equal_keys(equal):
    """Ready sets in which `equal` futures share each key, around the counts at
    which a bin ranks mates one by one or by a network, over enough futures for
    the bins of a full pass (1.2M: more bins than workgroups resident) and of an
    incremental store pass (ties by workflow and id)."""
    n = 1_200_000
    rng = np.random.default_rng(equal)
    W = 200
    wf = np.repeat(np.arange(W), n // W).astype(np.int32)
    p = _independent(n, 24, 5, equal)
    p = p.copy(wf=wf, deadline_us=np.full(W, p.now_us + 10**7, np.int64),
               est_us=(rng.permutation(n) // equal).astype(np.int64))
    with nalar.Policy() as pol:
        for rep in range(2):
            check(pol, p, f"{equal} equal keys pass {rep}")
    q = _independent(90_000, 24, 5, equal)
    q = q.copy(wf=rng.integers(0, W, 90_000).astype(np.int32), deadline_us=np.full(W, q.now_us + 10**7, np.int64),
               est_us=(rng.permutation(90_000) // equal).astype(np.int64), wf_contiguous=False)
    with nalar.Policy() as pol, nalar.Store(pol) as st:
        prev = feed(st, q, 0, None)
        store_pass(pol, st, q)
        for tick in range(2):
            q = _extended(q, rng.choice(q.n_nodes, 50, replace=False), rng.integers(0, q.n_nodes, 60), tick)
            prev = feed(st, q, *prev)
            g, inc = store_pass(pol, st, q)
            assert inc, st.last_fallback
            assert_parity(g, oracle.run(q), f"{equal} equal keys, store tick {tick}")


# ---------------------------------------------------------------- record sweep

def _grown_workflows(sizes, seed):
    """Workflows of these sizes with ids by creation, the workflows interleaved:
    most futures independent, the others on one earlier future (the last one, any,
    or the first: a hub), some on several, a few on hundreds."""
    rng = np.random.default_rng(seed)
    sizes = np.asarray(sizes)
    W, N = len(sizes), int(sizes.sum())
    first = np.concatenate([[0], np.cumsum(sizes)])
    kinds = rng.choice(6, size=N, p=[0.62, 0.12, 0.12, 0.08, 0.055, 0.005])
    kinds[:sizes[0]] = 1  # one workflow is a single chain: as deep as it is long
    counts, flat = np.zeros(N, np.int64), []
    for w in range(W):
        for i in range(sizes[w]):
            k = kinds[first[w] + i]
            if k == 0 or i < 2 and k != 1 or i == 0:
                continue
            if k == 1:
                par = [i - 1]
            elif k == 2:
                par = [int(rng.integers(0, i))]
            elif k == 3:
                par = [0]
            elif k == 4:
                par = [int(x) for x in rng.integers(0, i, int(rng.integers(2, 6)))]
            else:
                par = [int(x) for x in rng.integers(0, i, int(rng.integers(33, 300)))]
            counts[first[w] + i] = len(par)
            flat += [int(first[w]) + q for q in par]
    M, K, now = 40, 6, 5_000
    p = wl.Problem(f"grown-{W}", now, 150_000, np.repeat(np.arange(W, dtype=np.int32), sizes),
                   rng.integers(0, K, N).astype(np.int32), rng.integers(0, 10**6, N).astype(np.int64),
                   (rng.random(N) < 0.1).astype(np.uint8),
                   np.where(rng.random(N) < 0.5, rng.integers(0, M, N), -1).astype(np.int32),
                   np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), np.asarray(flat, np.int32),
                   (now + rng.integers(0, 10**7, W)).astype(np.int64), (np.arange(M) % K).astype(np.int32),
                   rng.integers(0, 10**6, M).astype(np.int64), rng.integers(300, 3000, M).astype(np.int32),
                   wf_contiguous=True)
    slots = np.argsort(rng.permutation(N) // 3, kind="stable")  # any interleaving
    owner = p.wf[slots]
    perm = np.argsort(owner, kind="stable")
    return wl.relabel(p, perm), p


@pytest.mark.parametrize("W,n", [(230, 520), (120, 1024), (118, 1025), (60, 2048), (59, 2049), (40, 3073), (9, 14_000),
                                 (9, 19_457), (9, 21_505), (300, 530)])
def test_record_sweep(W, n):
    """Workflows around whole chunks of 1,024 positions and around the chunks kept
    in LDS (19, or 9 for more workflows than the chip holds at once; the last size:
    two such workflows among 298 small ones), ids by creation: the first pass sorts in
    tiles, the next ones take the record sweep; under other policies; with a
    dependency on another workflow; and with ids that are not in topological order,
    which go back to the block sweep."""
    sizes = np.full(W, n)
    if W > 256:
        sizes[1:3] = 10_500
    p, grouped = _grown_workflows(sizes, W + n)
    with nalar.Policy() as pol:
        pol.set_timing(True)
        for rep, policy in enumerate((0, 0, nalar.NALAR_ORDER_LPT, nalar.NALAR_ORDER_SRTF | nalar.NALAR_ROUTE_STATEFUL)):
            check(pol, p, f"records W={W} n={n} pass {rep}", policy=policy)
            assert rep not in (1, 2) or "records" in [k for k, _ in pol.timing()]
        pol.set_timing(False)
        q = p.copy()
        v = np.flatnonzero((np.diff(q.dep_off) == 1) & (q.wf != q.wf[0]))[5]
        q.dep_idx[q.dep_off[v]] = 0                         # a lower id, of another workflow
        assert oracle.run(q).status == oracle.EINVAL
        check(pol, q, f"records W={W} n={n} foreign dependency")
        check(pol, p, f"records W={W} n={n} after it")
        rng = np.random.default_rng(n)
        mixed = wl.relabel(grouped, rng.permutation(p.n_nodes))
        for rep in range(4):
            check(pol, mixed if rep % 2 == 0 else p, f"records W={W} n={n} order {rep}")
    with nalar.Policy() as pol:
        for rep in range(2):
            dp = nalar.DeviceProblem.from_host(p)
            out = nalar.DeviceResult.alloc(dp.n_nodes, rem=False)
            assert pol.run_pass(dp, out) == nalar.NALAR_OK
            o = oracle.run(p)
            R = out.n_ready
            assert R == o.n_ready and np.array_equal(out.order[:R].cpu().numpy(), o.order)
            assert np.array_equal(out.cost[:R].cpu().numpy(), o.cost)


def _rooted(W, n, deps_of, seed):
    """W workflows of n futures: a finished root, its children, and for each
    (i, parents) of deps_of(w, rng) a future i of many dependencies; ids by creation,
    the workflows interleaved (position i of every workflow before i + 1)."""
    rng = np.random.default_rng(seed)
    lists = [[[]] + [[0]] * (n - 1) for _ in range(W)]
    for w in range(W):
        for i, par in deps_of(w, rng):
            lists[w][i] = [int(q) for q in par]
    done = np.zeros((W, n), np.uint8)
    done[:, 0] = 1
    done[::3, 1:] = 1                      # every third workflow: only its futures of many dependencies are left
    for w in range(W):
        for i, par in enumerate(lists[w]):
            if len(par) > 1:
                done[w, i] = 0
    counts = np.array([len(par) for ls in lists for par in ls], np.int64)
    flat = np.array([w * n + q for w, ls in enumerate(lists) for par in ls for q in par], np.int64)
    N, M, K, now = W * n, 40, 6, 5_000
    p = wl.Problem(f"rooted-{W}x{n}", now, 150_000, np.repeat(np.arange(W, dtype=np.int32), n),
                   rng.integers(0, K, N).astype(np.int32), rng.integers(0, 10**6, N).astype(np.int64), done.reshape(-1),
                   np.where(rng.random(N) < 0.5, rng.integers(0, M, N), -1).astype(np.int32),
                   np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), flat.astype(np.int32),
                   (now + rng.integers(0, 10**7, W)).astype(np.int64), (np.arange(M) % K).astype(np.int32),
                   rng.integers(0, 10**6, M).astype(np.int64), rng.integers(300, 3000, M).astype(np.int32),
                   wf_contiguous=True)
    local, w = np.tile(np.arange(n), W), np.repeat(np.arange(W), n)
    return wl.relabel(p, local * W + w)


def test_record_sweep_fan_ins_created_together():
    """One fan-in over a whole workflow each, all created last (map/reduce sessions
    started together): the fan-ins' ids lie side by side, and whatever takes their
    dependencies must spread over the workflows' workgroups.  Taken by the one
    workgroup that holds their ids it was 4.6 ms at 256 workflows of 4,098 futures,
    0.03 ms without; the bound leaves a factor of ten to either side."""
    W, n = 256, 2050
    p = _rooted(W, n, lambda w, rng: [(n - 1, range(1, n - 1))], 1)
    with nalar.Policy() as pol:
        pol.set_timing(True)
        for rep in range(3):
            check(pol, p, f"fan-ins pass {rep}")
            ms = dict(pol.timing())
            say(f"  {ms}")
            if rep:
                assert ms["records"] < 0.3


@pytest.mark.parametrize("n_many,deg", [(1, 33), (1, 1200), (64, 33), (65, 40), (700, 34)])
def test_record_sweep_many_dependencies(n_many, deg):
    """Futures of more than 32 dependencies, one to 700 in a workflow (a chunk of
    the sweep lists 64 of them, the others push alone): ready and blocked ones, and
    the problems only they have: a dependency on another workflow, on itself, at a
    higher id (the block sweep then does the pass) and in a cycle."""
    W, n = 100, 2100

    def deps_of(w, rng):
        return [(i, rng.choice(np.arange(1, n - n_many), deg, replace=False)) for i in range(n - n_many, n)]

    p = _rooted(W, n, deps_of, n_many + deg)
    deg_of = np.diff(p.dep_off)
    many = np.flatnonzero(deg_of > 32)
    assert many.size == W * n_many
    ref = oracle.run(p)
    assert 0 < np.isin(many, ref.order).sum() < many.size    # some ready, some blocked
    v = int(many[many.size // 2])
    other = int(np.flatnonzero(p.wf != p.wf[v])[7])
    later = int(p.n_nodes - W + p.wf[v])                     # the last future of v's workflow
    cases = [("foreign", v, other, oracle.EINVAL), ("itself", v, v, oracle.ECYCLE)]
    if later != v:
        cases.append(("higher", v, later, oracle.OK))
    with nalar.Policy() as pol:
        pol.set_timing(True)
        for rep, policy in enumerate((0, 0, nalar.NALAR_ORDER_LPT)):
            check(pol, p, f"many {n_many}x{deg} pass {rep}", policy=policy)
            assert rep == 0 or "records" in [k for k, _ in pol.timing()]
        for name, at, dep, status in cases:
            q = p.copy()
            q.dep_idx[q.dep_off[at] + deg // 2] = dep
            assert oracle.run(q).status == status
            check(pol, q, f"many {n_many}x{deg} {name}")
            for rep in range(3):
                check(pol, p, f"many {n_many}x{deg} after {name} {rep}")
        if later != v:                                       # higher, and the other way round: a cycle
            q.dep_idx[q.dep_off[later] + 1] = v
            assert oracle.run(q).status == oracle.ECYCLE
            check(pol, q, f"many {n_many}x{deg} cycle")
            check(pol, p, f"many {n_many}x{deg} after the cycle")


def test_store_greedy_without_instances_after_a_load_overflow():
    """A load overflow of one greedy pass is not reported by the next pass of the
    handle that has nothing to route: an incremental store pass without instances."""
    G = nalar.NALAR_ROUTE_GREEDY
    p = _independent(500, 4, 3, 1).copy(loc=np.full(500, -1, np.int32), wf_contiguous=False)
    none = {f: getattr(p, f)[:0].copy() for f in ("inst_type", "inst_load_us", "inst_speed_permille")}
    p = p.copy(**none)
    n = 5000
    over = _one_type(1, np.array([1 << 60]), np.array([1]), np.full(n, (1 << 40) - 1, np.int64))
    assert oracle.run(over, policy=G).status == oracle.ERANGE
    with nalar.Policy() as pol, nalar.Store(pol) as st:
        prev = feed(st, p, 0, None)
        store_pass(pol, st, p, policy=G)
        check(pol, over, "load overflow", policy=G)
        p = p.copy()
        p.done[:40] = 1
        prev = feed(st, p, *prev)
        g, inc = store_pass(pol, st, p, policy=G)
        assert inc, st.last_fallback
        assert_parity(g, oracle.run(p, policy=G), "without instances")


@pytest.mark.parametrize("first", ["ordered", "unordered"])
def test_record_sweep_is_left_alone_on_unordered_ids(first):
    """A stream of snapshots whose ids are not in topological order never takes the
    record sweep (which would do each pass twice), one that comes into order takes
    it again within the passes between two looks, and one pass done twice is what a
    stream that falls out of order costs."""
    p, grouped = _grown_workflows(np.full(150, 900), 3)
    mixed = wl.relabel(grouped, np.random.default_rng(3).permutation(p.n_nodes))
    with nalar.Policy() as pol:
        pol.set_timing(True)

        def took_records(snapshot, passes):
            taken = []
            for rep in range(passes):
                check(pol, snapshot, f"{snapshot is p} {rep}")
                taken.append("records" in [k for k, _ in pol.timing()])
            return taken

        if first == "ordered":
            assert took_records(p, 4) == [False, True, True, True]
            assert sum(took_records(mixed, 12)) == 1
        else:
            assert not any(took_records(mixed, 12))
        assert any(took_records(p, 18))


@pytest.mark.parametrize("seeds", [8_000, 10_000, 40_000])
def test_store_delta_behind_idle_passes(seeds):
    """A delta of many futures behind passes without any: above 8,192 seeds the
    rounds after the first get launches of their own, whatever the passes before
    had to do (one workgroup takes them otherwise).  Chains of two and fan-ins make
    several rounds."""
    rng = np.random.default_rng(seeds)
    W, n = 40, 3000
    p = _rooted(W, n, lambda w, r: [(n - 1, range(1, n - 1, 29))], seeds)
    with nalar.Policy() as pol, nalar.Store(pol) as st:
        pol.set_timing(True)
        prev = feed(st, p, 0, None)
        store_pass(pol, st, p)
        for tick in range(3):
            for idle in range(2):
                g, inc = store_pass(pol, st, p)
                assert inc and st.last_fallback == 0
            assert "inc_close_r1" not in [k for k, _ in pol.timing()]
            open_ids = np.flatnonzero(p.done == 0)
            ids = rng.choice(open_ids, seeds // 4, replace=False)
            # children of children: the second half of the new futures hang on the first
            first = rng.integers(0, p.n_nodes, (seeds - seeds // 4) // 2)
            q = _extended(p, ids, first, tick)
            q = _extended(q, [], p.n_nodes + np.arange(first.size), tick + 10)
            prev = feed(st, q, *prev)
            g, inc = store_pass(pol, st, q)
            assert inc, st.last_fallback
            assert_parity(g, oracle.run(q), f"{seeds} seeds, tick {tick}")
            assert ("inc_close_r2" in [k for k, _ in pol.timing()]) == (seeds > 8192)
            p = q


def test_record_sweep_on_a_handle_with_bins():
    """A handle whose passes so far needed no grouping (nothing was looked at) takes
    the record sweep at its first snapshot with ids by creation."""
    p, grouped = _grown_workflows(np.full(150, 900), 4)
    with nalar.Policy() as pol:
        pol.set_timing(True)
        for rep in range(2):
            check(pol, grouped, f"grouped ids {rep}")
        for rep in range(2):
            check(pol, p, f"ids by creation {rep}")
            assert "records" in [k for k, _ in pol.timing()]
