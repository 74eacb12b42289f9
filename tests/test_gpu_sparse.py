"""GPU: candidates solved on the few stages that each interval of thresholds leaves (tables whose latencies do not fall with the
number of stages behind), against the CPU oracle or, where that takes too long, the general kernel: at the edges of eight layers and
of the devices' size classes, with stages that are least only at first, memory that ends early, many ties, more candidates than kept
plans, intervals whose stages are too many, and tables in which one entry falls.  Whole numbers: no tolerance."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("T_star", "t_max", "num_stages", "n_evaluated", "first_layer", "shape_idx")
# layers, mesh; whether the oracle is quick enough
SIZES = [(1, 2, 1, True), (8, 2, 8, True), (9, 9, 1, True), (17, 4, 8, True), (16, 1, 64, True), (24, 33, 1, True), (20, 17, 8, False),
         (33, 2, 64, False), (31, 2, 128, False), (48, 1, 128, False)]


BELOW, PASS, SECOND_PASS, LAYERS, LEFT = range(5)      # how a candidate was settled


def _routes(h):
    """The graphs of the intervals, (first, stages, cells, chunks, from, twice, ..) each, stages < 0: none; and how many candidates of the
    last solve with the counting flag were settled in each way."""
    heads, routes = np.zeros((120, 8), np.int32), np.zeros(5, np.int32)
    B._check(B.load().alpa_dp_routes_(h, ctypes.c_void_p(heads.ctypes.data), ctypes.c_void_p(routes.ctypes.data)))
    return heads, routes


def _plan_is(plan, ref):
    assert all(plan[k] == (getattr(ref, k) if not isinstance(ref, dict) else ref[k]) for k in KEYS)


def _tables(K, N, M):
    """Unstructured entries put in order of the number of stages: few values, many values with and without much that does not fit;
    latencies that do not depend on it and grow with the layers; the same layer everywhere; one entry that falls."""
    for x, (inf, hi) in enumerate(((0.05, 9), (0.3, 200_000), (0.9, 5000))):
        yield np.sort(W.random_problem(K + x, K, N, M, inf_frac=inf, value_hi=hi).table, axis=0)
    base = W.deep_model_problem(K, K, N, M, B=7).table
    yield base
    same = np.broadcast_to(base[:, :1, :, :], base.shape).copy()            # (a stage's latency by its length alone)
    for k in range(1, K):
        same[:, k, k:] = base[:, 0, :K - k]
        same[:, k, :k] = oracle.INF32
    yield same
    fell = base.copy()
    if K > 2 and fell[1, 0, 1, 0] != oracle.INF32:
        fell[1, 0, 1, 0] -= 1
    yield fell


@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_few_stages(size):
    K, N, M, small = size
    shapes = W.submesh_shapes(N, M)
    for table in _tables(K, N, M):
        h = B.alpa_dp_create(table, K, N, M, 1, shapes)
        try:
            for Bv in (1, 7, 3000):
                B.alpa_dp_set_B(h, Bv)
                for flags in (0, B.ALPA_DP_PRUNE):
                    T, plan = B.alpa_dp_solve(h, None, 300, flags)
                    T_ref, ref = B.alpa_dp_solve(h, None, 300, flags | B.ALPA_DP_GENERIC)
                    assert np.array_equal(T, T_ref)
                    _plan_is(plan, ref)
                    _plan_is(B.alpa_dp_solve(h, None, 300, flags, want_T=False)[1], ref)
            every = oracle.all_candidates(table, shapes) if small else []
            if len(every):
                cand = oracle.quantiles(every, 60) if len(every) > 60 else every
                T_ref, ref = oracle.solve_parallel(table, N, M, 3000, shapes, cand, False, 8)
                T, plan = B.alpa_dp_solve(h, cand, flags=0)
                assert np.array_equal(T, T_ref)
                _plan_is(plan, ref)
        finally:
            B.alpa_dp_destroy(h)


@pytest.mark.parametrize("n", [2047, 2049, 4096, 4097, 9000])
def test_more_candidates_than_kept_plans(n):
    K, N, M = 17, 4, 8
    shapes = W.submesh_shapes(N, M)
    table = np.sort(W.random_problem(3, K, N, M, inf_frac=0.2, value_hi=1_000_000).table, axis=0)
    h = B.alpa_dp_create(table, K, N, M, 40, shapes)
    try:
        Bs = [1, 2, 5, 40, 3000]
        plans = B.alpa_dp_solve_sweep(h, None, Bs, n)
        for b, Bv in enumerate(Bs):
            B.alpa_dp_set_B(h, Bv)
            T_ref, ref = B.alpa_dp_solve(h, None, n, B.ALPA_DP_GENERIC)
            T, plan = B.alpa_dp_solve(h, None, n, 0)
            assert np.array_equal(T, T_ref)
            _plan_is(plan, ref)
            _plan_is(B.alpa_dp_solve(h, None, n, B.ALPA_DP_PRUNE, want_T=False)[1], B.alpa_dp_solve(h, None, n, B.ALPA_DP_PRUNE | B.ALPA_DP_GENERIC)[1])
            _plan_is(plans[b], ref)
    finally:
        B.alpa_dp_destroy(h)


# ordered tables on which hardly an interval has a graph: the recurrence does not run for more of their candidates than it does for
# the same table with one entry that falls, which no graphs are made for
@pytest.mark.parametrize("size", [(24, 2, 8), (40, 16, 8), (30, 32, 8)], ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
@pytest.mark.parametrize("n", [513, 4096, 9000])
def test_candidates_without_graphs(size, n):
    K, N, M = size
    shapes = W.submesh_shapes(N, M)
    table = np.sort(W.random_problem(1, K, N, M, inf_frac=0.2, value_hi=100_000).table, axis=0)
    fell = table.copy()
    at = np.argwhere(fell[1] != oracle.INF32)[-1]                            # (a long stage with one behind it)
    fell[(1, *at)] = fell[(0, *at)] - 1
    work = []
    for t in (table, fell):
        h = B.alpa_dp_create(t, K, N, M, 7, shapes)
        try:
            B.alpa_dp_solve(h, None, n)                                      # (the table's bounds, and better ones with the second)
            B.alpa_dp_solve(h, None, n)
            T, plan = B.alpa_dp_solve(h, None, n, B.ALPA_DP_COUNT_WORK)
            work.append(B.alpa_dp_last_counters(h)["wave_relaxations"])
            T_ref, ref = B.alpa_dp_solve(h, None, n, B.ALPA_DP_GENERIC)
            assert np.array_equal(T, T_ref)
            _plan_is(plan, ref)
            _plan_is(B.alpa_dp_solve(h, None, n, want_T=False)[1], ref)
            T_ref, ref = B.alpa_dp_solve(h, None, n, B.ALPA_DP_GENERIC | B.ALPA_DP_PRUNE)
            T, plan = B.alpa_dp_solve(h, None, n, B.ALPA_DP_PRUNE)
            assert np.array_equal(T, T_ref)
            _plan_is(plan, ref)
            _plan_is(B.alpa_dp_solve(h, None, n, B.ALPA_DP_PRUNE, want_T=False)[1], ref)
            for flags in (0, B.ALPA_DP_PRUNE):
                for plan, Bv in zip(B.alpa_dp_solve_sweep(h, None, [1, 7, 300], n, flags), (1, 7, 300)):
                    B.alpa_dp_set_B(h, Bv)
                    _plan_is(plan, B.alpa_dp_solve(h, None, n, flags | B.ALPA_DP_GENERIC)[1])
            B.alpa_dp_set_B(h, 7)
        finally:
            B.alpa_dp_destroy(h)
    # (knots lie evenly over all candidates, settled or not)
    print(size, n, work)
    assert work[0] <= 1.5 * work[1] + 100, work


# graphs of 12 900 stages in all, few layers on many devices: they find room, and the same ones each time
def test_graphs_find_room():
    K, N, M = 20, 24, 8
    w = W.many_stage_problem(3, K, N, M)
    sizes = []
    for _ in range(3):
        h = B.alpa_dp_create(w.table, K, N, M, 64, w.shapes)
        try:
            B.alpa_dp_solve(h, None, 1000, B.ALPA_DP_COUNT_WORK)
            heads, routes = _routes(h)
        finally:
            B.alpa_dp_destroy(h)
        assert routes[LEFT] == 0
        sizes.append(heads[:, 1])
    assert sizes[0][sizes[0] > 0].sum() > max(12 * K * K, 8192)
    assert np.array_equal(sizes[0], sizes[1]) and np.array_equal(sizes[0], sizes[2])


# each way of settling candidates is taken by tables made for it, with the general kernel's results
WAYS = {BELOW: "deep", PASS: "deep", SECOND_PASS: "deep", LAYERS: "ordered", LEFT: "deep"}


@pytest.mark.parametrize("way", WAYS, ids=["below", "pass", "second-pass", "layers", "left"])
def test_ways_of_settling(way):
    if WAYS[way] == "deep":
        K, N, M = (32, 16, 8)
        table = W.deep_model_problem(7, K, N, M).table
    else:
        K, N, M = (20, 8, 8)
        table = np.sort(W.random_problem(1, K, N, M, inf_frac=0.2, value_hi=100_000).table, axis=0)
    h = B.alpa_dp_create(table, K, N, M, 40, W.submesh_shapes(N, M))
    try:
        T, plan = B.alpa_dp_solve(h, None, 2000, B.ALPA_DP_COUNT_WORK)
        heads, routes = _routes(h)
        assert routes[way] > 0 and routes.sum() <= 2000
        assert way != BELOW or (heads[:, 4] > 0).any()
        T_ref, ref = B.alpa_dp_solve(h, None, 2000, B.ALPA_DP_GENERIC)
        assert np.array_equal(T, T_ref)
        _plan_is(plan, ref)
    finally:
        B.alpa_dp_destroy(h)


# graphs of more stages than the list in LDS holds: the cells are looked at again to write them
def test_graph_larger_than_the_list():
    K, N, M = 100, 16, 8
    w = W.deep_model_problem(3, K, N, M)
    h = B.alpa_dp_create(w.table, K, N, M, 40, w.shapes)
    try:
        T, plan = B.alpa_dp_solve(h, None, 300)
        heads, _ = _routes(h)
        assert heads[:, 5].any()
        T_ref, ref = B.alpa_dp_solve(h, None, 300, B.ALPA_DP_GENERIC)
        assert np.array_equal(T, T_ref)
        _plan_is(plan, ref)
    finally:
        B.alpa_dp_destroy(h)
