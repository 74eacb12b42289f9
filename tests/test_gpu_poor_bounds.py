"""GPU: tables whose latencies depend on how many stages lie behind in ways that the band kernel's front costs do not see (stages
that do not fit with many behind them, stages of equal layers, latencies without any order): results against the oracle or the
general kernel on every solve of a table, as its bounds get better, and the work that the better bounds save.  Whole numbers: no
tolerance."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("T_star", "t_max", "num_stages", "n_evaluated", "first_layer", "shape_idx")


def _plan_is(plan, ref):
    assert {k: plan[k] for k in KEYS} == {k: ref[k] if isinstance(ref, dict) else getattr(ref, k) for k in KEYS}


def _short_of_memory(K, N, M, cap):
    """Stages with s - 1 behind need (2 + s) units of memory a layer, shared by the stage's devices."""
    w = W.many_stage_problem(K, K, N, M)
    s = np.arange(1, K + 1)[:, None, None, None]
    length = np.arange(K)[None, :] - np.arange(K)[:, None] + 1
    a = (w.shapes[:, 0] * w.shapes[:, 1])[None, None, None, :]
    table = np.where((2 + s) * length[None, :, :, None] > cap * a, oracle.INF32, w.table)
    return np.ascontiguousarray(table.astype(np.int32)), w.shapes


# layers, mesh, candidates (more than 512: two rounds; the size classes of the kernel)
SIZES = [(12, 2, 8, 0), (20, 3, 8, 700), (16, 9, 8, 40), (12, 17, 8, 40), (66, 1, 8, 40), (3, 1, 16, 0), (1, 1, 16, 0)]


@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}-n{s[3]}")
def test_every_solve_of_a_table(size):
    K, N, M, n = size
    rand = W.random_problem(K, K, N, M, inf_frac=0.3, value_hi=200_000)
    deep = W.deep_model_problem(K, K, N, M)
    tables = [(rand.table, rand.shapes, False), (deep.table, deep.shapes, True), (*_short_of_memory(K, N, M, 9), False),
              (*_short_of_memory(K, N, M, 4), False)]
    for table, shapes, equal in tables:
        ref_table = oracle.equal_layer_table(table) if equal else table
        every = oracle.all_candidates(ref_table, shapes)
        cand = oracle.quantiles(every, n) if n and len(every) > n else every
        n_solve = n if n and len(every) > n else 0
        refs = {(Bv, prune): oracle.solve_parallel(ref_table, N, M, Bv, shapes, cand, prune, 8)
                for Bv in (1, 30) for prune in (False, True)}
        for prune in (False, True):
            for plan_only in (False, True):
                h = B.alpa_dp_create(table, K, N, M, 1, shapes)
                try:
                    if equal:
                        B.alpa_dp_restrict_equal_layers(h)
                    for solve in range(4):
                        Bv = (1, 30)[solve & 1]
                        B.alpa_dp_set_B(h, Bv)
                        T, plan = B.alpa_dp_solve(h, None, n_solve, B.ALPA_DP_PRUNE if prune else 0, want_T=not plan_only)
                        T_ref, p_ref = refs[Bv, prune]
                        _plan_is(plan, p_ref)
                        assert plan_only or np.array_equal(T, T_ref)
                    for Bv, plan in zip((1, 30), B.alpa_dp_solve_sweep(h, None, [1, 30], n_tmax=n_solve)):
                        _plan_is(plan, refs[Bv, False][1])
                finally:
                    B.alpa_dp_destroy(h)


def _work(h, n, want_T):
    plan = B.alpa_dp_solve(h, None, n, B.ALPA_DP_COUNT_WORK, want_T=want_T)[1]
    return plan, B.alpa_dp_last_counters(h)["wave_relaxations"]


def test_work_of_a_table_without_any_order():
    """A later solve knows how little the layers behind the first few can give (without that every solve did the same work)."""
    w = W.random_problem(3, 48, 8, 8, inf_frac=0.2, value_hi=200_000)
    h = B.alpa_dp_create(w.table, 48, 8, 8, 8, w.shapes)
    try:
        ref = B.alpa_dp_solve(h, None, 2000, B.ALPA_DP_GENERIC)[1]
    finally:
        B.alpa_dp_destroy(h)
    h = B.alpa_dp_create(w.table, 48, 8, 8, 8, w.shapes)
    try:
        got = [_work(h, 2000, True) for _ in range(3)]
        for plan, _ in got:
            _plan_is(plan, ref)
        assert got[1][1] < got[0][1] / 3 and got[2][1] == got[1][1]
    finally:
        B.alpa_dp_destroy(h)


def test_work_for_a_plan_where_memory_is_short():
    """A plan that fits is found beforehand, so the plan alone needs few candidates on the first solve already (without one it
    needed all of them)."""
    w = W.deep_model_problem(5, 48, 32, 8)
    h = B.alpa_dp_create(w.table, 48, 32, 8, 8, w.shapes)
    try:
        plan, alone = _work(h, 300, False)
        plan_T, whole = _work(h, 300, True)
        _plan_is(plan, plan_T)
        assert alone < whole / 2
    finally:
        B.alpa_dp_destroy(h)
