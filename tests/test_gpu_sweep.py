"""GPU parity of the sweep over the number of microbatches B (Sec. 5.2: B is found by
enumeration): one call for a vector of B values against one oracle run per value."""
import hashlib
import json
import os

import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

INF64 = oracle.INF64
GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
KERNELS = {"fast": 0, "generic": B.ALPA_DP_GENERIC}
B_VALUES = [1, 2, 3, 8, 32, 1000, 3, 100000]        # unordered, one repeated


def _same_plan(gpu: dict, ref: oracle.Plan):
    assert gpu["T_star"] == ref.T_star
    assert gpu["t_max"] == ref.t_max
    assert gpu["num_stages"] == ref.num_stages
    assert gpu["n_evaluated"] == ref.n_evaluated
    assert gpu["first_layer"] == ref.first_layer
    assert gpu["shape_idx"] == ref.shape_idx


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("prune", [False, True])
@pytest.mark.parametrize("idx", [1, 2])
def test_sweep_small_workloads(idx, prune, kernel):
    w = W.make_workload(idx)
    cand = oracle.all_candidates(w.table, w.shapes)
    flags = KERNELS[kernel] | (B.ALPA_DP_PRUNE if prune else 0)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        plans = B.alpa_dp_solve_sweep(h, None, B_VALUES, flags=flags)
        assert len(plans) == len(B_VALUES)
        for Bv, plan in zip(B_VALUES, plans):
            _, p_ref = oracle.solve(w.table, w.N, w.M, Bv, w.shapes, cand, prune)
            _same_plan(plan, p_ref)
        # the handle's own B and its running best are as before the sweep
        _, p_own = oracle.solve(w.table, w.N, w.M, w.B, w.shapes, cand, prune)
        _, plan = B.alpa_dp_solve(h, None, 0, flags)
        _same_plan(plan, p_own)
        _same_plan(B.alpa_dp_best(h), p_own)
    finally:
        B.alpa_dp_destroy(h)


SWEEP_RANDOM = [(2, 3, 2, 2), (6, 9, 3, 4), (7, 12, 2, 8), (11, 20, 5, 4), (12, 10, 8, 8),
                (13, 40, 3, 8), (14, 64, 1, 2), (21, 64, 8, 8), (22, 37, 6, 8)]


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("case", SWEEP_RANDOM, ids=lambda c: f"s{c[0]}-K{c[1]}-{c[2]}x{c[3]}")
def test_sweep_random_tables_with_a_caller_list(case, kernel):
    seed, K, N, M = case
    rng = np.random.default_rng(1000 + seed)
    w = W.random_problem(seed, K, N, M, inf_frac=float(rng.choice([0.0, 0.2, 0.6])),
                         value_hi=int(rng.choice([4, 50, 5000])))
    cand = oracle.all_candidates(w.table, w.shapes)
    if len(cand) > 120:
        cand = oracle.quantiles(cand, 120)
    if len(cand) == 0:
        pytest.skip("no finite entry")
    mine = np.concatenate([cand, cand[:5]]).astype(np.int32)     # caller order, duplicates
    rng.shuffle(mine)
    Bs = [int(x) for x in rng.choice([1, 2, 4, 7, 16, 64, 300, 5000], 5, replace=False)]
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        for prune in (False, True):
            flags = KERNELS[kernel] | (B.ALPA_DP_PRUNE if prune else 0)
            plans = B.alpa_dp_solve_sweep(h, mine, Bs, flags=flags)
            for Bv, plan in zip(Bs, plans):
                _, p_ref = oracle.solve_parallel(w.table, w.N, w.M, Bv, w.shapes, cand, prune, 8)
                _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


def test_sweep_sizes_one_and_maximum_and_growth():
    """n_B = 1, then the maximum, then a smaller one again on the same handle."""
    w = W.make_workload(1)
    cand = oracle.all_candidates(w.table, w.shapes)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        for Bs in ([5], list(range(1, B.MAX_SWEEP + 1)), [9, 2]):
            plans = B.alpa_dp_solve_sweep(h, None, Bs, flags=B.ALPA_DP_PRUNE)
            for Bv, plan in zip(Bs, plans):
                _, p_ref = oracle.solve(w.table, w.N, w.M, Bv, w.shapes, cand, True)
                _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


def test_sweep_infeasible_and_argument_errors():
    w = W.random_problem(1, 4, 2, 2, inf_frac=1.0)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        for plan in B.alpa_dp_solve_sweep(h, None, [1, 4]):
            assert plan["T_star"] == INF64 and plan["num_stages"] == 0
        for plan in B.alpa_dp_solve_sweep(h, [3, 9], [1, 4], flags=B.ALPA_DP_PRUNE):
            assert plan["T_star"] == INF64 and plan["num_stages"] == 0 and plan["n_evaluated"] == 2
        L = B.load()
        Bs = np.asarray([1, 2], np.int32)
        out = (B.alpa_plan_t * 2)()
        import ctypes
        po = ctypes.addressof(out)
        assert L.alpa_dp_solve_sweep(h, None, 0, 0, Bs.ctypes.data, 0, po) == -1
        assert L.alpa_dp_solve_sweep(h, None, 0, 0, Bs.ctypes.data, B.MAX_SWEEP + 1, po) == -1
        assert L.alpa_dp_solve_sweep(h, None, 0, 0, None, 2, po) == -1
        assert L.alpa_dp_solve_sweep(h, None, 0, 0, Bs.ctypes.data, 2, None) == -1
        assert L.alpa_dp_solve_sweep(None, None, 0, 0, Bs.ctypes.data, 2, po) == -1
        bad = np.asarray([1, 0], np.int32)
        assert L.alpa_dp_solve_sweep(h, None, 0, 0, bad.ctypes.data, 2, po) == -1
        assert L.alpa_dp_solve_sweep(h, None, 1, 0, Bs.ctypes.data, 2, po) == -1
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("idx", [3, 4, 5])
def test_sweep_full_size_workloads_against_stored_oracle_results(idx):
    """Expected plans were written by tests/golden/make_golden.py --sweep, one oracle run per B."""
    g = json.load(open(os.path.join(GOLD, f"sweep_{idx}.json")))
    w = W.make_workload(idx)
    assert hashlib.sha256(w.table.tobytes()).hexdigest() == g["table_sha256"]
    assert bool(w.prune) == g["prune"]
    Bs = [p["B"] for p in g["plans"]]
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        nq = w.n_quantiles if w.candidates == "quantiles" else 0
        plans = B.alpa_dp_solve_sweep(h, None, Bs, n_tmax=nq,
                                      flags=B.ALPA_DP_PRUNE if w.prune else 0)
        for plan, ref in zip(plans, g["plans"]):
            for key in ("T_star", "t_max", "num_stages", "n_evaluated", "first_layer", "shape_idx"):
                assert plan[key] == ref[key], (ref["B"], key)
    finally:
        B.alpa_dp_destroy(h)


def test_sweep_general_kernel_on_a_mesh_larger_than_64_devices():
    w = W.random_problem(78, 66, 10, 8, inf_frac=0.3, value_hi=900)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 6)
    Bs = [2, 64]
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        plans = B.alpa_dp_solve_sweep(h, cand, Bs)
        for Bv, plan in zip(Bs, plans):
            _, p_ref = oracle.solve_parallel(w.table, w.N, w.M, Bv, w.shapes, cand, False, 8)
            _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


def test_times_of_a_sweep_end_with_its_last_plan():
    """A sweep whose first plan has one stage and the second one 32, and the other way round: the longer walk, a quarter of the last
    phase, is in its time both ways.  (The least of 20 repetitions; within 15 %.)"""
    K, N, M = 32, 8, 8
    shapes = W.submesh_shapes(N, M)
    k, i = np.arange(K)[:, None, None], np.arange(K)[None, :, None]
    a = (shapes[:, 0] * shapes[:, 1])[None, None, :]
    once = np.where(i >= k, (i - k + 1) * 1000 / np.sqrt(a), B.INF_I32).astype(np.int32)
    table = np.repeat(once[None], K, axis=0)
    table[1, 0, K - 2] -= 1                                  # (no plan is kept where a latency falls with the stages behind)
    h = B.alpa_dp_create(table, K, N, M, 1, shapes)
    try:
        ms = []
        for order in ((1, 100_000), (100_000, 1)):
            plans = B.alpa_dp_solve_sweep(h, None, order, 200)
            assert [p["num_stages"] for p in plans] == ([1, K] if order[0] == 1 else [K, 1])
            least = 1e9
            for _ in range(20):
                B.alpa_dp_solve_sweep(h, None, order, 200)
                least = min(least, B.alpa_dp_last_timing(h)["ms_epilogue"])
            ms.append(least)
        print(ms)
        assert abs(ms[0] - ms[1]) < 0.15 * max(ms)
    finally:
        B.alpa_dp_destroy(h)
