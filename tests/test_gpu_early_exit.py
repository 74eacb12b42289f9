"""GPU: where the early exit of Alg. 1 ends the loop, against the sequential oracle: candidates that are not values of the table,
device lists with values that no candidate should have, on both sides of the one-block sort's longest list.
Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("T_star", "t_max", "num_stages", "n_evaluated", "first_layer", "shape_idx")
FORMS = {"own": 0, "generic": B.ALPA_DP_GENERIC}


def _plan_is(plan, ref):
    assert {k: plan[k] for k in KEYS} == {k: getattr(ref, k) for k in KEYS}


def _solve_dev(h, t, flags, want_T=True):
    import torch
    d = torch.from_numpy(t).cuda()
    T = torch.full((len(t),), -7, dtype=torch.int64, device="cuda")
    plan = torch.zeros(B.PLAN_BYTES, dtype=torch.uint8, device="cuda")
    B.alpa_dp_solve_dev(h, d, len(t), flags, T if want_T else None, plan)
    torch.cuda.synchronize()
    return T.cpu().numpy(), B.plan_from_bytes(plan.cpu().numpy().tobytes())


def _sorted_as_the_library(t):
    """Ascending distinct candidates, negative ones (sorted as unsigned) behind the others."""
    return np.unique(t.view(np.uint32)).view(np.int32)


# (13 layers on 2 x 4: the register/LDS kernel; on 2 x 8: the band kernel)
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("mesh", [(2, 4), (2, 8)], ids=lambda m: f"{m[0]}x{m[1]}")
@pytest.mark.parametrize("negative", [1, 7, 300, 900])
def test_early_exit_in_front_of_negative_values(negative, mesh, form):
    """The loop ends among the values that are not negative, however many of the others lie behind them."""
    w = W.random_problem(21, 13, *mesh, inf_frac=0.2, value_hi=250_000)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 300)
    t = np.concatenate([cand, -2 - 3 * np.arange(negative)]).astype(np.int32)
    np.random.default_rng(negative).shuffle(t)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, 1, w.shapes)
    try:
        for Bv in (1, 3, 40, 100_000):
            B.alpa_dp_set_B(h, Bv)
            u = _sorted_as_the_library(t)
            for prune in (True, False):
                T_ref, p_ref = oracle.solve_parallel(w.table, w.N, w.M, Bv, w.shapes, u, prune, 8)
                flags = FORMS[form] | (B.ALPA_DP_PRUNE if prune else 0)
                T, plan = _solve_dev(h, t, flags)
                assert np.array_equal(T, T_ref[np.searchsorted(u.view(np.uint32), t.view(np.uint32))])
                _plan_is(plan, p_ref)
                _plan_is(_solve_dev(h, t, flags, want_T=False)[1], p_ref)
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("n", [9, 8192, 8193])
def test_minus_one_is_no_candidate(n):
    """The value -1 marks an entry without a candidate, in lists of every length."""
    w = W.random_problem(22, 9, 2, 8, inf_frac=0.2, value_hi=50_000)
    rng = np.random.default_rng(n)
    t = rng.choice(oracle.all_candidates(w.table, w.shapes), n).astype(np.int32)
    t[rng.permutation(n)[: n // 3]] = -1
    u = np.unique(t[t >= 0])
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, 5, w.shapes)
    try:
        for prune in (False, True):
            T_ref, p_ref = oracle.solve_parallel(w.table, w.N, w.M, 5, w.shapes, u, prune, 8)
            T, plan = _solve_dev(h, t, B.ALPA_DP_PRUNE if prune else 0)
            assert np.array_equal(B.alpa_dp_candidates(h), u)
            assert (T[t < 0] == oracle.INF64).all()
            assert np.array_equal(T[t >= 0], T_ref[np.searchsorted(u, t[t >= 0])])
            _plan_is(plan, p_ref)
        T, plan = _solve_dev(h, np.full(n, -1, np.int32), 0)
        assert (T == oracle.INF64).all() and plan["num_stages"] == 0 and plan["n_evaluated"] == 0
        assert len(B.alpa_dp_candidates(h)) == 0
    finally:
        B.alpa_dp_destroy(h)


def _one_stage_or_eight(one, each):
    """8 layers on 1 x 16: one stage on all devices, or eight of two devices each."""
    shapes = W.submesh_shapes(1, 16)
    table = np.full((8, 8, 8, len(shapes)), oracle.INF32, np.int32)
    q = [int(a * b) for a, b in shapes]
    table[0, 0, 7, q.index(16)] = one
    for s in range(8):
        table[s, 7 - s, 7 - s, q.index(2)] = each
    return table, shapes


@pytest.mark.parametrize("form", list(FORMS))
def test_early_exit_at_a_value_far_above_the_plan(form):
    """t_max = 9000 admits a plan of 5000, T* 14000 with B = 2, but B t_max = 18000: the loop ends at it if a lower candidate
    has reached that, though the lower one's T* of 17920 is above 14000."""
    table, shapes = _one_stage_or_eight(5000, 1990)
    h = B.alpa_dp_create(table, 8, 1, 16, 2, shapes)
    try:
        for t in ([2000, 9000], [2000, 8000], [2000, 8961], [2000, 8960], [1, 2000, 2100, 9000, 9500], [9000]):
            t = np.array(t, np.int32)
            for prune in (True, False):
                flags = FORMS[form] | (B.ALPA_DP_PRUNE if prune else 0)
                _, ref = oracle.solve(table, 1, 16, 2, shapes, t, prune)
                _plan_is(B.alpa_dp_solve(h, t, flags=flags)[1], ref)
                _plan_is(B.alpa_dp_solve(h, t, flags=flags, want_T=False)[1], ref)
                Bs = [1, 2, 3, 50]
                for Bv, plan in zip(Bs, B.alpa_dp_solve_sweep(h, t, Bs, flags=flags)):
                    _plan_is(plan, oracle.solve(table, 1, 16, Bv, shapes, t, prune)[1])
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("size", [(8, 1, 16), (12, 2, 8), (10, 3, 16)], ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_early_exit_of_sparse_lists(size):
    """Short lists whose values lie anywhere between and beyond the table's, and a few quantiles of it."""
    K, N, M = size
    tables = [W.deep_model_problem(K, K, N, M), W.many_stage_problem(K, K, N, M),
              W.random_problem(K, K, N, M, inf_frac=0.5, value_hi=30_000)]
    for x, w in enumerate(tables):
        rng = np.random.default_rng(100 * K + x)
        hi = int(oracle.all_candidates(w.table, w.shapes)[-1])
        h = B.alpa_dp_create(w.table, K, N, M, 1, w.shapes)
        try:
            for trial in range(25):
                n = int(rng.integers(2, 9))
                t = np.unique(np.exp(rng.uniform(np.log(hi / 300), np.log(3 * hi), n)).astype(np.int32))
                Bs = [int(v) for v in np.unique(rng.integers(1, 12, 4))]
                for prune in (True, False):
                    flags = B.ALPA_DP_PRUNE if prune else 0
                    refs = [oracle.solve(w.table, N, M, Bv, w.shapes, t, prune)[1] for Bv in Bs]
                    for Bv, ref, plan in zip(Bs, refs, B.alpa_dp_solve_sweep(h, t, Bs, flags=flags)):
                        _plan_is(plan, ref)
                        B.alpa_dp_set_B(h, Bv)
                        _plan_is(B.alpa_dp_solve(h, t, flags=flags, want_T=False)[1], ref)
                        if n > 2:
                            q = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), n)
                            ref = oracle.solve(w.table, N, M, Bv, w.shapes, q, prune)[1]
                            _plan_is(B.alpa_dp_solve(h, None, n, flags, want_T=False)[1], ref)
        finally:
            B.alpa_dp_destroy(h)


def test_long_list_with_negative_values():
    """Beyond the one-block sort a value's result is found by bisection, also with most of the list negative."""
    w = W.random_problem(23, 9, 2, 8, inf_frac=0.2, value_hi=50_000)
    cand = oracle.all_candidates(w.table, w.shapes)[::3]
    t = np.concatenate([cand, -2 - 2 * np.arange(9000)]).astype(np.int32)
    np.random.default_rng(4).shuffle(t)
    T_ref, _ = oracle.eval_candidates(w.table, w.N, w.M, 5, w.shapes, np.maximum(t, 0), threads=8)
    T_ref[t < 0] = oracle.INF64
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, 5, w.shapes)
    try:
        assert np.array_equal(_solve_dev(h, t, 0)[0], T_ref)
    finally:
        B.alpa_dp_destroy(h)
