"""GPU: the band kernel and what it takes from a table beforehand (windows, front costs, plans) against the CPU
oracle, or against the general kernel where that takes too long, at the sizes where they change form: the size classes of
devices (16 | 17, 32 | 33, 64 | 65, 128 | 129, 256), blocks of eight layers, front costs in registers (64 | 65,
128 | 129 layers), two and three layers in LDS, the most layers that fit, shapes beyond sixteen.  Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("T_star", "t_max", "num_stages", "n_evaluated", "first_layer", "shape_idx")
# layers, mesh
SIZES = [(1, 9, 1), (7, 2, 8), (8, 17, 1), (9, 1, 16), (16, 3, 8), (17, 4, 8), (24, 33, 1), (33, 8, 8), (8, 33, 2),
         (40, 16, 8), (12, 1, 128), (20, 17, 8), (31, 2, 128), (24, 32, 8), (59, 1, 256)]
DEEP = [(64, 3, 8), (65, 5, 1), (96, 2, 4), (128, 8, 8), (129, 1, 2), (123, 16, 8), (140, 1, 16)]


def _tables(K, N, M):
    """Unstructured entries of a few values (many ties), of many, hardly any plan; stages that grow with their length."""
    yield W.random_problem(K, K, N, M, inf_frac=0.1, value_hi=9)
    yield W.random_problem(K + 1, K, N, M, inf_frac=0.6, value_hi=200_000)
    yield W.random_problem(K + 2, K, N, M, inf_frac=0.97, value_hi=5000)
    yield W.deep_model_problem(K, K, N, M, B=7)


def _plan_is(plan, ref):
    assert all(plan[k] == (getattr(ref, k) if not isinstance(ref, dict) else ref[k]) for k in KEYS)


@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_band_kernel_against_the_oracle(size):
    K, N, M = size
    for w in _tables(K, N, M):
        h = B.alpa_dp_create(w.table, K, N, M, 1, w.shapes)
        try:
            every = oracle.all_candidates(w.table, w.shapes)
            n = 600 if K * N * M < 2000 else 40        # (the oracle's time; 600: two rounds)
            cand = oracle.quantiles(every, n) if len(every) > n else every
            n = n if len(every) > n else 0
            for Bv, prune in ((3000, False), (6, True), (3000, True)):
                B.alpa_dp_set_B(h, Bv)
                T_ref, p_ref = oracle.solve_parallel(w.table, N, M, Bv, w.shapes, cand, prune, 8)
                flags = B.ALPA_DP_PRUNE if prune else 0
                T, plan = B.alpa_dp_solve(h, None, n, flags)
                assert np.array_equal(T, T_ref)
                _plan_is(plan, p_ref)
                _plan_is(B.alpa_dp_solve(h, None, n, flags, want_T=False)[1], p_ref)
            # values between and beyond those of the table, alone and together (the kernel's filter and the thresholds)
            hi = int(cand[-1]) if len(cand) else 5
            odd = np.array([0, 1, max(hi - 1, 0), hi, hi + 1, 2 * hi + 3, 2**30 - 1, 2**30, 2**31 - 2, hi // 2 + 1, hi // 2 + 1], np.int32)
            T_ref, p_ref = oracle.solve_parallel(w.table, N, M, 3000, w.shapes, np.unique(odd), False, 8)
            T, plan = B.alpa_dp_solve(h, odd, flags=0)
            assert np.array_equal(T, T_ref[np.searchsorted(np.unique(odd), odd)])
            assert plan["T_star"] == p_ref.T_star
        finally:
            B.alpa_dp_destroy(h)


@pytest.mark.parametrize("size", DEEP, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_band_kernel_against_the_general_kernel(size):
    K, N, M = size
    for w in (W.random_problem(K, K, N, M, inf_frac=0.3, value_hi=100_000), W.deep_model_problem(K, K, N, M, B=7)):
        h = B.alpa_dp_create(w.table, K, N, M, 7, w.shapes)
        try:
            for flags in (0, B.ALPA_DP_PRUNE):
                T, plan = B.alpa_dp_solve(h, None, 40, flags)
                T_ref, ref = B.alpa_dp_solve(h, None, 40, flags | B.ALPA_DP_GENERIC)
                assert np.array_equal(T, T_ref)
                _plan_is(plan, ref)
                _plan_is(B.alpa_dp_solve(h, None, 40, flags, want_T=False)[1], ref)
            # a sweep's plans, recovered in one launch, and in several where their layers take more than 1 GiB
            Bs = [1 + 3 * b for b in range(256 if K > 120 else 5)]
            plans = B.alpa_dp_solve_sweep(h, None, Bs, 12)
            for b in (0, 4, len(Bs) - 1):
                B.alpa_dp_set_B(h, Bs[b])
                _plan_is(plans[b], B.alpa_dp_solve(h, None, 12, B.ALPA_DP_GENERIC)[1])
        finally:
            B.alpa_dp_destroy(h)


@pytest.mark.parametrize("size", [(9, 2, 8), (24, 1, 16), (20, 17, 8), (66, 2, 4)], ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_repeated_shapes(size):
    """Shapes listed up to four times, each with latencies of its own: the kernel takes the smallest of them, the plan names the one
    that has it."""
    K, N, M = size
    rng = np.random.default_rng(K)
    for x, w in enumerate((W.random_problem(K, K, N, M, inf_frac=0.5, value_hi=60), W.deep_model_problem(K, K, N, M, B=7))):
        which = rng.permutation(np.repeat(np.arange(len(w.shapes)), rng.integers(1, 5, len(w.shapes))))
        table = w.table[..., which].copy()
        table[(table != oracle.INF32) & (rng.random(table.shape) < 0.3)] += 3
        table[rng.random(table.shape) < 0.2] = oracle.INF32
        shapes = np.ascontiguousarray(w.shapes[which])
        cand = oracle.quantiles(oracle.all_candidates(table, shapes), 30)
        h = B.alpa_dp_create(table, K, N, M, 5, shapes)
        try:
            for prune in (False, True):
                T_ref, p_ref = oracle.solve_parallel(table, N, M, 5, shapes, cand, prune, 8)
                flags = B.ALPA_DP_PRUNE if prune else 0
                T, plan = B.alpa_dp_solve(h, cand, flags=flags)
                assert np.array_equal(T, T_ref)
                _plan_is(plan, p_ref)
                _plan_is(B.alpa_dp_solve(h, cand, flags=flags, want_T=False)[1], p_ref)
            _plan_is(B.alpa_dp_solve_sweep(h, cand, [5, 9])[0], oracle.solve_parallel(table, N, M, 5, shapes, cand, False, 8)[1])
        finally:
            B.alpa_dp_destroy(h)
