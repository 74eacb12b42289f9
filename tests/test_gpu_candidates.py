"""GPU: the candidates of a solve against the oracle where finding them changes form: bitmaps in LDS, in memory and the sort
(largest value 2**19, a word per table entry), numbers of stages that are not a multiple of eight; callers' lists around
the sizes of the one-block sort.  Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

# layers, mesh, largest value (17 layers on 8 x 8: 17 * 153 * 11 = 28611 entries, 28611 words hold values below 915552)
TABLES = [(17, 8, 8, 2**19 - 1), (17, 8, 8, 2**19), (17, 8, 8, 28611 * 32 - 1), (17, 8, 8, 28611 * 32),
          (33, 4, 8, 2**20), (9, 1, 4, 70_000), (8, 2, 8, 32), (1, 1, 1, 31), (40, 8, 8, 2**24)]


@pytest.mark.parametrize("case", TABLES, ids=lambda c: f"K{c[0]}-{c[1]}x{c[2]}-{c[3]}")
def test_distinct_values_of_a_table(case):
    K, N, M, hi = case
    for repeat in (False, True):                   # entries that differ by the number of stages behind, or hardly
        tab = W.random_problem(K, K, N, M, inf_frac=0.3, value_hi=hi).table.copy()
        if repeat:
            tab[1:] = np.where(np.arange(1, K).reshape(-1, 1, 1, 1) % 5 == 3, tab[1:], tab[:1])
        used = np.argwhere(tab[0, 0] != oracle.INF32)
        if len(used):
            tab[0, 0, used[0][0], used[0][1]] = hi
            tab[0, 0, used[-1][0], used[-1][1]] = 0 if len(used) > 1 else hi
        shapes = W.random_problem(K, K, N, M).shapes
        ref = oracle.all_candidates(tab, shapes)
        h = B.alpa_dp_create(tab, K, N, M, 4, shapes)
        try:
            assert B.alpa_dp_count_candidates(h) == len(ref)
            for n in (0, 40):
                B.alpa_dp_solve(h, None, n, B.ALPA_DP_PRUNE)
                want = oracle.quantiles(ref, n) if 0 < n < len(ref) else ref
                assert np.array_equal(B.alpa_dp_candidates(h), want)
        finally:
            B.alpa_dp_destroy(h)


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 128, 129, 1023, 1025, 1500, 4097, 8191, 8192, 8193])
def test_callers_lists(n):
    w = W.random_problem(5, 6, 1, 4, inf_frac=0.2, value_hi=3000, B=9)
    rng = np.random.default_rng(n)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        for hi in (4, 3100, 2**31 - 1):            # long runs of one value, few, none
            t = rng.integers(0, hi, size=n).astype(np.int32)
            u, place = np.unique(t, return_inverse=True)
            T_ref, p_ref = oracle.solve(w.table, w.N, w.M, w.B, w.shapes, u, False)
            T, plan = B.alpa_dp_solve(h, t)
            assert np.array_equal(B.alpa_dp_candidates(h), u)
            assert np.array_equal(T, T_ref[place])
            assert (plan["T_star"], plan["t_max"], plan["n_evaluated"]) == (p_ref.T_star, p_ref.t_max, p_ref.n_evaluated)
            _, again = B.alpa_dp_solve(h, t[::-1].copy(), want_T=False)
            assert again["T_star"] == p_ref.T_star and again["first_layer"] == p_ref.first_layer
    finally:
        B.alpa_dp_destroy(h)
