"""GPU parity where a candidate list is evaluated in rounds (one, two and three of them, lists of
every form's length), where the range worth searching is cut down beforehand, and where layers are
left out on the table's bound: everything returned against the CPU oracle, bit for bit.  All
figures are whole numbers, so there is no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

FORMS = {"own": 0, "generic": B.ALPA_DP_GENERIC}


def _same_plan(gpu: dict, ref: oracle.Plan):
    assert (gpu["T_star"], gpu["t_max"], gpu["num_stages"], gpu["n_evaluated"], gpu["first_layer"],
            gpu["shape_idx"]) == (ref.T_star, ref.t_max, ref.num_stages, ref.n_evaluated,
                                  ref.first_layer, ref.shape_idx)


def _table(seed, K, N, M, value_hi, inf_frac):
    """Unstructured entries of a wide range: nearly as many candidates as entries, and a staircase of
    results with many steps."""
    return W.random_problem(seed, K, N, M, inf_frac=inf_frac, value_hi=value_hi)


# seed, K, N, M, share of infinite entries, candidates (0: every distinct value)
CASES = [(1, 9, 1, 8, 0.2, 0), (2, 14, 2, 8, 0.2, 0), (3, 20, 2, 8, 0.5, 0),
         (4, 20, 2, 8, 0.97, 0),                     # hardly any plan
         (5, 12, 8, 8, 0.1, 2048), (6, 12, 8, 8, 0.1, 2049), (7, 33, 2, 4, 0.3, 513), (8, 17, 3, 4, 0.0, 8193),
         (9, 10, 10, 8, 0.3, 2100), (10, 1, 1, 1, 0.0, 0), (11, 6, 2, 1, 1.0, 0)]


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"s{c[0]}-K{c[1]}-{c[2]}x{c[3]}-n{c[5]}")
def test_rounds_match_the_oracle(case, form):
    seed, K, N, M, inf_frac, n = case
    w = _table(seed, K, N, M, 250_000, inf_frac)
    cand = oracle.all_candidates(w.table, w.shapes)
    if n and len(cand) > n:
        cand = oracle.quantiles(cand, n)
    h = B.alpa_dp_create(w.table, K, N, M, 1, w.shapes)
    try:
        for Bv in (1, 7, 1000):
            B.alpa_dp_set_B(h, Bv)
            for prune in (False, True):
                T_ref, p_ref = oracle.solve_parallel(w.table, N, M, Bv, w.shapes, cand, prune, 8)
                flags = FORMS[form] | (B.ALPA_DP_PRUNE if prune else 0)
                T, plan = B.alpa_dp_solve(h, None, n, flags)
                assert np.array_equal(T, T_ref)
                _same_plan(plan, p_ref)
                if len(cand):
                    _, plan = B.alpa_dp_solve(h, cand[::-1].copy(), flags=flags, want_T=False)
                    _same_plan(plan, p_ref)
                _, plan = B.alpa_dp_solve(h, None, n, flags, want_T=False)
                _same_plan(plan, p_ref)
        Bs = [1, 2, 30, 5000]
        for prune in (False, True):
            flags = FORMS[form] | (B.ALPA_DP_PRUNE if prune else 0)
            for Bv, plan in zip(Bs, B.alpa_dp_solve_sweep(h, None, Bs, n_tmax=n, flags=flags)):
                _, p_ref = oracle.solve_parallel(w.table, N, M, Bv, w.shapes, cand, prune, 8)
                _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("form", list(FORMS))
def test_device_list_with_values_out_of_range(form):
    """solve_dev does not check its candidates: negative values and INT32_MAX must not disturb the others."""
    import torch
    w = _table(21, 13, 2, 8, 250_000, 0.2)
    cand = oracle.all_candidates(w.table, w.shapes)
    mine = np.concatenate([cand[::2], [-5, -2, -2**31, 2**31 - 1, 0]]).astype(np.int32)
    np.random.default_rng(3).shuffle(mine)
    ref, _ = oracle.eval_candidates(w.table, w.N, w.M, w.B, w.shapes, np.maximum(mine, 0), threads=8)
    good = (mine >= 0) & (mine < 2**31 - 1)
    h = B.alpa_dp_create(w.table, w.K, w.N, w.M, w.B, w.shapes)
    try:
        d = torch.from_numpy(mine).cuda()
        T = torch.zeros(len(mine), dtype=torch.int64, device="cuda")
        B.alpa_dp_solve_dev(h, d, len(mine), FORMS[form], T, None)
        torch.cuda.synchronize()
        T = T.cpu().numpy()
        assert np.array_equal(T[good], ref[good])
        assert (T[mine < 0] == oracle.INF64).all()
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("size", [(23, 4, 8), (40, 1, 64), (40, 12, 8)], ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_bound_on_late_layers(size):
    """Tables on which the best plan has nearly as many stages as layers or devices allow, where the
    bound must not stop early, and the same after the restriction to equal stages (a new table)."""
    K, N, M = size
    w = W.many_stage_problem(5, K, N, M)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 300)
    for equal in (False, True):
        table = oracle.equal_layer_table(w.table) if equal else w.table
        T_ref, p_ref = oracle.solve_parallel(table, N, M, w.B, w.shapes, cand, False, 8)
        h = B.alpa_dp_create(w.table, K, N, M, w.B, w.shapes)
        try:
            if equal:
                B.alpa_dp_restrict_equal_layers(h)
            T, plan = B.alpa_dp_solve(h, cand)
            assert np.array_equal(T, T_ref)
            _same_plan(plan, p_ref)
        finally:
            B.alpa_dp_destroy(h)


# sizes of the kernel with a workgroup per candidate: 65 layers and more, 129-256 devices; one, odd and even numbers of blocks
# of 8 layers, device counts at the edges of 16, 32, 64 and their multiples, many shapes; deep models (97 layers
# on 1 x 4 are the register/LDS kernel's)
ROW_CASES = [(65, 3, 2), (72, 1, 16), (73, 3, 8), (96, 4, 8), (121, 5, 4), (128, 8, 8), (97, 1, 4), (88, 60, 1),
             (66, 10, 8), (86, 16, 8),
             (1, 17, 8), (8, 24, 8), (9, 32, 8), (17, 12, 16), (23, 60, 4), (40, 31, 8), (48, 16, 16), (54, 16, 16),
             (129, 1, 2), (244, 1, 1), (191, 1, 4), (240, 2, 8), (195, 4, 8), (130, 8, 8), (138, 8, 8), (99, 64, 1), (120, 32, 2)]


@pytest.mark.parametrize("size", ROW_CASES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
@pytest.mark.parametrize("inf_frac", [0.0, 0.6])
def test_workgroup_per_candidate_sizes(size, inf_frac):
    K, N, M = size
    if inf_frac and (K > 128 and N * M > 16 or K * N * M > 6300 and M <= 2):
        pytest.skip("one share of infinite entries for the sizes that take the oracle longest")
    w = W.random_problem(K + 7 * N, K, N, M, inf_frac=inf_frac, value_hi=9000)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 12)
    cand = np.unique(np.concatenate([cand, cand[:3] // 2, [2**31 - 2]])).astype(np.int32)
    h = B.alpa_dp_create(w.table, K, N, M, w.B, w.shapes)
    try:
        for prune in (False, True):
            T_ref, p_ref = oracle.solve_parallel(w.table, N, M, w.B, w.shapes, cand, prune, 8)
            flags = B.ALPA_DP_PRUNE if prune else 0
            for extra in (0, B.ALPA_DP_COUNT_WORK):
                T, plan = B.alpa_dp_solve(h, cand, flags=flags | extra)
                assert np.array_equal(T, T_ref)
                _same_plan(plan, p_ref)
        Bs = [1, 40]
        for Bv, plan in zip(Bs, B.alpa_dp_solve_sweep(h, cand, Bs)):
            _, p_ref = oracle.solve_parallel(w.table, N, M, Bv, w.shapes, cand, False, 8)
            _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


# sizes of 65-128 layers that stay with the register/LDS kernel: the smallest meshes; lists in the share of each of its forms
# (sixteen and eight waves per candidate, four; lane groups)
DEEP_CASES = [(65, 1, 1), (65, 1, 2), (128, 1, 1), (72, 1, 2), (81, 3, 1), (96, 1, 4), (112, 2, 1), (128, 1, 2), (97, 4, 1), (128, 2, 2)]


@pytest.mark.parametrize("size", DEEP_CASES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_deep_models_in_the_register_kernel(size):
    K, N, M = size
    w = W.random_problem(K + N, K, N, M, inf_frac=0.3, value_hi=9000)
    few = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 5)
    h = B.alpa_dp_create(w.table, K, N, M, w.B, w.shapes)
    try:
        for prune in (0, B.ALPA_DP_PRUNE):
            T_ref, p_ref = oracle.solve_parallel(w.table, N, M, w.B, w.shapes, few, bool(prune), 8)
            for n in (5, 300, 700, 2500):
                T_gen, p_gen = B.alpa_dp_solve(h, None, n, prune | B.ALPA_DP_GENERIC)
                for key, value in ((B.ALPA_DP_TUNE_CANDIDATES_PER_WG, 0), (B.ALPA_DP_TUNE_CANDIDATES_PER_WG, 1),
                                   (B.ALPA_DP_TUNE_CANDIDATES_PER_WG, 2), (B.ALPA_DP_TUNE_LANE_GROUPS, 1)):
                    B.alpa_dp_set_tuning(h, key, value)
                    for extra in (0, B.ALPA_DP_COUNT_WORK):
                        T, plan = B.alpa_dp_solve(h, None, n, prune | extra)
                        assert np.array_equal(T, T_gen) and plan == p_gen, (n, key, value, extra)
                    B.alpa_dp_set_tuning(h, key, 0)
                if n == 5:
                    assert np.array_equal(T_gen, T_ref)
                    _same_plan(p_gen, p_ref)
        for Bv, plan in zip([1, 40], B.alpa_dp_solve_sweep(h, few, [1, 40])):
            _, p_ref = oracle.solve_parallel(w.table, N, M, Bv, w.shapes, few, False, 8)
            _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


# 65-128 devices with so many layers and shapes that the band kernel does not fit: the register/LDS kernel's two-window form, for each
# number of waves along the layers (6, 7, 8)
WINDOW_CASES = [(96, 110, 1), (110, 49, 2), (112, 63, 2), (128, 28, 4)]


@pytest.mark.parametrize("size", WINDOW_CASES, ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_two_windows_of_the_register_kernel(size):
    K, N, M = size
    shapes = W.submesh_shapes(N, M)[:64]
    rng = np.random.default_rng(K)
    k, i = np.arange(K)[:, None], np.arange(K)[None, :]
    # stages that take longer the longer they are and the fewer devices they have, with noise; many have no entry
    a = (shapes[:, 0] * shapes[:, 1])[None, None, :]
    t = (900 * (i - k + 1))[:, :, None] // a + 30 * a + rng.integers(0, 200, (K, K, len(shapes)))
    t = np.where(((i >= k) & (rng.random((K, K)) < 0.8))[:, :, None], t, oracle.INF32).astype(np.int32)
    table = np.broadcast_to(t, (K, *t.shape)).copy()
    table[K // 2:, :, :, ::3] = oracle.INF32
    few = oracle.quantiles(np.unique(t[t != oracle.INF32]).astype(np.int32), 7)
    many = np.concatenate([few, few[-1] + 1 + np.arange(300)]).astype(np.int32)
    h = B.alpa_dp_create(table, K, N, M, 20, shapes)
    try:
        for prune in (0, B.ALPA_DP_PRUNE):
            T_gen, p_gen = B.alpa_dp_solve(h, few, flags=prune | B.ALPA_DP_GENERIC)
            assert p_gen["num_stages"] > 0
            for extra in (0, B.ALPA_DP_COUNT_WORK):
                T, plan = B.alpa_dp_solve(h, few, flags=prune | extra)        # sixteen waves a candidate
                assert np.array_equal(T, T_gen) and plan == p_gen
                T, plan = B.alpa_dp_solve(h, many, flags=prune | extra)       # eight
                assert np.array_equal(T[:7], T_gen) and plan["T_star"] == p_gen["T_star"]
                assert plan["first_layer"] == p_gen["first_layer"] and plan["shape_idx"] == p_gen["shape_idx"]
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("solved_before", [False, True])
@pytest.mark.parametrize("size", [(12, 2, 4), (70, 2, 2), (20, 18, 8)], ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}")
def test_bounds_follow_the_table(size, solved_before):
    """What is known of a table is computed by its first solve, and again when the table changes."""
    K, N, M = size
    w = _table(31 + K, K, N, M, 20_000, 0.1)
    h = B.alpa_dp_create(w.table, K, N, M, 9, w.shapes)
    try:
        if solved_before:
            B.alpa_dp_solve(h, None, 40, B.ALPA_DP_PRUNE)
        B.alpa_dp_restrict_equal_layers(h)
        masked = oracle.equal_layer_table(w.table)
        cand = oracle.quantiles(oracle.all_candidates(masked, w.shapes), 40)
        for prune in (True, False):
            T_ref, p_ref = oracle.solve_parallel(masked, N, M, 9, w.shapes, cand, prune, 8)
            T, plan = B.alpa_dp_solve(h, None, 40, B.ALPA_DP_PRUNE if prune else 0)
            assert np.array_equal(T, T_ref)
            _same_plan(plan, p_ref)
    finally:
        B.alpa_dp_destroy(h)


def test_first_solve_recorded_into_a_graph():
    """The first solve of a table as a graph: the replays compute what they need, and so does an eager solve
    made before the first replay."""
    import torch
    w = _table(51, 14, 2, 8, 20_000, 0.1)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 300)
    T_ref, p_ref = oracle.solve_parallel(w.table, 2, 8, 9, w.shapes, cand, False, 8)
    h = B.alpa_dp_create(w.table, 14, 2, 8, 9, w.shapes)
    try:
        stream = torch.cuda.Stream()
        d_T = torch.zeros(len(cand), dtype=torch.int64, device="cuda")
        d_plan = torch.zeros(B.PLAN_BYTES, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        B.alpa_dp_set_stream(h, stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.alpa_dp_solve_dev(h, None, 300, 0, d_T, d_plan)
        for replay in range(4):
            T, plan = B.alpa_dp_solve(h, None, 300, 0)             # eager, on the same buffers
            assert np.array_equal(T, T_ref)
            _same_plan(plan, p_ref)
            d_T.zero_()
            d_plan.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(d_T.cpu().numpy(), T_ref)
            _same_plan(B.plan_from_bytes(d_plan.cpu().numpy().tobytes()), p_ref)
    finally:
        B.alpa_dp_destroy(h)


def test_recorded_solve_outlives_longer_lists():
    """A recorded solve, then eager ones with lists that the handle's arrays have to grow for, replays in
    between: the graph's kernels still find their memory."""
    import torch
    w = _table(52, 14, 2, 8, 20_000, 0.1)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 300)
    T_ref, p_ref = oracle.solve_parallel(w.table, 2, 8, 9, w.shapes, cand, False, 8)
    rng = np.random.default_rng(4)
    h = B.alpa_dp_create(w.table, 14, 2, 8, 9, w.shapes)
    try:
        stream = torch.cuda.Stream()
        d_T = torch.zeros(len(cand), dtype=torch.int64, device="cuda")
        d_plan = torch.zeros(B.PLAN_BYTES, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        B.alpa_dp_set_stream(h, stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.alpa_dp_solve_dev(h, None, 300, 0, d_T, d_plan)
        for length in (2000, 7350, 20_000, 90_000):      # the table has 7350 entries
            mine = rng.choice(cand, length).astype(np.int32)
            T, _ = B.alpa_dp_solve(h, mine)
            assert np.array_equal(T, T_ref[np.searchsorted(cand, mine)])
            # whatever took the place of outgrown memory would be written by the graph
            guard = torch.full((1 << 20,), 77, dtype=torch.int32, device="cuda")
            d_T.zero_()
            d_plan.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(d_T.cpu().numpy(), T_ref)
            _same_plan(B.plan_from_bytes(d_plan.cpu().numpy().tobytes()), p_ref)
            assert bool((guard == 77).all())
    finally:
        B.alpa_dp_destroy(h)


def test_long_list_recorded_as_the_first_call():
    """The handle's arrays grow while its stream is recorded."""
    import torch
    w = _table(53, 14, 2, 8, 20_000, 0.1)
    cand = oracle.quantiles(oracle.all_candidates(w.table, w.shapes), 300)
    T_ref, p_ref = oracle.solve_parallel(w.table, 2, 8, 9, w.shapes, cand, False, 8)
    mine = np.random.default_rng(5).choice(cand, 50_000).astype(np.int32)
    mine[: len(cand)] = cand
    h = B.alpa_dp_create(w.table, 14, 2, 8, 9, w.shapes)
    try:
        stream = torch.cuda.Stream()
        d_mine = torch.from_numpy(mine).cuda()
        d_T = torch.zeros(len(mine), dtype=torch.int64, device="cuda")
        d_plan = torch.zeros(B.PLAN_BYTES, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        B.alpa_dp_set_stream(h, stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.alpa_dp_solve_dev(h, d_mine, len(mine), 0, d_T, d_plan)
        for replay in range(3):
            T, _ = B.alpa_dp_solve(h, cand)                         # eager, in between
            assert np.array_equal(T, T_ref)
            d_T.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(d_T.cpu().numpy(), T_ref[np.searchsorted(cand, mine)])
            _same_plan(B.plan_from_bytes(d_plan.cpu().numpy().tobytes()), p_ref)
    finally:
        B.alpa_dp_destroy(h)


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("size", [(3, 1, 2, 0), (12, 1, 8, 0), (24, 2, 8, 513), (14, 2, 8, 4000), (20, 4, 8, 600), (9, 8, 8, 300),
                                  (8, 10, 8, 300), (7, 17, 8, 40), (66, 1, 2, 300)],
                         ids=lambda s: f"K{s[0]}-{s[1]}x{s[2]}-n{s[3]}")
def test_first_and_later_solves_of_a_table(size, form):
    """A small problem's first solve does without the bounds, the second computes them, the third finds them:
    the same results from a new handle's first three calls, whatever they ask for, and from a recorded one."""
    import torch
    K, N, M, n = size
    w = _table(61 + K, K, N, M, 250_000, 0.15)
    cand = oracle.all_candidates(w.table, w.shapes)
    if n and len(cand) > n:
        cand = oracle.quantiles(cand, n)
    ref = {p: oracle.solve_parallel(w.table, N, M, 11, w.shapes, cand, p, 8) for p in (False, True)}
    calls = {"T": lambda h, f: B.alpa_dp_solve(h, None, n, f),
             "plan": lambda h, f: B.alpa_dp_solve(h, None, n, f, want_T=False),
             "list": lambda h, f: B.alpa_dp_solve(h, cand, flags=f),
             "sweep": lambda h, f: (None, B.alpa_dp_solve_sweep(h, None, [11, 3], n_tmax=n, flags=f)[0])}
    for first in calls:
        for prune in (False, True):
            flags = FORMS[form] | (B.ALPA_DP_PRUNE if prune else 0)
            h = B.alpa_dp_create(w.table, K, N, M, 11, w.shapes)
            try:
                for call in (first, "T", first):
                    T, plan = calls[call](h, flags)
                    if T is not None:
                        assert np.array_equal(T, ref[prune][0])
                    _same_plan(plan, ref[prune][1])
            finally:
                B.alpa_dp_destroy(h)
    h = B.alpa_dp_create(w.table, K, N, M, 11, w.shapes)
    try:
        stream = torch.cuda.Stream()
        d_T = torch.zeros(len(cand), dtype=torch.int64, device="cuda")
        d_plan = torch.zeros(B.PLAN_BYTES, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        B.alpa_dp_set_stream(h, stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.alpa_dp_solve_dev(h, None, n, FORMS[form], d_T, d_plan)
        for replay in range(3):
            d_T.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(d_T.cpu().numpy(), ref[False][0])
            _same_plan(B.plan_from_bytes(d_plan.cpu().numpy().tobytes()), ref[False][1])
            T, plan = B.alpa_dp_solve(h, None, n, FORMS[form])
            assert np.array_equal(T, ref[False][0])
    finally:
        B.alpa_dp_destroy(h)
