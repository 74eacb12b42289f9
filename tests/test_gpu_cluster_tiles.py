"""GPU parity of operator clustering at the sizes where its row kernel changes form: one tile of prefix
lengths and several (the last one ragged), one lane per candidate and many, windows beyond what a
lane keeps in registers, more layers than rows of one launch.  Whole numbers, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2201_12023_amd import binding as B
from paper_2201_12023_amd import workloads as W

pytestmark = pytest.mark.gpu

# seed, operators, edges, layers, delta (ppm), largest FLOP figure
CASES = [(1, 1, 0, 1, 0, 9), (2, 63, 200, 5, 500000, 9), (3, 64, 200, 64, 10**9, 9), (4, 65, 300, 9, 300000, 40),
         (5, 511, 2000, 20, 500000, 9), (6, 512, 2000, 3, 200000, 9), (7, 513, 2000, 20, 500000, 9),
         (8, 576, 3000, 128, 10**6, 5), (9, 577, 3000, 129, 10**6, 5), (10, 700, 1500, 257, 2 * 10**6, 3),
         (11, 640, 4000, 2, 0, 1), (12, 900, 6000, 4, 10**9, 9), (13, 520, 0, 7, 500000, 0), (14, 600, 900, 300, 0, 50)]


# one tile of 56 prefix lengths and the next, a window of one candidate a lane and more, as many as a wave walks at a time and more
EDGES = [(15, 55, 200, 4, 500000, 9), (16, 56, 200, 5, 500000, 9), (17, 57, 200, 6, 500000, 9), (18, 112, 500, 2, 10**6, 3),
         (19, 113, 500, 14, 500000, 9), (20, 256, 900, 2, 0, 1), (21, 257, 900, 4, 10**6, 1), (22, 300, 900, 1, 0, 9)]

# windows around 128 operators, from where on sixteen lanes share a prefix length (tiles of 24), and of more than those keep (256)
WIDE = [(23, 300, 900, 4, 700000, 1), (24, 400, 1500, 5, 600000, 9), (25, 400, 1500, 5, 650000, 9), (26, 512, 3000, 3, 0, 9),
        (27, 777, 4000, 3, 200000, 5), (28, 1200, 6000, 4, 10**6, 9), (29, 1200, 300, 9, 0, 1), (30, 1200, 5000, 9, 20000, 1)]


def _edges(seed, K, E, hi):
    return W.random_op_graph(seed, K, E, flop_hi=hi)


@pytest.mark.parametrize("case", CASES + EDGES + WIDE, ids=lambda c: f"K{c[1]}-L{c[3]}")
@pytest.mark.parametrize("rule", ["cell", "exact", "static"])
def test_tiles_and_windows(case, rule):
    import torch
    seed, K, E, L, delta, hi = case
    if rule == "static" and max(K, L) > B.CLUSTER_STATIC_MAX_OPS:
        pytest.skip("beyond the fixed work memory")
    g = _edges(seed, K, E, hi)
    args = (g.flop, g.src, g.dst, g.nbytes)
    want = (oracle.cluster_exact if rule == "exact" else oracle.cluster)(*args, L, delta)
    for _ in range(2):                              # the second call finds the first one's work memory
        if rule == "static":
            out = torch.zeros(3, dtype=torch.int64, device="cuda")
            first = torch.zeros(L + 1, dtype=torch.int32, device="cuda")
            B.alpa_cluster_layers_static(*[torch.from_numpy(a).cuda() for a in args], L, delta, out, first)
            comm, sumsq, status = out.tolist()
            assert status == 0
            got = (comm, sumsq, first.tolist() if comm != B.INF_I64 else [])
        else:
            call = B.alpa_cluster_layers_exact if rule == "exact" else B.alpa_cluster_layers
            r = call(*args, L, delta)
            got = (r["comm"], r["sumsq"], r["first_op"])
        assert got == want


def test_refused_figures_reach_no_wait():
    """Negative FLOP figures, refused by the check on the device, whose wrapped sum of squares over the first
    four operators is -1: the value by which a row says that it is not there yet, in a tile that the
    next one waits for."""
    import torch
    f = [3122172103, 2200318541, 3694363990, 2942074529]
    assert sum(x * x for x in f) % 2**64 == 2**64 - 1
    flop = np.array([x - 2**32 for x in f] + [-1] * 146, dtype=np.int32)
    none32, none64 = torch.zeros(0, dtype=torch.int32).cuda(), torch.zeros(0, dtype=torch.int64).cuda()
    for L in (5, 140):
        out = torch.zeros(3, dtype=torch.int64, device="cuda")
        first = torch.zeros(L + 1, dtype=torch.int32, device="cuda")
        B.alpa_cluster_layers_static(torch.from_numpy(flop).cuda(), none32, none32, none64, L, 500000, out, first)
        torch.cuda.synchronize()
        assert out.tolist() == [B.INF_I64, 0, -1] and first.tolist() == [-1] * (L + 1)


@pytest.mark.parametrize("exact", [0, 1])
def test_a_wait_that_runs_out_is_reported(exact):
    """With no time to wait in, the first value that is not there yet ends the call with a status; with the usual
    time the same call, on the memory that the first one gave back, is right."""
    import ctypes
    g = W.make_op_graph(3, 60)                       # 12 tiles, 31 rows that wait
    L, first = 32, np.zeros(33, np.int32)
    comm, sumsq = ctypes.c_int64(), ctypes.c_int64()
    ptr = lambda a: ctypes.c_void_p(a.ctypes.data)
    rc = B.load().alpa_cluster_layers_waiting_(ptr(g.flop), g.K, ptr(g.src), ptr(g.dst), ptr(g.nbytes), len(g.src), L,
                                               500000, exact, 0, ctypes.byref(comm),
                                               ctypes.byref(sumsq), ptr(first))
    assert rc == -4 and b"wait" in B.load().alpa_dp_last_error()
    call = B.alpa_cluster_layers_exact if exact else B.alpa_cluster_layers
    r = call(g.flop, g.src, g.dst, g.nbytes, L, 500000)
    want = (oracle.cluster_exact if exact else oracle.cluster)(g.flop, g.src, g.dst, g.nbytes, L, 500000)
    assert (r["comm"], r["sumsq"], r["first_op"]) == want
