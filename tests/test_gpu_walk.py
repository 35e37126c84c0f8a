"""The walk of a candidate that has a compute unit to itself (csrc/spdy_dp.hip, dp_backtrace_alone): blocks of
one to 15 layers, windows cut at bucket 0 and at the end of a row, shifts too wide for windows, several words of
levels, one candidate more than there are units, rows of an incumbent below, and a table that is not there."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def instance(rng, K, L, S, B, widest):
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=widest,
                                            integer_err=int(rng.choice([0, 3])) or None,
                                            inf_err_frac=0.05, over_budget_frac=0.05)
    tau[L // 2] = np.minimum(tau[L // 2], 3)                 # rows of very different windows
    tau[:, 0] = np.minimum(tau[:, 0], B // (2 * L))          # mostly feasible
    return tau, err


@pytest.mark.parametrize("L, S, B, widest", [
    (1, 1, 0, 1), (1, 64, 300, 300), (2, 3, 65, 40), (4, 64, 63, 63), (5, 65, 1000, 400), (15, 64, 9000, 700),
    (16, 64, 9001, 700), (17, 200, 9000, 700), (54, 40, 10000, 370), (40, 255, 3000, 90), (200, 2, 4000, 21),
    (9, 20, 60000, 30000), (9, 70, 60000, 9000), (33, 16, 40000, 5000), (6, 8, 100000, 99000)])
def test_walks(dp, L, S, B, widest):
    rng = np.random.default_rng(L * 300 + S)
    for K in (1, 3):
        tau, err = instance(rng, K, L, S, B, widest)
        err[K // 2, L // 2] = np.inf if K > 1 else err[0, L // 2]      # one candidate is not feasible
        print(f"[walk] K={K} L={L} S={S} B={B} widest={widest}", flush=True)
        tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
        want = oracle.solve_ref(tau, err, B)
        ws = dp.alloc_workspace(K, L, S, B)
        p, c = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)
        assert_same(p.cpu().numpy(), c.cpu().numpy(), *want, f"L={L} S={S} B={B}")
        p.fill_(7)
        dp.spdy_dp_backtrace(tau_d, err_d, B, p, c, ws)
        assert_same(p.cpu().numpy(), c.cpu().numpy(), *want, f"again L={L} S={S} B={B}")
        if K > 1:
            first = torch.from_numpy(np.array([0, L // 3, L], dtype=np.int32)).cuda()
            inc = dp.alloc_workspace(1, L, S, B)
            dp.spdy_dp_solve_batched(tau_d, err_d[:1].contiguous(), B, workspace=inc)
            err[1, :L // 3] = err[0, :L // 3]
            err[2] = err[0]
            p, c = dp.spdy_dp_solve_from_incumbent(tau_d, torch.from_numpy(err).cuda(), first, B, inc)
            assert_same(p.cpu().numpy(), c.cpu().numpy(), *oracle.solve_ref(tau, err, B),
                        f"resumed L={L} S={S} B={B}")


# More candidates than units: layer by layer, and from 48 layers on by guesses (blocks of eight layers, the last of them of
# one, seven or all eight; guesses that hold for smooth tables and fail in every layer for others; levels far from the
# guess; ties), and the level record's two layers at a time (odd and even numbers of layers, levels around the words of
# 64).
@pytest.mark.parametrize("S", [1, 2, 40, 63, 64, 65, 200])
@pytest.mark.parametrize("L", [1, 2, 7, 8, 9, 17, 40, 47, 48, 49, 52, 55, 65])
def test_walks_of_many(dp, L, S):
    rng = np.random.default_rng(L * 500 + S)
    K, B = 300, 60 * L + 200
    for smooth, values in ((True, None), (False, None), (False, 2)):
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=240, integer_err=values,
                                                inf_err_frac=0.0 if smooth else 0.05, over_budget_frac=0.05)
        if smooth:                                # less time, more error, at falling returns
            q = np.linspace(1.0, 0.05, S)
            tau = np.round(rng.uniform(40, 240, (L, 1)) * q).astype(np.int32)
            err = (rng.random((K, L, 1)) * (1.0 - q) ** 2).astype(np.float32)
        tau[:, -1] = np.minimum(tau[:, -1], 60)   # mostly feasible
        err[K // 3, L // 2] = np.inf              # one is not
        print(f"[walk] L={L} S={S} smooth={smooth} values={values}", flush=True)
        tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
        want = oracle.solve_ref(tau, err, B, threads=16)
        for compact in (False, True):
            ws = dp.alloc_workspace(K, L, S, B, compact=compact)
            p, c = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)
            assert_same(p.cpu().numpy(), c.cpu().numpy(), *want, f"L={L} S={S} compact={compact}")
            p.fill_(7)
            dp.spdy_dp_backtrace(tau_d, err_d, B, p, c, ws)
            assert_same(p.cpu().numpy(), c.cpu().numpy(), *want, f"again L={L} S={S} compact={compact}")


# As many candidates as have a wave each, and one more: the D record goes back to layer by layer, the level record to a
# lane per candidate (at fewer candidates where layers are few).  One in seven is not feasible.
@pytest.mark.parametrize("K, L, S", [(4096, 49, 6), (4097, 49, 6), (4096, 9, 70), (4097, 9, 70), (4097, 15, 3),
                                     (8192, 16, 70), (8193, 16, 70), (8193, 17, 5), (9000, 45, 2)])
def test_walks_of_very_many(dp, K, L, S):
    rng = np.random.default_rng(K + L + S)
    n, B = 35, 25 * L + 60
    tau, err, _ = workloads.random_instance(rng, n, L, S, B, tau_max=90, integer_err=7, inf_err_frac=0.05)
    tau[:, -1] = np.minimum(tau[:, -1], 25)
    err[::7, L // 2] = np.inf
    which = np.arange(K) % n
    want_p, want_c = (x[which] for x in oracle.solve_ref(tau, err, B))
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err[which]).cuda()
    for compact in (False, True):
        print(f"[walk] K={K} L={L} S={S} compact={compact}", flush=True)
        ws = dp.alloc_workspace(K, L, S, B, compact=compact)
        p, c = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)
        assert_same(p.cpu().numpy(), c.cpu().numpy(), want_p, want_c, f"compact={compact}")
        p.fill_(7)
        dp.spdy_dp_backtrace(tau_d, err_d, B, p, c, ws)
        assert_same(p.cpu().numpy(), c.cpu().numpy(), want_p, want_c, f"again compact={compact}")
        dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws)            # leaves no table
        dp.spdy_dp_backtrace(tau_d, err_d, B, p, c, ws)
        assert (p == -2).all() and torch.isnan(c).all()


# (several budgets over a table of eight layers are not tried by the reduced solve first)
@pytest.mark.parametrize("K, J, L", [(256, 1, 18), (257, 1, 18), (128, 2, 8), (42, 6, 8), (43, 6, 8), (128, 2, 18)])
def test_as_many_as_units(dp, K, J, L):
    rng = np.random.default_rng(K)
    S, B = 20, 700
    tau, err = instance(rng, K, L, S, B, 1600 // L)
    budgets = [B - 37 * j for j in range(J)]
    print(f"[walk] K={K} budgets={J}", flush=True)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    ws = dp.alloc_workspace(K, L, S, B)
    if J == 1:
        p, c = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)
        p, c = p[None], c[None]
    else:
        p, c = dp.spdy_dp_solve_budgets(tau_d, err_d, budgets, workspace=ws)
    for j, b in enumerate(budgets):
        assert_same(p[j].cpu().numpy(), c[j].cpu().numpy(), *oracle.solve_ref(tau, err, b), f"B={b}")


def test_no_table(dp):
    rng = np.random.default_rng(5)
    K, L, S, B = 2, 20, 8, 3000
    tau, err = instance(rng, K, L, S, B, 500)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    ws = dp.alloc_workspace(K, L, S, B)
    dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws)           # leaves none
    profile = torch.full((K, L), 7, dtype=torch.int16, device="cuda")
    cost = torch.full((K,), 7.0, dtype=torch.float32, device="cuda")
    dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
    assert (profile == -2).all() and torch.isnan(cost).all()


def test_replays_from_a_graph(dp):
    rng = np.random.default_rng(6)
    K, L, S, B = 1, 30, 16, 6000
    tau, err = instance(rng, K, L, S, B, 500)
    other = instance(rng, K, L, S, B, 500)[1]
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    profile = torch.empty((K, L), dtype=torch.int16, device="cuda")
    cost = torch.empty((K,), dtype=torch.float32, device="cuda")
    ws = dp.alloc_workspace(K, L, S, B)
    dp.spdy_dp_solve_batched(tau_d, err_d, B, profile, cost, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dp.spdy_dp_solve_batched(tau_d, err_d, B, profile, cost, workspace=ws,
                                 stream=torch.cuda.current_stream())
    for now in (err, other, err, other):
        err_d.copy_(torch.from_numpy(now))
        profile.fill_(9)
        graph.replay()
        torch.cuda.synchronize()
        assert_same(profile.cpu().numpy(), cost.cpu().numpy(), *oracle.solve_ref(tau, now, B), "replay")
