"""Toy tables solved in one launch (csrc/dp_small.h): on either side of its limits, rows of odd lengths,
one to 64 levels, ties, negative and infinite errors, infeasible candidates, through the entry points whose
workspace nobody sees; and what such a call leaves in a workspace that it was given."""
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


@pytest.mark.parametrize("L, S, B", [(1, 1, 0), (1, 64, 1), (2, 3, 62), (2, 64, 63), (8, 8, 256), (9, 5, 64),
                                     (20, 8, 511), (21, 8, 513), (8, 20, 512), (8, 21, 512), (65, 2, 300),
                                     (130, 1, 255), (4, 4, 12000), (3, 4, 16000), (8, 8, 1700), (8, 8, 1800)])
def test_around_the_limits(dp, L, S, B):
    rng = np.random.default_rng(L * 70 + S)
    for K, kind in ((1, "static"), (3, "profiles"), (256, "static"), (256, "profiles")):
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=max(1, 2 * B // max(1, L)),
                                                integer_err=int(rng.choice([0, 3])) or None,
                                                inf_err_frac=0.05, over_budget_frac=0.05)
        if S > 1:
            tau[:, 0] = np.minimum(tau[:, 0], B // (2 * L))        # mostly feasible
        err[::2] -= np.float32(0.25)
        err[K // 2, L // 2] = np.inf                               # one candidate is not
        print(f"[small] {kind} K={K} L={L} S={S} B={B}", flush=True)
        tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
        if kind == "static":
            p, c = dp.spdy_dp_solve_batched_static(tau_d, err_d, B)
        else:
            p, c = dp.spdy_dp_solve_profiles(tau_d, err_d, B)
        torch.cuda.synchronize()
        assert_same(p.cpu().numpy(), c.cpu().numpy(), *oracle.solve_ref(tau, err, B),
                    f"{kind} K={K} L={L} S={S} B={B}")


def test_the_workspace_of_a_toy_call_holds_no_table(dp):
    rng = np.random.default_rng(8)
    K, L, S, B = 5, 8, 8, 256
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=40)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    want = oracle.solve_ref(tau, err, B)
    ws = dp.alloc_workspace(K, L, S, B)
    p, c = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)             # leaves a table
    p2, c2 = dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws)          # and this none
    torch.cuda.synchronize()
    for got in ((p, c), (p2, c2)):
        assert_same(got[0].cpu().numpy(), got[1].cpu().numpy(), *want, "toy")
    profile = torch.full((K, L), 7, dtype=torch.int16, device="cuda")
    cost = torch.full((K,), 7.0, dtype=torch.float32, device="cuda")
    dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
    assert (profile == -2).all() and torch.isnan(cost).all()
    dp.spdy_dp_fill(tau_d, err_d, B, cost, ws)
    dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
    assert_same(profile.cpu().numpy(), cost.cpu().numpy(), *want, "filled again")
    # a candidate by itself leaves its table, whose rows a resumed call of these sizes takes
    inc = dp.alloc_workspace(1, L, S, B)
    dp.spdy_dp_solve_profiles(tau_d, err_d[:1].contiguous(), B, workspace=inc)
    err[:, :4] = err[0, :4]
    first = torch.full((K,), 4, dtype=torch.int32, device="cuda")
    p, c = dp.spdy_dp_solve_from_incumbent(tau_d, torch.from_numpy(err).cuda(), first, B, inc)
    torch.cuda.synchronize()
    assert_same(p.cpu().numpy(), c.cpu().numpy(), *oracle.solve_ref(tau, err, B), "resumed")


def test_a_toy_call_replays_from_a_graph(dp):
    rng = np.random.default_rng(9)
    K, L, S, B = 2, 8, 8, 256
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=40, integer_err=3)
    other = workloads.random_instance(rng, K, L, S, B, tau_max=40)[1]
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    profile = torch.empty((K, L), dtype=torch.int16, device="cuda")
    cost = torch.empty((K,), dtype=torch.float32, device="cuda")
    dp.spdy_dp_solve_batched_static(tau_d, err_d, B, profile, cost)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dp.spdy_dp_solve_batched_static(tau_d, err_d, B, profile, cost,
                                        stream=torch.cuda.current_stream())
    for now in (err, other, err, other):
        err_d.copy_(torch.from_numpy(now))
        profile.fill_(9)
        graph.replay()
        torch.cuda.synchronize()
        assert_same(profile.cpu().numpy(), cost.cpu().numpy(), *oracle.solve_ref(tau, now, B), "replay")
