"""What stands behind the reduced solve (csrc/spdy_dp.hip, dp_rest) where it has something to do and there are more
candidates than compute units: one and several candidates to a workgroup, rows of one chunk to rows that fit no LDS, up
to 64 levels and more, every third candidate, one of them and all of them given up, under one budget, with
checkpoints, from an incumbent, and under as many budgets as are walked back in the same launch and more.  Bit for bit
against the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_core import smooth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# in place (one to four to a workgroup), in place by sixteen waves or two rows in LDS, rows in memory
SHAPES = [(300, 11, 40, 8000), (600, 30, 70, 500), (600, 20, 66, 40), (700, 12, 20, 6000), (1100, 14, 130, 2500),
          (2100, 40, 12, 800), (2000, 11, 40, 3000), (300, 12, 40, 15000), (520, 9, 40, 25000), (600, 8, 70, 20000),
          (300, 8, 130, 45000), (300, 11, 5, 70000)]


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def instance(K, L, S, B, given_up):
    """Candidates that repeat; which of them the reduced solve refuses (a negative error in the last layer)."""
    rng = np.random.default_rng(K + 7 * L + 31 * S)
    n = 17
    tau, err = smooth(rng, n, L, S, B)
    base = err.copy()
    err[:, L - 1, S // 2] = -2.0 ** -10
    which = np.arange(K) % n
    refused = {"third": which % 3 == 1, "one": np.arange(K) == K // 2, "all": np.ones(K, bool)}[given_up]
    both = np.concatenate([base, err])
    return rng, tau, both, which + n * refused, refused


def same(got, want, which, what):
    (p, c), (p_ref, c_ref) = got, want
    assert (c.cpu().numpy().view(np.uint32) == c_ref[which].view(np.uint32)).all(), f"{what}: costs"
    assert (p.cpu().numpy() == p_ref[which]).all(), f"{what}: profiles"


@pytest.mark.parametrize("given_up", ["third", "one", "all"])
@pytest.mark.parametrize("K, L, S, B", SHAPES)
def test_one_budget_and_checkpoints(dp, K, L, S, B, given_up):
    rng, tau, err, which, refused = instance(K, L, S, B, given_up)
    print(f"[rest] K={K} L={L} S={S} B={B} {given_up}", flush=True)
    want = oracle.solve_ref(tau, err, B, threads=16)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err[which]).cuda()
    ws = dp.alloc_workspace(K, L, S, B)
    at = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["tstar_offset"]
    ws[at:at + 4 * K].fill_(0xAB)
    same(dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws), want, which, "profiles")
    filled = ws[at:at + 4 * K].cpu().numpy().view(np.uint32) != 0xABABABAB
    assert filled[refused].all() and (given_up == "all" or not filled.all())
    small = dp.alloc_workspace(K, L, S, B, compact=True)
    same(dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=small), want, which, "level record")
    del ws, small
    for stride in (0, 1, 4, L):
        same(dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, stride), want, which, f"stride {stride}")


@pytest.mark.parametrize("given_up", ["third", "one"])
@pytest.mark.parametrize("K, L, S, B", SHAPES)
def test_from_an_incumbent(dp, K, L, S, B, given_up):
    rng, tau, err, which, refused = instance(K, L, S, B, given_up)
    base = err[:1].copy()
    first = rng.integers(0, L, size=err.shape[0]).astype(np.int32)
    first[:3] = [0, L - 1, 1]
    for i, f in enumerate(first):
        err[i, :f] = base[0, :f]
    print(f"[rest] resume K={K} L={L} S={S} B={B} {given_up}", flush=True)
    want = oracle.solve_ref(tau, err, B, threads=16)
    tau_d = torch.from_numpy(tau).cuda()
    inc = dp.alloc_workspace(1, L, S, B)
    dp.spdy_dp_solve_batched(tau_d, torch.from_numpy(base).cuda(), B, workspace=inc)
    for order in (np.arange(K), np.argsort(first[which], kind="stable")):
        w = which[order]
        got = dp.spdy_dp_solve_from_incumbent(tau_d, torch.from_numpy(err[w]).cuda(),
                                              torch.from_numpy(first[w]).cuda(), B, inc)
        same(got, want, w, "resumed")


@pytest.mark.parametrize("J", [2, 4, 9, 70])
@pytest.mark.parametrize("K, L, S, B", [(20, 11, 40, 8000), (20, 12, 20, 100), (3, 12, 40, 70000)] + SHAPES)
def test_several_budgets(dp, K, L, S, B, J):
    if J > 9 and B > 3000:
        J = 17
    rng, tau, err, which, refused = instance(K, L, S, B, "one" if J == 4 else "third")
    least = int(tau.min(axis=1).sum())
    budgets = [B // 2, B, least, 0][:J] + [B - (B - least) * j // J for j in range(4, J)]
    print(f"[rest] {J} budgets K={K} L={L} S={S} B={B}", flush=True)
    want = oracle.solve_budgets_ref(tau, err, budgets, threads=16)
    p, c = dp.spdy_dp_solve_budgets(torch.from_numpy(tau).cuda(), torch.from_numpy(err[which]).cuda(), budgets)
    for j, b in enumerate(budgets):
        same((p[j], c[j]), (want[0][j], want[1][j]), which, f"budget {b}")


# blocks of layers in one launch, replayed: the marks of what is given up change from replay to replay
@pytest.mark.parametrize("K, L, S, B", [(300, 11, 40, 8000), (520, 9, 40, 25000)])
def test_checkpoints_replay_from_a_graph(dp, K, L, S, B):
    tables = [instance(K, L, S, B, given_up) for given_up in ("third", "one", "all")]
    tau = tables[0][1]
    tau_d = torch.from_numpy(tau).cuda()
    err_d = torch.from_numpy(tables[0][2][tables[0][3]]).cuda()
    ws = torch.empty(dp.spdy_dp_workspace_bytes_checkpointed(K, L, S, B), dtype=torch.uint8, device="cuda")
    profile = torch.empty((K, L), dtype=torch.int16, device="cuda")
    cost = torch.empty((K,), dtype=torch.float32, device="cuda")
    dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, 0, profile, cost, ws)
    torch.cuda.synchronize()
    print(f"[rest] graph K={K} L={L} S={S} B={B}", flush=True)
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, 0, profile, cost, ws)
    for rep in range(6):
        _, _, err, which, _ = tables[rep % 3]
        err_d.copy_(torch.from_numpy(err[which]).cuda())
        profile.fill_(-9)
        cost.fill_(-9.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        same((profile, cost), oracle.solve_ref(tau, err, B, threads=16), which, f"replay {rep}")
