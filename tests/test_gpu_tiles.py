"""GPU parity of the fill that cuts a candidate's rows into tiles, one workgroup each: profiles, costs
and the whole record against the oracle, bit for bit, at the sizes where tiles, their aprons, the
staging of the entries and the final argmin over the tiles can go wrong."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import CPU_THREADS, assert_same, check_tables, gpu_solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES_WORD = 19      # of the header: tiles | long kind << 11 | quads of the apron << 12


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def plan(dp, ws, K, L, S, B):
    off = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["meta_offset"]
    word = int(ws[off:off + 80].cpu().numpy().view(np.int32)[TILES_WORD])
    return word & 0xFF, word >> 11 & 1


def check(dp, tau, err, B, what):
    K, L, S = err.shape
    p_gpu, c_gpu, ws = gpu_solve(dp, tau, err, B)
    p_ref, c_ref = oracle.solve_ref(tau, err, B, threads=CPU_THREADS)
    assert_same(p_gpu, c_gpu, p_ref, c_ref, what)
    for k in sorted({0, K // 2, K - 1}):
        check_tables(dp, tau, err[k], B, ws, k, K)
    return plan(dp, ws, K, L, S, B)


@pytest.mark.parametrize("S", [1, 5, 8, 40, 64, 65, 129, 255])
def test_rows_around_tile_boundaries(dp, S):
    """Reduced rows of a few chunks more or less one, shifts from far below a chunk to the whole row
    (aprons that reach over several tiles and past the start of the row), one to many candidates."""
    rng = np.random.default_rng(300 + S)
    seen = set()
    for B in (0, 1, 62, 63, 64, 127, 251, 252, 253, 1000, 2015, 2016, 4031, 4033, 7000):
        for tau_max in (1, max(1, B // 30), max(1, B // 3), B + 1):
            K, L = int(rng.integers(1, 9)), int(rng.integers(1, 13))
            tau, err, _ = workloads.random_instance(
                rng, K, L, S, B, tau_max=tau_max, integer_err=3 if rng.random() < 0.5 else None,
                inf_err_frac=0.05 if rng.random() < 0.3 else 0.0)
            what = f"K={K} L={L} S={S} B={B} tau_max={tau_max}"
            print(f"[tiles] {what}", flush=True)
            seen.add(check(dp, tau, err, B, what))
    assert S < 40 or max(tiles for tiles, _ in seen) > 1


@pytest.mark.parametrize("K, L, S, B, tau_max, kinds, least", [
    (1, 30, 20, 40000, 3000, None, 5),       # many tiles
    (40, 8, 12, 33000, 9000, None, 2),       # aprons over two and three of them
    (128, 6, 30, 60000, 20000, 1, 3),        # more tiles than the chip holds at once
    (128, 6, 10, 30000, 300, None, 1),
    (200, 5, 9, 60000, 25000, None, 0),      # more than one tile per compute unit, or rows in memory
    (2, 200, 64, 5000, 60, 0, 2),            # most layers that are staged at once (see staged_layers)
    (3, 120, 200, 3000, 60, 0, 2),           # more than 64 levels
    (1, 300, 3, 2000, 20, 0, 2),             # more layers than a wave plans at once
    (130, 9, 20, 3000, 700, 0, 1),           # a tile per compute unit
])
def test_tiles_of_either_kind(dp, K, L, S, B, tau_max, kinds, least):
    rng = np.random.default_rng(K * 1000 + L)
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=tau_max, zero_tau_frac=0.05)
    tau[:, 0] = 0
    tiles, long_kind = check(dp, tau, err, B, "tiles")
    print(f"[tiles] K={K} L={L} S={S} B={B}: {tiles} of kind {long_kind}", flush=True)
    assert tiles >= least and kinds in (None, long_kind)


def test_ties_across_tiles_and_zeros_of_either_sign(dp):
    """Costs that tie at times in different tiles (the smallest time wins), and least costs that are
    zeros of either sign."""
    rng = np.random.default_rng(77)
    L, S, B = 30, 48, 9000
    for zero in (0.0, -0.0):
        tau = rng.integers(0, 900, size=(L, S)).astype(np.int32)
        err = np.full((2, L, S), np.float32(zero))
        err[1] = rng.integers(0, 2, size=(L, S)).astype(np.float32)
        tiles, _ = check(dp, tau, err, B, f"zero {zero}")
        assert tiles > 1


def test_infeasible_candidates(dp):
    rng = np.random.default_rng(78)
    tau = rng.integers(50, 900, size=(9, 7)).astype(np.int32)
    err = rng.random((5, 9, 7), dtype=np.float32)
    err[2, 4] = np.inf
    for B in (10, int(tau.min(axis=1).sum()) - 1, int(tau.min(axis=1).sum()), 5000):
        check(dp, tau, err, B, f"B={B}")


def test_two_streams_at_once(dp):
    """Solves that fill the chip with waiting tiles, on two streams at the same time: every tile must
    still get its turn."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(79)
    L, S, B = 20, 16, 9000
    jobs = []
    for i in range(2):
        K = 60 + i
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=B // 12)
        jobs.append(dict(tau=torch.from_numpy(tau).to(dev), err=torch.from_numpy(err).to(dev),
                         ws=dp.alloc_workspace(K, L, S, B, dev),
                         profile=torch.empty((K, L), dtype=torch.int16, device=dev),
                         cost=torch.empty(K, dtype=torch.float32, device=dev),
                         stream=torch.cuda.Stream(), want=oracle.solve_ref(tau, err, B, threads=CPU_THREADS)))
    torch.cuda.synchronize()
    for _ in range(5):
        for j in jobs:
            with torch.cuda.stream(j["stream"]):
                dp.spdy_dp_solve_batched(j["tau"], j["err"], B, j["profile"], j["cost"], j["ws"])
    torch.cuda.synchronize()
    for j in jobs:
        assert_same(j["profile"].cpu().numpy(), j["cost"].cpu().numpy(), *j["want"], "streams")


LDS_FLOATS = (160 * 1024 - 1024) // 4            # of a tile's workgroup


def staged_layers(dp, ws, K, L, S, B):
    """Layers whose entries lie in LDS at a time, from the plan in the header."""
    lay = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())
    off, header = lay["meta_offset"], lay["header_words"]
    meta = ws[off:off + 4 * (header + 2 * L)].cpu().numpy().view(np.int32)
    word = int(meta[TILES_WORD])
    tiles, long_kind, apron = word & 0xFF, word >> 11 & 1, (word >> 12) * 4
    grain = 252 if long_kind else 64
    units = -(-int(meta[header + 2 * L - 1]) * 64 // grain)
    lines = (1 if long_kind else 2) * (apron + -(-units // tiles) * grain)
    s8 = (S + 7) // 8 * 8
    return min((LDS_FLOATS - lines) // (2 * s8 + 1), L), tiles, long_kind


@pytest.mark.parametrize("K, L, S, B, tau_max, kind", [
    (2, 400, 64, 5000, 60, 0),           # short tiles
    (100, 300, 64, 12000, 80, 1),        # long tiles: one row, its entries overwritten mid-solve
    (3, 200, 255, 3000, 60, 0),          # most levels
])
def test_entries_staged_more_than_once(dp, K, L, S, B, tau_max, kind):
    rng = np.random.default_rng(90 + L)
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=tau_max, zero_tau_frac=0.05)
    tau[:, 0] = 0
    p_gpu, c_gpu, ws = gpu_solve(dp, tau, err, B)
    room, tiles, long_kind = staged_layers(dp, ws, K, L, S, B)
    assert room < L and tiles > 1 and long_kind == kind, (room, tiles, long_kind)
    assert_same(p_gpu, c_gpu, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), "staged again")
    for k in sorted({0, K - 1}):
        check_tables(dp, tau, err[k], B, ws, k, K)


@pytest.mark.parametrize("K, L, S, B, tau_max, most", [
    (3, 9, 100, 30000, 6000, 16),        # the books lie where rows in memory would
    (130, 20, 70, 30000, 2000, 16),      # fewer workgroups than tiles: each takes several
    (300, 10, 40, 60000, 7000, 16),
    (130, 3, 70, 45000, 20000, 0),       # aprons that leave no room for tiles
    (600, 4, 9, 30000, 200, 0),          # rows that fit LDS after all: no tiles
])
def test_tiles_where_rows_may_lie_in_memory(dp, K, L, S, B, tau_max, most):
    rng = np.random.default_rng(K + S)
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=tau_max, zero_tau_frac=0.05)
    tau[:, 0] = 0 if most else B // L - 5
    tau[:, 1:] += tau[:, :1]
    tiles, _ = check(dp, tau, err, B, "rows in memory")
    assert 1 < tiles <= most or tiles == most


def test_budgets_and_a_resumed_call_behind_tiles(dp):
    """Several budgets on a table short enough to be filled at once, and candidates that start from rows
    that tiles have filled."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(81)
    K, L, S, B = 5, 5, 7, 900
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=B // 3, integer_err=3)
    tau_d, err_d = torch.from_numpy(tau).to(dev), torch.from_numpy(err).to(dev)
    ws = dp.alloc_workspace(K, L, S, B, dev)
    budgets = [B, B // 2, int(tau.min(axis=1).sum()), 0]
    profile = torch.empty((len(budgets), K, L), dtype=torch.int16, device=dev)
    cost = torch.empty((len(budgets), K), dtype=torch.float32, device=dev)
    dp.spdy_dp_solve_budgets(tau_d, err_d, budgets, profile, cost, ws)
    torch.cuda.synchronize()
    assert plan(dp, ws, K, L, S, B)[0] >= 1
    for j, b in enumerate(budgets):
        assert_same(profile[j].cpu().numpy(), cost[j].cpu().numpy(), *oracle.solve_ref(tau, err, b), f"{b}")

    K, L, S, B = 9, 12, 20, 30000
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=B // 5, integer_err=4)
    first = np.sort(rng.integers(0, L + 1, size=K)).astype(np.int32)
    for k in range(K):
        err[k, :first[k]] = err[0, :first[k]]
    tau_d, err_d = torch.from_numpy(tau).to(dev), torch.from_numpy(err).to(dev)
    incumbent = dp.alloc_workspace(1, L, S, B, dev)
    dp.spdy_dp_solve_batched(tau_d, err_d[:1].contiguous(), B, workspace=incumbent)
    assert plan(dp, incumbent, 1, L, S, B)[0] > 1
    ws = dp.alloc_workspace(K, L, S, B, dev)
    profile = torch.empty((K, L), dtype=torch.int16, device=dev)
    cost = torch.empty((K,), dtype=torch.float32, device=dev)
    dp.spdy_dp_solve_from_incumbent(tau_d, err_d, torch.from_numpy(first).to(dev), B, incumbent, profile,
                                    cost, ws)
    torch.cuda.synchronize()
    assert_same(profile.cpu().numpy(), cost.cpu().numpy(),
                *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), "resumed")


def test_rows_that_fit_after_all_cost_no_idle_launch(dp):
    """The same reduced table under a budget from which rows may lie in memory and under one below it: the
    first has one more launch to enqueue (1.1 of the time), and no thousands of workgroups that find no
    tiles (1.3)."""
    dev = torch.device("cuda:0")
    K, L, S, B = 1024, 8, 16, 30000
    rng = np.random.default_rng(3)
    tau = np.sort(rng.integers(3600, 3900, size=(L, S)), axis=1)[:, ::-1].astype(np.int32)
    err = torch.from_numpy(rng.random((K, L, S), dtype=np.float32)).to(dev)
    cost = torch.empty(K, dtype=torch.float32, device=dev)

    def least_time(less):
        b = B - L * less
        tau_d = torch.from_numpy((tau - less).copy()).to(dev)
        ws = dp.alloc_workspace(K, L, S, b, dev)
        best = float("inf")
        for _ in range(12):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            for _ in range(30):
                dp.spdy_dp_fill(tau_d, err, b, cost, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end))
        assert plan(dp, ws, K, L, S, b)[0] == 0
        return best

    ratios = []
    for _ in range(6):                           # (one quiet attempt is enough)
        ratios.append(least_time(0) / least_time(500))
        if ratios[-1] < 1.2:
            break
    assert min(ratios) < 1.2, ratios
