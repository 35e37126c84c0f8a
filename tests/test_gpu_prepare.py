"""The kernel that reduces the timing table ahead of every fill: what it writes down at the numbers of
layers and levels where its split can go wrong, levels beyond the budget among them, and that
these cost no more than levels within it."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import CPU_THREADS, assert_same, check_tables, gpu_solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


# around 8 and 32 layers (of a wave and of a workgroup at a time), 256 (layers of a block), 64 levels
# (what a group of lanes reads at once), and the most levels
@pytest.mark.parametrize("L, S", [(1, 1), (7, 8), (8, 9), (9, 63), (31, 64), (32, 65), (33, 2), (10, 255),
                                  (255, 3), (256, 5), (257, 64), (300, 65), (520, 4)])
@pytest.mark.parametrize("compact", [False, True], ids=["d_record", "level_record"])
def test_levels_beyond_the_budget(dp, L, S, compact):
    rng = np.random.default_rng(1000 * L + S)
    for B, share in ((130, 0.0), (130, 0.4), (777, 0.05), (777, 0.9)):
        tau, err, _ = workloads.random_instance(rng, 2, L, S, B, tau_max=max(1, 3 * B // L),
                                                over_budget_frac=share, huge_tau_frac=share / 8,
                                                zero_tau_frac=0.1)
        tau[:, int(rng.integers(0, S))] = rng.integers(0, 1 + B // L, size=L)    # feasible
        # some layers have only just usable and only just unusable levels
        bp = B - int(tau.min(axis=1).sum())
        for l in range(0, L, 5):
            tau[l, 0] = tau[l].min() + bp + (l // 5) % 2
        what = f"L={L} S={S} B={B} share={share}"
        print(f"[prepare] {what}", flush=True)
        p_gpu, c_gpu, ws = gpu_solve(dp, tau, err, B, compact=compact)
        assert_same(p_gpu, c_gpu, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), what)
        for k in (0, 1):
            check_tables(dp, tau, err[k], B, ws, k, 2)


def test_levels_beyond_the_budget_cost_nothing(dp):
    """A fill of tables with one level of each layer beyond the budget against one of the same tables with
    that level as fast as its neighbour: the same rows and a level fewer.  Read one after the other by
    one thread such levels made it 1.12 of that; the bound lies between that and the runs' spread."""
    dev = torch.device("cuda:0")
    K, L, S, B = 1, 8, 40, 500
    rng = np.random.default_rng(5)
    inside = np.sort(rng.integers(5, 100, size=(L, S)), axis=1)[:, ::-1].astype(np.int32).copy()
    beyond = inside.copy()
    inside[:, 0] = inside[:, 1]
    beyond[:, 0] = 2 * B
    err = torch.from_numpy(rng.random((K, L, S), dtype=np.float32)).to(dev)
    ws = dp.alloc_workspace(K, L, S, B, dev)
    cost = torch.empty(K, dtype=torch.float32, device=dev)

    def least_time(tau):
        best = float("inf")
        for _ in range(12):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            for _ in range(40):
                dp.spdy_dp_fill(tau, err, B, cost, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end))
        return best

    inside, beyond = torch.from_numpy(inside).to(dev), torch.from_numpy(beyond).to(dev)
    ratios = []
    for _ in range(6):                            # (one quiet attempt is enough)
        ratios.append(least_time(beyond) / least_time(inside))
        if ratios[-1] < 1.06:
            break
    assert min(ratios) < 1.06, ratios
