"""Times of 10^8 buckets and more: two or three layers, whose optimum the enumerator finds whatever the budget
is.  Rows lie in memory then and are too long for windows, and a shift or a row counted in bytes passes 2^31."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def tables(times, S=0):
    """The later levels of a layer are the better ones; S: with worthless levels in front."""
    tau = np.array(times, dtype=np.int32)
    L, n = tau.shape
    rng = np.random.default_rng(L * 100 + n)
    err = np.sort(rng.random((1, L, n), dtype=np.float32))[:, :, ::-1].copy()
    if S:
        tau = np.concatenate([np.repeat(tau[:, :1] + 1, S - n, axis=1), tau], axis=1)
        err = np.concatenate([np.full((1, L, S - n), 8.0, dtype=np.float32), err], axis=2)
    return np.ascontiguousarray(tau), np.ascontiguousarray(err)


def best(tau, err, B):
    used = err[0].min(axis=1) < 8.0
    assert used.all()
    keep = (err[0] < 8.0).all(axis=0)             # the enumerator tries all S^L profiles
    profile, cost, _, ties = oracle.brute_force(tau[:, keep], err[:, :, keep], B)
    assert ties == 1
    return np.where(profile >= 0, np.flatnonzero(keep)[profile], profile), cost


def check(profile, cost, want, what):
    assert (profile.cpu().numpy()[0] == want[0]).all(), f"{what}: {profile.cpu().numpy()} {want}"
    assert cost.cpu().numpy().view(np.uint32)[0] == np.float32(want[1]).view(np.uint32), f"{what}: cost"


# the walk's windows: a shift beyond what their sums hold, over a short row and over a long one
@pytest.mark.parametrize("S", [0, 70])
@pytest.mark.parametrize("times, B", [
    ([[0, 1], [0, 150_000_000]], 150_000_010),
    ([[0, 1], [2, (1 << 27) + 1], [0, 3], [5, 6]], (1 << 27) + 100),
    ([[0, 140_000_000], [0, 3], [0, 150_000_000]], 300_000_000),
    ([[0, 140_000_000], [0, 3], [0, 150_000_000]], 200_000_000)])
def test_walks_of_far_levels(dp, times, B, S):
    tau, err = tables(times, S)
    print(f"[far] L={len(times)} S={tau.shape[1]} B={B}", flush=True)
    want = best(tau, err, B)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    ws = dp.alloc_workspace(1, *tau.shape, B)
    profile, cost = dp.spdy_dp_solve_batched(tau_d, err_d, B, workspace=ws)
    check(profile, cost, want, "solve")
    profile.fill_(7)
    dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
    check(profile, cost, want, "walk by itself")


# layers swept from memory by a shift whose bytes pass 2^31 and 2^32 - 1, at every residue
@pytest.mark.parametrize("far", [(1 << 29) - 1, 1 << 29, (1 << 29) + 1, (1 << 29) + 2, 600_000_003])
@pytest.mark.parametrize("third", [[[0, 1]], [[0, 5]]])
def test_rows_in_memory_and_far_shifts(dp, far, third):
    tau, err = tables([[0, 4100], [0, far]] + third)
    B = far + 6000
    print(f"[far] far={far} third={third}", flush=True)
    for budget in (B, far - 1):                   # (without the far level, and with it)
        want = best(tau, err, budget)
        tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
        profile, cost = dp.spdy_dp_solve_batched(tau_d, err_d, budget,
                                                 workspace=dp.alloc_workspace(1, *tau.shape, budget))
        check(profile, cost, want, f"far={far} B={budget}")


# two rows in memory that are more than 2^31 floats together, and shifts whose bytes pass 2^32: either record, entries
# from LDS and from lanes
@pytest.mark.parametrize("S, compact", [(0, False), (66, False), (0, True)])
@pytest.mark.parametrize("far", [(1 << 30) + 1, 1_500_000_003])
def test_rows_of_more_than_a_billion_buckets(dp, far, S, compact):
    tau, err = tables([[0, 4100], [0, far]], S)
    B = far + 5000
    print(f"[far] far={far} S={tau.shape[1]} compact={compact}", flush=True)
    want = best(tau, err, B)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    profile, cost = dp.spdy_dp_solve_batched(tau_d, err_d, B,
                                             workspace=dp.alloc_workspace(1, *tau.shape, B, compact=compact))
    check(profile, cost, want, f"far={far}")
