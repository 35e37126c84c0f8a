"""Resumed calls that take the full table at once (csrc/spdy_dp.hip, table_is_short, and what the reduced solve does
not take), from a workspace whose last call left no table: every candidate is solved from layer 0, by the fill
as by the walk back."""
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


def leave_no_table(dp, how, tau_d, err_d, B, ws):
    L, S = tau_d.shape
    if how == "profiles":                        # toy tables are solved without one
        dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws)
    elif how == "checkpointed":
        dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, 2, workspace=ws)
    else:                                        # a resumed call's rows begin at its first layer
        base = dp.alloc_workspace(1, L, S, B)
        dp.spdy_dp_solve_batched(tau_d, err_d[:1].contiguous(), B, workspace=base)
        first = torch.full((1,), L // 2, dtype=torch.int32, device="cuda")
        dp.spdy_dp_solve_from_incumbent(tau_d, err_d[:1].contiguous(), first, B, base, workspace=ws)


# toy tables; more layers than the reduced solve takes, in few and in many levels, more candidates than units;
# rows in memory.  (Only a toy call through spdy_dp_solve_profiles leaves no table at such sizes.)
SIZES = [(8, 8, 256, 7), (9, 5, 700, 40), (300, 3, 500, 3), (260, 70, 300, 5), (290, 3, 400, 300), (3, 5, 4_300_000, 2)]
CASES = [("profiles", before, *SIZES[0]) for before in (5, 100)]
CASES += [(how, 1, *size) for how in ("checkpointed", "resumed") for size in SIZES]


@pytest.mark.parametrize("how, before, L, S, B, K", CASES)
def test_resumed_from_no_table(dp, how, before, L, S, B, K):
    rng = np.random.default_rng(L * S + before)
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=max(2, 3 * B // L))
    old = rng.random((before, L, S), dtype=np.float32)          # other errors than the candidates'
    print(f"[resume] {how} before={before} K={K} L={L} S={S} B={B}", flush=True)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    ws = dp.alloc_workspace(before, L, S, B)
    ws.zero_()
    leave_no_table(dp, how, tau_d, torch.from_numpy(old).cuda(), B, ws)
    first = torch.from_numpy(rng.integers(0, L + 1, K).astype(np.int32)).cuda()
    first[0] = L // 2
    profile, cost = dp.spdy_dp_solve_from_incumbent(tau_d, err_d, first, B, ws)
    torch.cuda.synchronize()
    assert_same(profile.cpu().numpy(), cost.cpu().numpy(), *oracle.solve_ref(tau, err, B, threads=8),
                f"{how} L={L} S={S} B={B}")
