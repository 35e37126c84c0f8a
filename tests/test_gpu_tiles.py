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


@pytest.mark.parametrize("K, L, S, B, tau_max, kinds", [
    (1, 30, 20, 40000, 3000, None),      # many tiles
    (40, 8, 12, 33000, 9000, None),      # long tiles, aprons over two and three of them
    (128, 6, 30, 60000, 20000, 1),       # more tiles than the chip holds at once
    (128, 6, 10, 30000, 300, None),
    (200, 5, 9, 60000, 25000, None),     # more than one tile per compute unit, or rows in memory
    (2, 200, 64, 5000, 60, 0),           # entries of all layers do not fit LDS: staged again
    (3, 120, 200, 3000, 60, 0),          # ... with more than 64 levels
    (1, 300, 3, 2000, 20, 0),            # more layers than a wave plans at once
    (130, 9, 20, 3000, 700, 0),          # a tile per compute unit
])
def test_tiles_of_either_kind(dp, K, L, S, B, tau_max, kinds):
    rng = np.random.default_rng(K * 1000 + L)
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=tau_max, zero_tau_frac=0.05)
    tau[:, 0] = 0
    tiles, long_kind = check(dp, tau, err, B, "tiles")
    if kinds is not None:
        assert tiles >= 1 and long_kind == kinds


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
