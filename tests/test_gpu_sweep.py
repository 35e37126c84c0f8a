"""The D-record sweep with 128-bit reads at the sizes where its split can go wrong: rows just below, at and
just above whole numbers of 252-bucket quad chunks per wave, for teams of eight, four and two waves, and
runs of entries of every residue with none, one, two or all of 64 levels in them."""
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


# more candidates than compute units (fewer are swept by twice the waves), two and four per unit
@pytest.mark.parametrize("K", [260, 600, 1100])
@pytest.mark.parametrize("row", [64, 252, 504, 1008, 1260, 2016, 3528, 5040, 7056, 13300])
def test_rows_around_whole_quad_chunks(dp, K, row):
    rng = np.random.default_rng(100 * row + K)
    # (rows of up to six chunks a wave only take quad chunks if levels times chunks are more than 120)
    for B, S in ((row - 2, 13), (row - 1, 8), (row, 3), (row - 1, 64), (row, 41)):
        L = 4
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=max(1, B // 2), integer_err=5,
                                                inf_err_frac=0.02)
        tau[:, 0] = 0                             # nothing is subtracted: the row is the budget's
        tau[0, 1] = B                             # and reaches its end at once
        what = f"K={K} S={S} B={B}"
        print(f"[sweep] {what}", flush=True)
        p, c, ws = gpu_solve(dp, tau, err, B)
        assert_same(p, c, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), what)
        for k in (0, K // 2, K - 1):
            check_tables(dp, tau, err[k], B, ws, k, K)


@pytest.mark.parametrize("K", [2, 260])           # by twice the waves (or in tiles), and by the usual number
@pytest.mark.parametrize("S", [1, 2, 5, 63, 64])
@pytest.mark.parametrize("residues", [(0,), (1,), (3,), (0, 2), (1, 2, 3), (0, 1, 2, 3)])
def test_runs_of_entries(dp, K, S, residues):
    rng = np.random.default_rng(S * 16 + sum(1 << r for r in residues))
    for B in (300, 2300, 9000):
        L = 3
        err = rng.random((K, L, S), dtype=np.float32)
        shifts = 4 * rng.permuted(np.tile(np.arange(max(S, B // 4 - 1)), (L, 1)), axis=1)[:, :S]
        tau = (shifts + rng.choice(residues, size=(L, S))).astype(np.int32)
        tau[:, 0] = 0                             # (shifts count from the least time)
        what = f"K={K} S={S} B={B} residues={residues}"
        print(f"[sweep] {what}", flush=True)
        p, c, ws = gpu_solve(dp, tau, err, B)
        assert_same(p, c, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), what)
        check_tables(dp, tau, err[K - 1], B, ws, K - 1, K)


# one to 49 levels in up to six chunks of 64 buckets a wave and one more, for teams of eight and of two waves
@pytest.mark.parametrize("K", [260, 1100])
@pytest.mark.parametrize("S", [1, 3, 4, 5, 8, 9, 12, 16, 24, 48, 49])
def test_few_levels_and_chunks(dp, K, S):
    rng = np.random.default_rng(S * 10000 + K)
    waves, L = (8 if K == 260 else 2), 4
    for chunks in (1, 2, 3, 4, 6, 7):
        B = 64 * chunks * waves - int(rng.integers(0, 3))
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=max(1, B // 2), integer_err=5,
                                                inf_err_frac=0.02, over_budget_frac=0.05)
        tau[:, 0] = 0
        if S > 1:
            tau[0, 1] = B
        err[::2] = err[::2] / np.float32(3.0) - np.float32(0.5)       # some without ties, some negative
        what = f"K={K} S={S} B={B}"
        print(f"[sweep] {what}", flush=True)
        p, c, ws = gpu_solve(dp, tau, err, B)
        assert_same(p, c, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), what)
        for k in (0, K - 1):
            check_tables(dp, tau, err[k], B, ws, k, K)
