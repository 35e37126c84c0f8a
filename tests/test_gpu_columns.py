"""Folded rows (four parts of a row side by side, so that any shift is an aligned read) where their arithmetic can go
wrong: rows around whole chunks of positions for every number of teams, rows that are folded anew from layer to
layer, shifts across one, two and three parts, ties between entries that lie on either side of a part, and numbers
of levels around the blocks of 64.  Bit for bit against the oracle, the record cell by cell."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import CPU_THREADS, assert_same, check_tables, gpu_solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KINDS = [(True, 13), (True, 14), (True, 40), (True, 64), (True, 65), (True, 130), (True, 255),
         (False, 65), (False, 129), (False, 255)]


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def compare(dp, tau, err, B, compact, what):
    print(f"[columns] {what}", flush=True)
    p, c, ws = gpu_solve(dp, tau, err, B, compact=compact)
    assert_same(p, c, *oracle.solve_ref(tau, err, B, threads=CPU_THREADS), what)
    K = err.shape[0]
    for k in (0, K // 2, K - 1):
        check_tables(dp, tau, err[k], B, ws, k, K)


# up to one to a compute unit, and more: one, two and four or more to a workgroup
@pytest.mark.parametrize("K", [3, 200, 260, 600, 2100])
@pytest.mark.parametrize("compact, S", KINDS)
def test_rows_around_whole_chunks(dp, compact, S, K):
    rng = np.random.default_rng(S * 3000 + K)
    chunks = [1, 4, 5, 17, 24, 33, 61, 111, 160] if S < 255 else [2, 24, 77]
    if not compact and S < 255:
        chunks += [209, 224]                      # the longest row of a workgroup with and without turns
    if K == 2100:
        chunks = [n for n in chunks if n < 70]
    for n in chunks:
        B = 64 * n - int(rng.integers(1, 4))
        L = 4
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=max(1, B // 2), integer_err=5,
                                                inf_err_frac=0.02, over_budget_frac=0.05)
        tau[:, 0] = 0                             # nothing is subtracted: the row is the budget's
        tau[0, 1] = B                             # and reaches its end at once
        compare(dp, tau, err, B, compact, f"K={K} S={S} B={B}")


# rows that grow by less than a chunk, by a few, and by parts of their own length a layer; two and three values tie
# within and across runs, and none does
@pytest.mark.parametrize("compact, S", KINDS)
@pytest.mark.parametrize("values", [2, 3, None])
def test_rows_that_grow(dp, compact, S, values):
    rng = np.random.default_rng(S * 7 + (values or 0))
    for K, B, tau_max in ((270, 9000, 40), (600, 4800, 300), (1100, 2500, 700), (2100, 1200, 900)):
        L = 30 if tau_max < 500 else 9
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=tau_max, integer_err=values,
                                                zero_tau_frac=0.1)
        tau[:, 0] = 0
        compare(dp, tau, err, B, compact, f"K={K} S={S} B={B} tau_max={tau_max} values={values}")


# every shift a multiple of a part, one less and one more, ascending and descending with the level
@pytest.mark.parametrize("compact, S", [(True, 14), (True, 33), (True, 64), (True, 70), (False, 66), (False, 200)])
@pytest.mark.parametrize("n", [8, 20, 31])
def test_shifts_across_parts(dp, compact, S, n):
    rng = np.random.default_rng(S + n)
    K, L, B = 520, 5, 256 * n - 1                 # parts of 64 n buckets
    near = (64 * n * np.arange(4)[:, None] + 9 * np.arange(-8, 9)).ravel()
    near = np.append(near, 64 * n * np.arange(4)[:, None] + [-1, 1])
    near = np.unique(near[(near > 0) & (near <= B)])
    tau = np.sort(rng.choice(near, size=(L, S)), axis=1).astype(np.int32)
    tau[1::2] = tau[1::2, ::-1]
    tau[:, S // 2] = 0
    for err in (rng.integers(0, 3, size=(K, L, S)).astype(np.float32), rng.random((K, L, S), dtype=np.float32)):
        compare(dp, tau, err, B, compact, f"S={S} n={n}")
