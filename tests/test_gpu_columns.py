"""Folded rows (four parts of a row side by side, so that any shift is an aligned read) where their arithmetic can go
wrong: rows around whole chunks of positions for every number of teams, rows that are folded anew from layer to
layer, shifts across one, two and three parts, ties between entries that lie on either side of a part, and numbers
of levels around the blocks of 64.  Bit for bit against the oracle, the record cell by cell; which launch did the work
and how it was planned is read from the header of the workspace."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import CPU_THREADS, assert_same, check_tables, gpu_solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KINDS = [(True, 13), (True, 14), (True, 15), (True, 16), (True, 17), (True, 40), (True, 64), (True, 65), (True, 130), (True, 255),
         (False, 65), (False, 129), (False, 255)]


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


def header(dp, ws, K, L, S, B):
    off = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["meta_offset"]
    return [int(x) for x in ws[off:off + 4 * 20].cpu().numpy().view(np.int32)]


def is_folded(K, L, S, B, compact):
    """Where a row updated in place is folded: the dispatch, written down a second time."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    if not compact:
        return K > units and S > 64
    return K > units and S >= 16 and B >= 800 and (K <= 4 * units or L * S >= 300)


def check_header(words, K, L, S, B, compact):
    """The words that name the launch and its plan; True if rows were folded."""
    in_place = words[3] == 1
    assert (words[19] < 0) == (in_place and is_folded(K, L, S, B, compact)), words
    if words[19] >= 0:
        return False
    waves, teams = words[4], words[5]
    assert words[19] in (-1, -4) and words[8] == 8 and 1 <= teams <= 8 and waves == 8 // teams
    assert words[9] == (20 if compact else 28)
    # bytes of LDS for windows of rows in memory: half of a unit's or all of it, whatever did the work
    assert words[7] >= words[10] > 0
    return True


def compare(dp, tau, err, B, compact, what, copies=None):
    """`copies`: that many candidates, those of `err` one after the other and again."""
    which = np.arange(copies or err.shape[0]) % err.shape[0]
    K, (L, S) = which.size, tau.shape
    print(f"[columns] {what}", flush=True)
    p, c, ws = gpu_solve(dp, tau, err[which], B, compact=compact)
    p_ref, c_ref = oracle.solve_ref(tau, err, B, threads=CPU_THREADS)
    assert_same(p, c, p_ref[which], c_ref[which], what)
    words = header(dp, ws, K, L, S, B)
    folded = check_header(words, K, L, S, B, compact)
    for k in (0, K // 2, K - 1):
        check_tables(dp, tau, err[which[k]], B, ws, k, K)
    return folded, words


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
        L = -(-300 // S) if compact and K > 1024 else 4
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


# reduced rows of a few chunks under a budget that is long: most of it is the least times'.  One to eight candidates to a
# workgroup, rows folded and not
@pytest.mark.parametrize("compact, S", [(True, 16), (True, 17), (True, 40), (True, 64), (True, 65), (True, 130),
                                        (False, 65), (False, 130)])
@pytest.mark.parametrize("K", [257, 600, 1100, 2100, 4000])
def test_short_rows_of_long_budgets(dp, compact, S, K):
    rng = np.random.default_rng(S * 70 + K)
    L, seen = 20, set()
    for n in (1, 2, 3, 4, 5, 6, 8, 9, 13, 17, 25):
        bp = 64 * n - int(rng.integers(1, 4))
        tau, err, _ = workloads.random_instance(rng, 37, L, S, bp, tau_max=max(1, bp // 3),
                                                integer_err=5 if n % 2 else None, inf_err_frac=0.02)
        tau[:, 0] = 0
        tau[0, 1] = bp
        floor = rng.integers(20, 90, size=(L, 1)).astype(np.int32)
        B = bp + int(floor.sum())
        folded, words = compare(dp, tau + floor, err, B, compact, f"K={K} S={S} B={B} row={bp}", copies=K)
        assert folded == (not compact or B >= 800)
        if folded:
            seen.add((words[5], words[19]))
    assert {cells for _, cells in seen} == {-1, -4}
    assert max(teams for teams, _ in seen) == min(8, -(-K // 512))


# on either side of every line of the rule that folds rows, and where nothing is feasible
@pytest.mark.parametrize("compact, K, L, S, B, folded", [
    (True, 256, 20, 16, 900, False), (True, 257, 20, 16, 900, True), (True, 300, 20, 15, 900, False),
    (True, 300, 20, 16, 799, False), (True, 300, 20, 16, 800, True), (True, 1024, 10, 16, 900, True),
    (True, 1025, 18, 16, 900, False), (True, 1025, 19, 16, 900, True), (False, 257, 5, 64, 900, False),
    (False, 256, 5, 65, 900, False), (False, 257, 5, 65, 900, True), (False, 300, 5, 65, 10, True),
    (False, 300, 5, 65, 0, True)])
def test_which_launch(dp, compact, K, L, S, B, folded):
    rng = np.random.default_rng(K + L + S + B)
    tau, err, _ = workloads.random_instance(rng, 30, L, S, B, tau_max=max(1, B // 4), zero_tau_frac=0.2)
    tau[:, 0] = 0
    assert compare(dp, tau, err, B, compact, f"K={K} L={L} S={S} B={B}", copies=K)[0] == folded
    tau += B // L + 1
    words = compare(dp, tau, err, B, compact, f"not feasible K={K} L={L} S={S} B={B}", copies=K)[1]
    assert words[0] == -1


# As many candidates to a workgroup as there is room for, but fewer where that saves most of a round of workgroups
@pytest.mark.parametrize("K, S, n, teams", [(3000, 128, 17, 4), (4000, 70, 19, 4), (4000, 40, 13, 4), (4000, 40, 17, 4),
                                            (2100, 40, 25, 3), (4000, 40, 6, 8), (2100, 40, 12, 5), (600, 40, 13, 2)])
def test_candidates_of_a_workgroup(dp, K, S, n, teams):
    rng = np.random.default_rng(K + S + n)
    L, B = 8, 64 * n - 3
    L = -(-300 // S) if L * S < 300 else L
    tau, err, _ = workloads.random_instance(rng, 37, L, S, B, tau_max=B // 2, integer_err=9)
    tau[:, 0] = 0
    tau[0, 1] = B
    tau[-1] += 900                                # a budget that is long enough for the level record
    folded, words = compare(dp, tau, err, B + 900, True, f"K={K} S={S} row={B}", copies=K)
    assert folded and words[5] == teams, words
