"""The reduced problem (csrc/dp_core.h) against the oracle, bit for bit, at the sizes where its
mapping changes: threads per layer and layers per workgroup, levels per thread, rows and records that
outgrow their LDS, and batches in which some candidates have to fall back to the full table."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dp():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2201_13096_amd as m
    m.binding.lib()
    return m


def smooth(rng, K, L, S, B, speedup=2.5):
    """Tables of a compressed network: times fall and errors rise with the level."""
    keep = 0.05 ** (np.arange(S) / max(1, S - 1))
    dense = rng.lognormal(0.0, 0.8, L)
    t = dense[:, None] * (0.2 + 0.8 * keep) * (speedup * B / dense.sum())
    err = rng.random((K, L, 1)) * (1.0 - keep) ** 2
    return np.floor(t + 0.5).astype(np.int32), err.astype(np.float32)


def same(got, want, what):
    (p, c), (p_ref, c_ref) = got, want
    assert (c.cpu().numpy().view(np.uint32) == c_ref.view(np.uint32)).all(), f"{what}: costs"
    assert (p.cpu().numpy() == p_ref).all(), f"{what}: profiles"


def check(dp, tau, err, B, what):
    print(f"[core] {what} K={err.shape[0]} L={err.shape[1]} S={err.shape[2]} B={B}", flush=True)
    want = oracle.solve_ref(tau, err, B, threads=16)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(np.ascontiguousarray(err)).cuda()
    same(dp.spdy_dp_solve_batched(tau_d, err_d, B), want, what)
    return tau_d, err_d, want


def solve_marked(dp, tau_d, err_d, B):
    """spdy_dp_solve_profiles on a workspace of a known pattern.  The words of t* are written by the
    launches of the full table alone, so which candidates went there can be read off them; the first
    word of a candidate's share of the record tells whether the reduced solve wrote to it."""
    K, L, S = err_d.shape
    ws = dp.alloc_workspace(K, L, S, B)
    lay = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())
    at, record = lay["tstar_offset"], lay["record_offset"]
    ws[at:at + 4 * K].fill_(0xAB)
    each = (ws.numel() - record) // K // 16 * 16
    of_each = ws[record:record + K * each].view(K, each)[:, :4]
    of_each.fill_(0xAB)
    profile, cost = dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=ws)
    torch.cuda.synchronize()
    words = ws[at:at + 4 * K].cpu().numpy().view(np.uint32)
    memory = of_each.contiguous().cpu().numpy().view(np.uint32)[:, 0] != 0xABABABAB
    return (profile, cost), words != 0xABABABAB, memory


# layers: one thread to 64 per layer, the last layer of a workgroup, one more than it takes;
# levels: remainders of four, of the threads of a layer and of 64 levels per thread
@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 31, 64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("S", [1, 2, 5, 64, 67])
def test_layers_and_levels(dp, L, S):
    rng = np.random.default_rng(1000 * L + S)
    B = 3 * L + 40
    K = 260 if L <= 10 else 5                    # (a few candidates of few layers take the table)
    tau, err = smooth(rng, K, L, S, B)
    check(dp, tau, err, B, "smooth")
    tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=8, zero_tau_frac=0.1,
                                            inf_err_frac=0.05, over_budget_frac=0.05)
    err[2] = -0.0                                # ties everywhere, and the sign of a zero
    check(dp, tau, err, B, "unstructured")


@pytest.mark.parametrize("S", [128, 129, 255])
def test_many_levels(dp, S):
    rng = np.random.default_rng(S)
    for L in (9, 130):                           # 130: more than 64 levels per thread, or no LDS
        tau, err = smooth(rng, 3, L, S, 1500)
        check(dp, tau, err, 1500, "many levels")


def test_rows_and_records_that_outgrow_their_lds(dp):
    """Few layers with large times: windows of thousands of buckets, records that spill, limits
    that are exceeded (then the target is halved, or the full table takes over)."""
    rng = np.random.default_rng(77)
    for (K, L, S, B) in [(6, 6, 40, 60000), (4, 24, 60, 30000), (5, 12, 12, 100000)]:
        tau, err = smooth(rng, K, L, S, B)
        check(dp, tau, err, B, "long rows")
        tau, err, _ = workloads.random_instance(rng, K, L, S, B, tau_max=B // 4)
        check(dp, tau, err, B, "long rows, unstructured")


def test_batches_that_only_partly_reduce(dp):
    """A negative error or a NaN-free overflow sends a candidate to the full table; its neighbours
    (teams share a workgroup there) must not be touched.  All calls that reduce."""
    rng = np.random.default_rng(5)
    K, L, S, B = 37, 20, 30, 3000
    tau, err = smooth(rng, K, L, S, B)
    err[3::5, L // 2] -= 0.125
    err[6] *= np.float32(2.0 ** 126)             # sums beyond the range of fp32
    tau[7, 3] = 2 ** 31 - 1
    tau_d, err_d, want = check(dp, tau, err, B, "mixed")
    for stride in (0, 3):
        same(dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, stride), want, f"stride {stride}")
    budgets = [B, B // 2, int(tau.min(axis=1).sum()) - 1, 0] + [B - 7 * j for j in range(66)]
    p, c = dp.spdy_dp_solve_budgets(tau_d, err_d, budgets)
    for j, b in enumerate(budgets):
        same((p[j], c[j]), oracle.solve_ref(tau, err, b, threads=16), f"budget {b}")
    # an incumbent whose workspace holds no table: the candidates are solved from the first layer
    first = torch.full((K,), L // 4, dtype=torch.int32, device="cuda")
    shared = err.copy()
    shared[:, :L // 4] = err[:1, :L // 4]
    for negative in (False, True):
        ws = dp.alloc_workspace(1, L, S, B)
        c0, w0 = torch.rand((1, L), device="cuda"), torch.rand(S, device="cuda")
        dp.spdy_dp_solve_sensitivities(tau_d, -c0 if negative else c0, w0, B, workspace=ws)
        got = dp.spdy_dp_solve_from_incumbent(tau_d, torch.from_numpy(shared).cuda(), first, B, ws)
        same(got, oracle.solve_ref(tau, shared, B, threads=16), "incumbent without a table")


def test_subnormal_and_infinite_errors(dp):
    rng = np.random.default_rng(9)
    for scale in (2.0 ** -140, 2.0 ** -126, 1.0):
        tau, err = smooth(rng, 6, 15, 20, 900)
        err = (err * np.float32(scale)).astype(np.float32)
        err[1, 4] = np.inf                       # a layer without a level
        err[2, :, ::2] = np.inf
        check(dp, tau, err, 900, f"scale {scale}")


def test_a_reduced_solve_replays_from_a_graph(dp):
    rng = np.random.default_rng(12)
    K, L, S, B = 9, 14, 20, 2500
    tables = [smooth(rng, K, L, S, B) for _ in range(2)]
    tau = tables[0][0]
    errs = [t[1] for t in tables]
    errs[1][4, 2] -= 0.5                         # one candidate for the full table
    want = [oracle.solve_ref(tau, e, B) for e in errs]
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(errs[0]).cuda()
    ws = torch.empty(dp.spdy_dp_workspace_bytes_checkpointed(K, L, S, B), dtype=torch.uint8,
                     device="cuda")
    profile = torch.empty((K, L), dtype=torch.int16, device="cuda")
    cost = torch.empty((K,), dtype=torch.float32, device="cuda")
    dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, 0, profile, cost, ws)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, 0, profile, cost, ws)
    for rep in range(4):
        err_d.copy_(torch.from_numpy(errs[rep % 2]).cuda())
        profile.fill_(-9)
        cost.fill_(-9.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        same((profile, cost), want[rep % 2], f"replay {rep}")


@pytest.mark.parametrize("B", [2 ** 22 - 1, 2 ** 22, 2 ** 22 + 1])
def test_a_shift_as_long_as_the_largest_budget(dp, B):
    """A level that takes the whole budget in a layer whose fastest takes none: its shift needs one
    bit more than the budget below, and must not run into the level it is packed with."""
    tau = np.array([[5, B, 0], [B - 100] * 3], dtype=np.int32)
    err = np.array([[[1, .5, .5], [.1, .2, .3]], [[9, 0, 5], [0, 0, 0]], [[5, 0, 9], [1, 0, 0]]],
                   dtype=np.float32)
    check(dp, tau, err, B, "three levels")
    tau = np.array([[B, 5, 0], [B - 100, B, B]], dtype=np.int32)
    check(dp, tau, np.array([[[0, 9, 5], [0, 0, 0]]], dtype=np.float32), B, "one usable level")


def test_more_solves_than_one_launch_takes(dp):
    """K * J beyond 2^24 workgroups of 256 threads, the largest grid: several launches, of the reduced
    solve and of what stands behind it (every tenth candidate has a negative error)."""
    rng = np.random.default_rng(24)
    n, L, S, B, J = 110, 2, 3, 9, 70
    K = 2 ** 24 // 64 + 37
    tau = rng.integers(0, 7, size=(L, S)).astype(np.int32)
    err = rng.random((n, L, S), dtype=np.float32)
    err[::10, 1, 1] = -0.25
    budgets = [int(b) for b in rng.integers(0, B + 1, size=J)]
    p_ref, c_ref = oracle.solve_budgets_ref(tau, err, budgets)
    which = torch.arange(K, device="cuda") % n
    print(f"[core] budgets J={J} K={K} L={L} S={S} B={B}", flush=True)
    p, c = dp.spdy_dp_solve_budgets(torch.from_numpy(tau).cuda(),
                                    torch.from_numpy(err).cuda()[which], budgets)
    want_p, want_c = torch.from_numpy(p_ref).cuda(), torch.from_numpy(c_ref).cuda()
    for j in range(J):
        assert torch.equal(p[j], want_p[j][which]), f"budget {j}: profiles"
        assert torch.equal(c[j].view(torch.int32), want_c[j][which].view(torch.int32)), \
            f"budget {j}: costs"


@pytest.mark.parametrize("L", [127, 128, 130, 255, 256])
def test_layers_without_a_level(dp, L):
    """Many layers without a level that may be chosen: the sum of their least times stays beyond
    every budget, so such a candidate is settled without the full table."""
    rng = np.random.default_rng(L)
    K, S, B = 300, 5, 4 * L
    tau, err = smooth(rng, K, L, S, B)
    err[::3] = np.inf
    err[1::3, ::2] = np.inf
    tau_d, err_d, want = check(dp, tau, err, B, "layers without a level")
    got, filled, _ = solve_marked(dp, tau_d, err_d, B)
    same(got, want, "marked workspace")
    assert np.isinf(want[1][::3]).all() and not filled.any()


def test_several_budgets_behind_the_reduced_solve(dp):
    """What one budget's reduced solve found stays when another budget sends the candidate to the
    full table, and the fill leaves that table's time for the largest budget."""
    rng = np.random.default_rng(41)
    K, L, S, B = 300, 3, 6, 4000
    tau, err = smooth(rng, K, L, S, B)
    fastest = int(tau.min(axis=1).sum())
    err[1::2, 1, 2] = -0.125                     # (refused before its tables are looked at further)
    budgets = [fastest - 1, B, fastest, B // 2]
    ws = dp.alloc_workspace(K, L, S, B)
    lay = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())
    at = lay["tstar_offset"]
    ws[at:at + 4 * K].fill_(0xAB)
    print(f"[core] budgets {budgets} K={K} L={L} S={S}", flush=True)
    p, c = dp.spdy_dp_solve_budgets(torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda(),
                                    budgets, workspace=ws)
    p_ref, c_ref = oracle.solve_budgets_ref(tau, err, budgets)
    for j, b in enumerate(budgets):
        same((p[j], c[j]), (p_ref[j], c_ref[j]), f"budget {b}")
    words = ws[at:at + 4 * K].cpu().numpy().view(np.uint32)
    filled = np.flatnonzero(words != 0xABABABAB)
    assert np.isin(np.arange(1, K, 2), filled).all() and filled.size < K
    for k in filled[::20]:
        D = oracle.tables_ref(tau, err[k], B)[0]
        assert words[k] == int(np.argmin(D[L - 1])) - fastest


@pytest.mark.parametrize("compact", [False, True], ids=["d_record", "level_record"])
@pytest.mark.parametrize("S", [30, 70])
def test_a_walk_back_through_a_workspace_that_was_scratch(dp, S, compact):
    """Whatever a call leaves in its scratch workspace, t* included, a walk back through it reads no
    table and says so; once it has been filled it walks."""
    rng = np.random.default_rng(50 + S)
    K, L, B = 21, 12, 2500
    tau, err = smooth(rng, K, L, S, B)
    tau_d, err_d = torch.from_numpy(tau).cuda(), torch.from_numpy(err).cuda()
    c = torch.rand((K, L), device="cuda")
    w = torch.from_numpy(err[0, 0]).cuda()
    want = oracle.solve_ref(tau, err, B, threads=16)
    inc = dp.alloc_workspace(1, L, S, B)
    dp.spdy_dp_solve_batched(tau_d, err_d[:1].contiguous(), B, workspace=inc)
    first = torch.zeros((K,), dtype=torch.int32, device="cuda")
    calls = {"sensitivities": lambda ws: dp.spdy_dp_solve_sensitivities(tau_d, c, w, B, workspace=ws)}
    if not compact:
        calls["budgets"] = lambda ws: dp.spdy_dp_solve_budgets(tau_d, err_d, [B, B // 2],
                                                               workspace=ws)
        calls["incumbent"] = lambda ws: dp.spdy_dp_solve_from_incumbent(tau_d, err_d, first, B, inc,
                                                                        workspace=ws)
        calls["checkpointed"] = lambda ws: dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, L,
                                                                         workspace=ws)
    for name, call in calls.items():
        ws = dp.alloc_workspace(K, L, S, B, compact=compact)
        at = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["tstar_offset"]
        ws[at:at + 4 * K].fill_(0x7A)            # a time far outside every row
        print(f"[core] walk back after {name} K={K} L={L} S={S} B={B}", flush=True)
        call(ws)
        profile = torch.full((K, L), 7, dtype=torch.int16, device="cuda")
        cost = torch.full((K,), 7.0, dtype=torch.float32, device="cuda")
        dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
        assert (profile == -2).all() and torch.isnan(cost).all(), name
        dp.spdy_dp_fill(tau_d, err_d, B, cost, ws)
        dp.spdy_dp_backtrace(tau_d, err_d, B, profile, cost, ws)
        same((profile, cost), want, f"filled after {name}")


@pytest.mark.parametrize("K, L, S, B", [(20, 17, 14, 43125), (9, 21, 10, 44234), (600, 12, 11, 50000),
                                        (5, 12, 24, 100000), (520, 12, 9, 90000)])
def test_few_layers_with_long_rows(dp, K, L, S, B):
    """Rows that span a tenth of the budget and more: in LDS as far as a workgroup can have it, in
    memory beyond that (hundreds of candidates share it).  None is given up after the work is done."""
    rng = np.random.default_rng(L * S)
    tau, err = smooth(rng, K, L, S, B)
    tau_d, err_d, want = check(dp, tau, err, B, "few layers, long rows")
    got, filled, memory = solve_marked(dp, tau_d, err_d, B)
    same(got, want, "marked workspace")
    assert not filled.any(), f"{int(filled.sum())} of {K} went to the full table"
    assert K < 500 or memory.any(), "some rows were meant to lie in memory"
    for stride in (0, 1):                        # less memory for the rows of each
        same(dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, stride), want, f"stride {stride}")


def test_short_tables_are_taken_at_once(dp):
    """Calls that go to the full table without the reduced solve, on either side of the limits; and one that
    resumes from an incumbent whose own call (K = 1) did not and left no table."""
    rng = np.random.default_rng(69)
    for (K, L, S, B, at_once) in [(428, 6, 16, 134, True), (8, 9, 33, 1000, True), (8, 9, 34, 1000, False),
                                  (8, 10, 29, 1000, False), (8, 8, 20, 24998, True),
                                  (8, 8, 20, 25000, False), (257, 8, 20, 12498, True),
                                  (257, 8, 20, 12500, False), (7, 9, 33, 1000, False), (1, 8, 8, 256, True)]:
        tau, err = smooth(rng, K, L, S, B)
        tau_d, err_d, want = check(dp, tau, err, B, "around the limits")
        got, filled, _ = solve_marked(dp, tau_d, err_d, B)
        same(got, want, "marked workspace")
        assert filled.all() if at_once else not filled.all()
    K, L, S, B = 40, 9, 30, 4000
    tau, err = smooth(rng, K, L, S, B)
    c, w = rng.random((1, L)).astype(np.float32), np.sort(rng.random(S)).astype(np.float32)
    err[:, :L // 2] = (c[0, :, None] * w)[:L // 2]
    tau_d = torch.from_numpy(tau).cuda()
    inc = dp.alloc_workspace(1, L, S, B)
    inc.fill_(0x3D)
    dp.spdy_dp_solve_sensitivities(tau_d, torch.from_numpy(c).cuda(), torch.from_numpy(w).cuda(), B,
                                   workspace=inc)
    first = torch.full((K,), L // 2, dtype=torch.int32, device="cuda")
    got = dp.spdy_dp_solve_from_incumbent(tau_d, torch.from_numpy(err).cuda(), first, B, inc)
    same(got, oracle.solve_ref(tau, err, B, threads=16), "incumbent without a table")


# Candidates that the reduced solve refuses (a negative error, seen as the tables are staged) among
# candidates that it takes, at the shapes of the launches behind it: teams of a workgroup and one
# candidate per workgroup, two waves per share, turns, long rows in LDS and in memory, many levels.
GIVEN_UP_SHAPES = [(48, 54, 40, 10000), (21, 12, 8, 2000), (9, 12, 40, 30000), (5, 11, 12, 70000),
                   (11, 10, 130, 5000), (4, 10, 70, 30000), (700, 10, 6, 1500), (1300, 10, 5, 300),
                   (300, 11, 5, 30000)]


def some_given_up(K, L, S, B):
    rng = np.random.default_rng(K + 7 * L + 31 * S)
    tau, err = smooth(rng, K, L, S, B)
    refused = np.arange(K) % 3 == 1
    return rng, tau, err, refused


@pytest.mark.parametrize("K, L, S, B", GIVEN_UP_SHAPES)
def test_given_up_candidates_of_profiles_and_checkpoints(dp, K, L, S, B):
    rng, tau, err, refused = some_given_up(K, L, S, B)
    err[refused, L - 1, S // 2] = -2.0 ** -10
    tau_d, err_d, want = check(dp, tau, err, B, "given up")
    got, filled, _ = solve_marked(dp, tau_d, err_d, B)
    same(got, want, "profiles")
    assert filled[refused].all() and not filled.all()
    small = dp.alloc_workspace(K, L, S, B, compact=True)
    small.fill_(0xC3)
    same(dp.spdy_dp_solve_profiles(tau_d, err_d, B, workspace=small), want, "level record")
    for stride in (0, 1, 4):
        same(dp.spdy_dp_solve_checkpointed(tau_d, err_d, B, stride), want, f"stride {stride}")


@pytest.mark.parametrize("K, L, S, B", GIVEN_UP_SHAPES)
def test_given_up_candidates_resume_from_the_incumbent(dp, K, L, S, B):
    rng, tau, err, refused = some_given_up(K, L, S, B)
    base = err[:1].copy()
    first = rng.integers(0, L, size=K).astype(np.int32)
    first[:3] = [0, L - 1, 1]
    for k in range(K):
        err[k, :first[k]] = base[0, :first[k]]
    err[refused, L - 1, S // 2] = -2.0 ** -10
    tau_d = torch.from_numpy(tau).cuda()
    inc, ws = dp.alloc_workspace(1, L, S, B), dp.alloc_workspace(K, L, S, B)
    dp.spdy_dp_solve_batched(tau_d, torch.from_numpy(base).cuda(), B, workspace=inc)
    at = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["tstar_offset"]
    for order in (np.arange(K), np.argsort(first, kind="stable")):
        print(f"[core] resume K={K} L={L} S={S} B={B}", flush=True)
        ws.fill_(0xAB)
        got = dp.spdy_dp_solve_from_incumbent(
            tau_d, torch.from_numpy(err[order]).cuda(), torch.from_numpy(first[order]).cuda(), B,
            inc, workspace=ws)
        same(got, oracle.solve_ref(tau, err[order], B, threads=16), "resumed")
        filled = ws[at:at + 4 * K].cpu().numpy().view(np.uint32) != 0xABABABAB
        assert filled[refused[order]].all() and not filled.all()


@pytest.mark.parametrize("K, L, S, B", GIVEN_UP_SHAPES[:6])
def test_given_up_candidates_of_budgets_and_sensitivities(dp, K, L, S, B):
    rng, tau, err, refused = some_given_up(K, L, S, B)
    err[refused, L - 1, S // 2] = -2.0 ** -10
    tau_d = torch.from_numpy(tau).cuda()
    budgets = [B // 2, B, int(tau.min(axis=1).sum()), 0]
    print(f"[core] budgets {budgets} K={K} L={L} S={S}", flush=True)
    p, c = dp.spdy_dp_solve_budgets(tau_d, torch.from_numpy(err).cuda(), budgets)
    p_ref, c_ref = oracle.solve_budgets_ref(tau, err, budgets)
    for j, b in enumerate(budgets):
        same((p[j], c[j]), (p_ref[j], c_ref[j]), f"budget {b}")
    sens = rng.random((K, L), dtype=np.float32)
    sens[refused, 0] *= -1
    w = np.square(np.arange(S) / (S - 1)).astype(np.float32)
    want = oracle.solve_sens_ref(tau, sens, w, B)
    for compact in (False, True):
        ws = dp.alloc_workspace(K, L, S, B, compact=compact)
        ws.fill_(0xAB)
        same(dp.spdy_dp_solve_sensitivities(tau_d, torch.from_numpy(sens).cuda(),
                                            torch.from_numpy(w).cuda(), B, workspace=ws), want,
             f"sensitivities compact={compact}")
        at = dp.spdy_dp_workspace_layout(K, L, S, B, ws.numel())["tstar_offset"]
        filled = ws[at:at + 4 * K].cpu().numpy().view(np.uint32) != 0xABABABAB
        assert filled[refused].all() and not filled.all()


@pytest.mark.parametrize("B", [70, 200, 500, 900, 1500, 2600, 5000, 12000])
@pytest.mark.parametrize("S", [3, 12, 67])
def test_rows_around_one_chunk(dp, B, S):
    """A row of at most 64 buckets stays in a register from step to step and goes back to LDS where the
    next one is wider: rows on either side of that line and across it, more than 64 steps, layers
    between two steps on either side of a block of 64, ties, levels of equal time."""
    rng = np.random.default_rng(B + S)
    tau, err = smooth(rng, 9, 140, S, B)
    check(dp, tau, err, B, "smooth")
    check(dp, tau, np.floor(err * 8).astype(np.float32), B, "ties")
    tau, err, _ = workloads.random_instance(rng, 9, 70, S, B, tau_max=max(2, B // 35),
                                            integer_err=50, zero_tau_frac=0.1)
    check(dp, tau, err, B, "unstructured")
