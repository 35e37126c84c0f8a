"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every function the
header declares, sizes its workspace as documented and rejects bad arguments before touching
the device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "spdy_dp.h")


@pytest.fixture(scope="module")
def binding():
    from paper_2201_13096_amd import binding as b
    if not os.path.exists(b.LIB_PATH):
        from paper_2201_13096_amd import build
        build.build_library()
    return b


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(spdy_dp_\w+)\s*\(", text)))


def test_library_exports_every_declared_function(binding):
    names = declared_functions()
    assert len(names) >= 9
    lib = ctypes.CDLL(binding.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(binding.EXPORTS) == names


def test_status_codes_match_header(binding):
    text = open(HEADER).read()
    codes = dict(re.findall(r"#define\s+SPDY_DP_(OK|ERR_\w+)\s+\(?(-?\d+)\)?", text))
    assert int(codes["OK"]) == binding.OK
    assert int(codes["ERR_NULL"]) == binding.ERR_NULL
    assert int(codes["ERR_DIM"]) == binding.ERR_DIM
    assert int(codes["ERR_LEVELS"]) == binding.ERR_LEVELS
    assert int(codes["ERR_WORKSPACE"]) == binding.ERR_WORKSPACE
    assert int(codes["ERR_OVERFLOW"]) == binding.ERR_OVERFLOW
    assert int(codes["ERR_LAUNCH"]) == binding.ERR_LAUNCH
    assert int(codes["ERR_STATIC_LIMIT"]) == binding.ERR_STATIC_LIMIT
    limit = re.search(r"#define\s+SPDY_DP_STATIC_WORKSPACE_BYTES\s+\(\(size_t\)(\d+)\s*<<\s*(\d+)\)",
                      text)
    assert int(limit.group(1)) << int(limit.group(2)) == binding.STATIC_WORKSPACE_BYTES
    for v in codes.values():
        assert binding.spdy_dp_strerror(int(v)) != "unknown status"
    assert binding.spdy_dp_strerror(-1234) == "unknown status"


def test_workspace_size(binding):
    K, L, S, B = 1024, 54, 40, 10000
    row = (B + 1 + 63) // 64 * 64
    fast = binding.spdy_dp_workspace_bytes(K, L, S, B)
    small = binding.spdy_dp_workspace_bytes_min(K, L, S, B)
    # fp32 D per cell (one extra row per candidate) vs one byte per cell, rows padded to 64
    # per (layer, level): shifts, visiting order, entry starts (8 more per layer), entry of a level
    tables = 4 * 4 * L * ((S + 7) // 8 * 8) + 4 * 8 * L
    assert 4 * K * L * row + tables <= fast <= 4 * K * L * row + tables + 16384
    assert K * L * row + tables <= small <= K * L * row + tables + 16384
    lay = binding.spdy_dp_workspace_layout(K, L, S, B, fast)
    assert lay["variant"] == 0 and lay["record_pitch"] == row and lay["record_rows"] == L
    lay = binding.spdy_dp_workspace_layout(K, L, S, B, fast - 1)
    assert lay["variant"] == 1 and lay["record_pitch"] == row and lay["record_rows"] == L
    assert lay["record_offset"] % 256 == 0 and lay["tstar_offset"] % 256 == 0
    assert lay["tstar_offset"] >= 4 * (8 + 2 * L) + tables
    assert lay["record_offset"] >= lay["tstar_offset"] + 4 * K
    with pytest.raises(binding.SpdyDpError) as e:
        binding.spdy_dp_workspace_layout(K, L, S, B, small - 1)
    assert e.value.status == binding.ERR_WORKSPACE
    # rows that may not fit LDS add two fp32 rows per candidate
    K, L, S, B = 256, 200, 64, 65536
    row = (B + 1 + 63) // 64 * 64
    assert binding.spdy_dp_workspace_bytes_min(K, L, S, B) >= K * L * row + 2 * K * row * 4
    assert binding.spdy_dp_workspace_bytes(K, L, S, B) >= 4 * K * L * row + 2 * K * row * 4
    # the record with checkpoints: L / stride - 1 checkpoint rows + stride block rows per candidate
    K, L, S, B = 256, 200, 64, 65536
    row = (B + 1 + 63) // 64 * 64
    full = binding.spdy_dp_workspace_bytes(K, L, S, B)
    auto = binding.spdy_dp_workspace_bytes_checkpointed(K, L, S, B, 0)      # stride 15
    spill = 2 * K * (row + 1792) * 4            # two rows per candidate in memory (long rows)
    assert 4 * K * (13 + 15) * row + spill <= auto <= 4 * K * (13 + 15) * row + spill + (1 << 20)
    assert auto * 5 < full
    assert binding.spdy_dp_workspace_bytes_checkpointed(K, L, S, B, 10) == \
        binding.spdy_dp_workspace_bytes_checkpointed(K, L, S, B, 20)        # 19 + 10 = 9 + 20
    assert binding.spdy_dp_workspace_bytes_checkpointed(K, L, S, B, 1000) >= full   # one block
    assert binding.spdy_dp_workspace_bytes_checkpointed(K, 0, S, B, 0) == 0
    # invalid sizes -> 0
    for f in (binding.spdy_dp_workspace_bytes, binding.spdy_dp_workspace_bytes_min):
        assert f(0, 1, 1, 1) == 0
        assert f(1, 1, 1, -1) == 0
        assert f(1, 1, 256, 1) == 0
        assert f(1, 1, 255, 1) > 0
        assert f(2 ** 31 - 1, 2 ** 31 - 1, 255, 2 ** 31 - 2000) == 0


# (a header of one word more would take 256 bytes more at 15 and 31 layers: buffers of a fixed size would be refused)
@pytest.mark.parametrize("L, sizes", [(15, (1820928, 464640, 856320)), (31, (3762176, 958976, 1350656))])
def test_workspace_size_stays(binding, L, sizes):
    shape = (3, L, 40, 10000)
    assert sizes == (binding.spdy_dp_workspace_bytes(*shape), binding.spdy_dp_workspace_bytes_min(*shape),
                     binding.spdy_dp_workspace_bytes_checkpointed(*shape))


def test_argument_errors_are_reported_before_any_launch(binding):
    lib = binding.lib()
    fake = 0x1000  # never dereferenced: every call below must fail validation first
    solve = lib.spdy_dp_solve_batched
    assert solve(None, fake, 1, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert solve(fake, None, 1, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert solve(fake, fake, 1, 1, 1, 1, None, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert solve(fake, fake, 1, 1, 1, 1, fake, None, fake, 1 << 20, None) == binding.ERR_NULL
    assert solve(fake, fake, 1, 1, 1, 1, fake, fake, None, 1 << 20, None) == binding.ERR_NULL
    assert solve(fake, fake, 0, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert solve(fake, fake, 1, 0, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert solve(fake, fake, 1, 1, 0, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert solve(fake, fake, 1, 1, 1, -1, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert solve(fake, fake, 1, 1, 256, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_LEVELS
    assert solve(fake, fake, 1, 1, 1, 1, fake, fake, fake, 8, None) == binding.ERR_WORKSPACE
    assert solve(fake, fake, 2 ** 31 - 1, 2 ** 31 - 1, 2, 2 ** 31 - 2000, fake, fake, fake,
                 1 << 20, None) == binding.ERR_OVERFLOW
    # the entry point with the built-in workspace: sizes are checked before the device is touched
    static = lib.spdy_dp_solve_batched_static
    assert static(None, fake, 1, 1, 1, 1, fake, fake, None) == binding.ERR_NULL
    assert static(fake, None, 1, 1, 1, 1, fake, fake, None) == binding.ERR_NULL
    assert static(fake, fake, 1, 1, 1, 1, None, fake, None) == binding.ERR_NULL
    assert static(fake, fake, 1, 1, 1, 1, fake, None, None) == binding.ERR_NULL
    assert static(fake, fake, 0, 1, 1, 1, fake, fake, None) == binding.ERR_DIM
    assert static(fake, fake, 1, 1, 300, 1, fake, fake, None) == binding.ERR_LEVELS
    assert binding.spdy_dp_workspace_bytes_min(123, 54, 40, 10000) <= \
        binding.STATIC_WORKSPACE_BYTES < binding.spdy_dp_workspace_bytes_min(124, 54, 40, 10000)
    assert static(fake, fake, 124, 54, 40, 10000, fake, fake, None) == binding.ERR_STATIC_LIMIT
    assert static(fake, fake, 1024, 54, 40, 10000, fake, fake, None) == binding.ERR_STATIC_LIMIT
    assert static(fake, fake, 2 ** 31 - 1, 2 ** 31 - 1, 2, 2 ** 31 - 2000, fake, fake, None) == \
        binding.ERR_OVERFLOW
    one = (ctypes.c_int32 * 2)(5, 9)
    neg = (ctypes.c_int32 * 2)(5, -1)
    multi = lib.spdy_dp_solve_budgets
    assert multi(fake, fake, 1, 1, 1, None, 2, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert multi(fake, fake, 1, 1, 1, one, 0, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert multi(fake, fake, 1, 1, 1, neg, 2, fake, fake, fake, 1 << 20, None) == binding.ERR_DIM
    assert multi(fake, fake, 1, 1, 1, one, 2, fake, fake, fake, 8, None) == binding.ERR_WORKSPACE
    sens = lib.spdy_dp_solve_sensitivities
    assert sens(fake, None, fake, 1, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert sens(fake, fake, None, 1, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert sens(fake, fake, fake, 1, 1, 300, 1, fake, fake, fake, 1 << 20, None) == \
        binding.ERR_LEVELS
    inc = lib.spdy_dp_solve_from_incumbent
    big = 1 << 20
    far = 0x40000000
    assert inc(fake, fake, None, 1, 1, 1, 1, far, big, fake, fake, fake, big, None) == \
        binding.ERR_NULL
    assert inc(fake, None, fake, 1, 1, 1, 1, far, big, fake, fake, fake, big, None) == \
        binding.ERR_NULL
    assert inc(fake, fake, fake, 1, 1, 1, 1, None, big, fake, fake, fake, big, None) == \
        binding.ERR_NULL
    assert inc(fake, fake, fake, 1, 0, 1, 1, far, big, fake, fake, fake, big, None) == \
        binding.ERR_DIM
    assert inc(fake, fake, fake, 1, 1, 1, 1, far, 8, fake, fake, fake, big, None) == \
        binding.ERR_WORKSPACE
    assert inc(fake, fake, fake, 1, 1, 1, 1, far, big, fake, fake, fake, 8, None) == \
        binding.ERR_WORKSPACE
    # overlapping workspaces: the fill would overwrite the rows it resumes from
    assert inc(fake, fake, fake, 1, 1, 1, 1, fake + 64, big, fake, fake, fake, big, None) == \
        binding.ERR_WORKSPACE
    # a level-record workspace keeps no rows of D to resume from
    small = binding.lib().spdy_dp_workspace_bytes_min(4, 8, 8, 1000)
    assert small < binding.lib().spdy_dp_workspace_bytes(4, 8, 8, 1000)
    assert inc(fake, fake, fake, 4, 8, 8, 1000, far, big, fake, fake, fake, small, None) == \
        binding.ERR_WORKSPACE
    ck = lib.spdy_dp_solve_checkpointed
    assert ck(fake, None, 1, 1, 1, 1, 0, fake, fake, fake, big, None) == binding.ERR_NULL
    assert ck(None, fake, 1, 1, 1, 1, 0, fake, fake, fake, big, None) == binding.ERR_NULL
    assert ck(fake, fake, 1, 1, 1, 1, 0, None, fake, fake, big, None) == binding.ERR_NULL
    assert ck(fake, fake, 1, 0, 1, 1, 0, fake, fake, fake, big, None) == binding.ERR_DIM
    assert ck(fake, fake, 1, 1, 300, 1, 0, fake, fake, fake, big, None) == binding.ERR_LEVELS
    assert ck(fake, fake, 1, 1, 1, 1, 0, fake, fake, fake, 8, None) == binding.ERR_WORKSPACE
    # the workspace of one stride does not serve a stride that needs more rows
    need4 = binding.spdy_dp_workspace_bytes_checkpointed(8, 64, 8, 4000, 4)
    need8 = binding.spdy_dp_workspace_bytes_checkpointed(8, 64, 8, 4000, 8)
    assert need8 < need4 < binding.spdy_dp_workspace_bytes(8, 64, 8, 4000)
    assert ck(fake, fake, 8, 64, 8, 4000, 4, fake, fake, fake, need8, None) == \
        binding.ERR_WORKSPACE
    assert lib.spdy_dp_fill(fake, fake, 1, 1, 1, 1, None, fake, 1 << 20, None) == binding.ERR_NULL
    bt = lib.spdy_dp_backtrace
    assert bt(fake, fake, 1, 1, 1, 1, None, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert bt(fake, None, 1, 1, 1, 1, fake, fake, fake, 1 << 20, None) == binding.ERR_NULL
    assert bt(fake, fake, 1, 1, 1, 1, fake, None, fake, 1 << 20, None) == binding.ERR_NULL
    assert bt(fake, fake, 1, 1, 1, 1, fake, fake, fake, 8, None) == binding.ERR_WORKSPACE


def test_binding_refuses_cpu_tensors(binding):
    import torch
    tau = torch.zeros((2, 2), dtype=torch.int32)
    err = torch.zeros((1, 2, 2), dtype=torch.float32)
    with pytest.raises(TypeError):
        binding.spdy_dp_solve_batched(tau, err, 4)


def test_every_declared_function_can_be_called_from_python(binding):
    import paper_2201_13096_amd as m
    for name in declared_functions():
        assert callable(getattr(m, name)), name


def test_executed_update_counts_bracket_the_necessary_work():
    """The roofline's numerator is the update count bench.py derives from tau.  It must cover every
    update Alg. 1 needs (a finite D_{l-1}[t - tau] that can still end within the budget) and may
    not exceed Alg. 1's own loop trips; folding levels of equal time can only lower it."""
    import numpy as np
    import bench
    import oracle
    import workloads
    rng = np.random.default_rng(5)
    for case in range(12):
        L = int(rng.integers(1, 7))
        S = int(rng.integers(1, 9))
        B = int(rng.choice([0, 9, 40, 150]))
        tau, err, _ = workloads.random_instance(rng, 2, L, S, B, tau_max=max(1, B // 2),
                                                zero_tau_frac=0.2, integer_err=3,
                                                layer_floor=int(rng.choice([0, 3])))
        D, _, _, _ = oracle.tables_ref(tau, err[0], B)
        t = tau.astype(np.int64)
        mn = t.min(axis=1)
        rest = np.concatenate([np.cumsum(mn[::-1])[::-1][1:], [0]])   # least time still to come
        needed = 0
        for l in range(L):
            prev = D[l - 1] if l > 0 else np.r_[0.0, np.full(B, np.inf)]
            for s in range(S):
                for u in range(B + 1):
                    tt = u + t[l, s]
                    if np.isfinite(prev[u]) and tt + rest[l] <= B:
                        needed += 1
        nominal = sum(max(0, B + 1 - int(t[l, s])) for l in range(L) for s in range(S))
        plain = bench.executed_updates_per_candidate(tau, B, False)
        folded = bench.executed_updates_per_candidate(tau, B, True)
        skipped = bench.executed_updates_level_record(tau, err, B)
        assert folded <= plain <= nominal, (case, folded, plain, nominal)
        assert 2 * folded <= skipped <= 2 * plain, (case, folded, skipped, plain)
        # every needed update is executed; with equal times folded, one update serves all levels
        # of a time, so compare per distinct time
        needed_folded = 0
        for l in range(L):
            prev = D[l - 1] if l > 0 else np.r_[0.0, np.full(B, np.inf)]
            for d in sorted(set(int(x) for x in t[l])):
                for u in range(B + 1):
                    if np.isfinite(prev[u]) and u + d + rest[l] <= B:
                        needed_folded += 1
        assert needed <= plain, (case, needed, plain)
        assert needed_folded <= folded, (case, needed_folded, folded)


def test_traffic_table_only_counts_for_the_source_it_was_taken_on(tmp_path, monkeypatch):
    """bench.py reports HBM traffic from a tracked table of counter runs; a line must only count
    for its workload and record and while the kernel source is the one the counters saw."""
    import bench
    table = tmp_path / "dp_fill_hbm_traffic.txt"
    here = bench.kernel_source_id()
    assert len(here) == 12 and int(here, 16) >= 0
    table.write_text("# comment\n"
                     f"rn50_k1024 d {here} 1000 2000\n"
                     f"rn50_k1024 level {'0' * 12} 5 6\n"
                     "short line\n")
    monkeypatch.setattr(bench, "PROFILES", str(tmp_path))
    assert bench.tracked_traffic("rn50_k1024", "d") == 3000.0
    assert bench.tracked_traffic("rn50_k1024", "level") is None      # another source
    assert bench.tracked_traffic("bert_k4096", "d") is None          # no line
    monkeypatch.setattr(bench, "PROFILES", str(tmp_path / "missing"))
    assert bench.tracked_traffic("rn50_k1024", "d") is None


def test_source_id_covers_every_kernel_source(tmp_path, monkeypatch):
    """A change in any file that the fill's launches are compiled from makes old counters stale."""
    import bench
    csrc = os.path.join(ROOT, "paper_2201_13096_amd", "csrc")
    text = open(os.path.join(csrc, "spdy_dp.hip")).read()
    included = re.findall(r'#include "(\w+\.h)"', text)
    own = {"spdy_dp.hip"} | {f for f in included if os.path.exists(os.path.join(csrc, f))}
    assert {os.path.basename(p) for p in bench.KERNEL_SOURCES} == own
    copies = []
    for p in bench.KERNEL_SOURCES:
        copies.append(str(tmp_path / os.path.basename(p)))
        with open(p, "rb") as src, open(copies[-1], "wb") as dst:
            dst.write(src.read())
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    ids = {bench.kernel_source_id()}
    for p in copies:
        with open(p, "ab") as f:
            f.write(b"// changed\n")
        ids.add(bench.kernel_source_id())
    assert len(ids) == 1 + len(copies)


# the kernel and the width of its reads by header word 19, not by the sizes: rows that are folded or not, rows beyond them
@pytest.mark.parametrize("word, record, S, kernel, wide, loop", [
    (0, "d", 64, "dp_fill", True, "sweep_b128"), (0, "d", 65, "dp_fill", False, "sweep_b32"),
    (-4, "d", 65, "dp_columns", True, "sweep_folded"), (-1, "d", 65, "dp_columns", False, "sweep_b32"),
    (-4, "level", 40, "dp_columns", True, "sweep_folded_levels"), (-1, "level", 40, "dp_columns", False, "sweep_b32"),
    (0, "level", 40, "dp_fill", False, "sweep_b32"), (3 | 1 << 11, "d", 40, "dp_tiles", True, "sweep_b128")])
def test_bench_names_what_did_the_fill(word, record, S, kernel, wide, loop):
    import bench
    assert bench.fill_launch([0] * 19 + [word], record, S) == (kernel, wide)
    assert bench.bare_sweep(kernel, wide, record) == loop


def test_rate_probe_output_is_optional(monkeypatch, tmp_path):
    import bench
    monkeypatch.setattr(bench, "PROBE", str(tmp_path / "no_such_probe"))
    assert bench.measured_peaks() is None


def test_no_kernel_needs_scratch_memory(binding):
    """A kernel with a private segment makes the runtime provide scratch memory at its first launch, and
    the library promises that nothing is allocated.  (What the compiler noted down for each kernel of
    this library, in the metadata of its own code object.)"""
    noted = re.findall(rb"\.name(?:\xd9.|\xda..)(_Z\w+)\xbb\.private_segment_fixed_size(.)",
                       open(binding.LIB_PATH, "rb").read(), flags=re.S)
    kernels = {name.decode(): size for name, size in noted}
    assert {"dp_fill", "dp_tiles", "dp_core", "dp_rest", "dp_prepare"} <= \
        {m.group() for m in (re.search(r"dp_[a-z]+", n) for n in kernels) if m}
    assert [n for n, size in kernels.items() if size != b"\0"] == []
