"""Rows of one, two and three chunks in the reduced problem (csrc/dp_core.h): budgets around 64 and 128 buckets
under tables that hardly reduce, so that rows grow from one chunk to the next and shrink again, with one to
many levels a step, ties, and layers between the steps."""
import numpy as np
import pytest

from test_gpu_core import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


@pytest.mark.parametrize("slack", [20, 62, 63, 64, 65, 100, 126, 127, 128, 129, 150, 191, 193, 260])
@pytest.mark.parametrize("L, S, steps", [(85, 2, 40), (60, 3, 9), (40, 5, 6), (70, 4, 3)])
def test_rows_around_two_chunks(dp, L, S, steps, slack):
    rng = np.random.default_rng(1000 * L + slack)
    # times in `steps`; errors linear in them but for a little, so that all levels and most cells stay
    tau = rng.integers(0, steps + 1, size=(L, S)).astype(np.int32)
    tau[::5] = tau[::5, :1]                        # layers without a choice of time
    tau += 1
    slope = 1.0 + 1e-6 * rng.integers(-3, 4, size=(9, L, S))
    err = (slope * (steps + 1 - tau) / 64.0).astype(np.float32)
    err[::3] = np.float32(1.0) * (steps + 1 - tau)                  # everything ties
    B = int(tau.min(axis=1).sum()) + slack
    print(f"[rows] L={L} S={S} steps={steps} slack={slack}", flush=True)
    check(dp, tau, err, B, f"L={L} S={S} slack={slack}")


@pytest.mark.parametrize("noise", [1e-5, 1e-4, 1e-3, 1e-2])
def test_rows_that_grow_and_shrink(dp, noise):
    rng = np.random.default_rng(int(noise * 1e6))
    for L, S, B in ((60, 8, 500), (150, 6, 1500), (200, 30, 9000)):
        dense = rng.uniform(0.2, 3.0, L)
        p = np.arange(S) / (S - 1)
        tau = np.floor(dense[:, None] * (1.0 - 0.7 * p) * (2.0 * B / dense.sum()) + 0.5).astype(np.int32)
        curve = dense[:, None] * (p + 0.3 * p * p)
        err = (curve * (1.0 + noise * rng.standard_normal((9, L, S)))).clip(0).astype(np.float32)
        check(dp, tau, err, B, f"noise {noise} L={L}")
