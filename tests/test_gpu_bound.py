"""The reduced problem's multiplier and known profile (csrc/dp_core.h) at the sizes where their mapping
changes: lanes per layer and blocks of 64 layers, levels of a lane that are no whole number of eight, lists of
exchanges that are empty, that need two registers a lane, and that do not fit."""
import numpy as np
import pytest

import oracle
from test_gpu_core import check, smooth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2201_13096_amd as m
    return m


@pytest.mark.parametrize("L", [2, 3, 8, 9, 16, 17, 32, 33, 63, 64, 65, 128, 129, 192, 193, 255, 256])
@pytest.mark.parametrize("S", [2, 4, 7, 9, 63, 65, 129, 255])
def test_lanes_and_blocks_of_layers(dp, L, S):
    if L * S > 13000:
        S = 13000 // L                            # the tables have to fit LDS
    rng = np.random.default_rng(300 * L + S)
    tau, err = smooth(rng, 3, L, S, 3000)
    check(dp, tau, err, 3000, "lanes and blocks")


# almost linear errors: the fewer the steps of the times, the more levels a known profile can afford
@pytest.mark.parametrize("B", [150, 700, 3000, 20000])
@pytest.mark.parametrize("bend", [0.0, 0.002, 0.05])
@pytest.mark.parametrize("L, S", [(5, 33), (40, 33), (140, 30)])
def test_lists_of_exchanges(dp, L, S, B, bend):
    rng = np.random.default_rng(int(1000 * bend) + B + L)
    p = np.arange(S) / (S - 1)
    dense = rng.uniform(0.5, 2.0, L)
    tau = np.floor(dense[:, None] * (1.0 - 0.8 * p) * (2.0 * B / dense.sum()) + 0.5).astype(np.int32)
    slope = dense[:, None] * (1.0 + bend * rng.standard_normal((7, L, 1)))
    err = (slope * (p + bend * p * p) + 1e-4 * bend * rng.random((7, L, S))).astype(np.float32)
    check(dp, tau, err, B, f"bend {bend}")


def test_steps_as_large_as_the_room(dp):
    """Few, large steps: the best pair of exchanges is far better than one, and a third would be needed."""
    rng = np.random.default_rng(11)
    for B in (60, 300, 1500):
        L, S = 30, 6
        tau = np.sort(rng.integers(1, 2 + B // 8, size=(L, S)), axis=1)[:, ::-1].astype(np.int32).copy()
        tau[:, -1] = 1
        err = np.sort(rng.random((24, L, S), dtype=np.float32), axis=2)
        check(dp, tau, err, B, "large steps")
