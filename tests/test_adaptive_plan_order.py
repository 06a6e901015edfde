"""The host plan's orders against the oracle's, where its digit passes could differ from a comparison sort:
counts and lengths over all digits, many equal keys, signed zeros and infinities, none, one and all candidates."""
import numpy as np
import pytest

from oracle import adaptive as OA
from paper_2603_27151_amd import raster as R


@pytest.mark.parametrize("T", [0, 1, 2, 700, 4099])
@pytest.mark.parametrize("spread", ["wide", "ties", "special"])
@pytest.mark.parametrize("prune,fill", [(False, False), (True, True), (False, True)])
def test_plan_orders(T, spread, prune, fill):
    rng = np.random.default_rng(T + 7)
    if spread == "wide":
        counts = rng.integers(0, 2 ** 32, T, dtype=np.uint64).astype(np.uint32) >> rng.integers(0, 32, T).astype(np.uint32)
        rel = np.exp(rng.normal(-2, 3, (T, 3))).astype(np.float32)
    else:
        counts = rng.integers(0, 3, T).astype(np.uint32)
        rel = rng.integers(0, 4, (T, 3)).astype(np.float32) / np.float32(8)
    if spread == "special" and T:
        rel[rng.integers(0, T, T // 5)] = np.float32(np.inf)
        rel[rng.integers(0, T, T // 5)] = np.float32(-0.0)
    for target in {0, T // 3, T, T + T // 4, 3 * T}:
        got = R.adaptive_plan(counts, rel, 0.2, target, prune, fill)
        want = OA.plan(counts, rel, 0.2, target, prune, fill)
        assert got[2] == want[2] and np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
