"""Attempts of the exact pass that have lost stop before their next tests.  Points appended to a
tetrahedron whose vertices lie 1e-18 to 1e21 from the origin: the filter decides no insphere sign
of it, nearly every attempt loses, and its exact tests are nearly all of the call's time."""
import numpy as np
import pytest

from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [971, 972, 973])
def test_losers_make_no_further_exact_tests(dtlib, oracle_mod, seed):
    say(f"exact pass: tests of attempts that lose, {seed}")
    frame = np.array([[-1e-18, 1e-18, 1e-18], [-2e-8, -2e-8, 1e-8], [7e20, 3e20, -8e20], [2e13, -2e13, 4e12]])
    points = np.random.default_rng(seed).random((150, 3))
    with dtlib.Triangulation() as tri:
        tri.insert(frame)
        tri.insert(points)
        st = tri.stats()
        assert_parity(oracle_mod, np.vstack([frame, points]), tri.tets()[0].astype(np.int64), "exact pass")
    say(f"{st['attempts']} attempts, {st['conflicts']} conflicts, {st['insphere_exact']} exact insphere tests")
    # 0.6 to 0.8 tests an attempt where a loser stops before its next step, 1.5 to 1.9 where it
    # makes that step's tests first
    assert st["conflicts"] > 0.9 * st["attempts"] and st["insphere_exact"] < 1.1 * st["attempts"]
