"""Appended calls whose walks start among the vertices of earlier calls: calls of very different
sizes, points outside the earlier box, duplicates of earlier points, the adaptive curve, a
context used again after a clear.  Exact equality with the oracle on all points."""
import numpy as np
import pytest

from synth import shell_points, uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)
from validators import check_invariants

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [{}, dict(adaptive_curve=True), dict(index_bits=64), dict(cavity_cap=12)])
def test_appended_calls(dtlib, oracle_mod, opts):
    say(f"append {opts}")
    a = uniform_points(3000, 811)
    parts = [a[:2500], a[2500:2501], a[2501:],                   # inside, in calls of 2500, 1 and 499
             4.0 * uniform_points(1500, 812) - 1.5,              # around the earlier box
             np.vstack([a[100:140], uniform_points(60, 813)]),   # duplicates of earlier points
             10.0 + uniform_points(5, 814), shell_points(700, 815)]
    xyz = np.vstack(parts)
    keep = np.sort(np.unique(xyz, axis=0, return_index=True)[1])
    with dtlib.Triangulation(**opts) as tri:
        for _ in range(2):
            tri.clear()
            for p in parts:
                tri.insert(np.ascontiguousarray(p))
            t, nb = tri.tets()
            assert_parity(oracle_mod, xyz, t.astype(np.int64), f"append {opts}")
    check_invariants(xyz, t.astype(np.int64), nb, oracle_mod, expect_vertices=keep)


def test_many_small_calls(dtlib, oracle_mod):
    say("append: 90 calls")
    xyz = uniform_points(1200, 816)
    cuts = np.r_[0, 600, np.sort(np.random.default_rng(3).choice(np.arange(601, 1200), 88, replace=False)), 1200]
    with dtlib.Triangulation() as tri:
        for lo, hi in zip(cuts[:-1], cuts[1:]):
            tri.insert(xyz[lo:hi])
        t, _ = tri.tets()
        assert_parity(oracle_mod, xyz, t.astype(np.int64), "90 calls")


def test_refused_first_call(dtlib, oracle_mod):
    """A first call that is refused leaves no records for the calls after it to start from."""
    say("append: after a refused call")
    line = np.outer(np.arange(5000.0), [1.0, 2.0, -1.0])
    xyz = uniform_points(1300, 817)
    with dtlib.Triangulation() as tri:
        with pytest.raises(dtlib.DTError):
            tri.insert(line)
        tri.insert(xyz[:300])
        tri.insert(xyz[300:])
        t, _ = tri.tets()
    assert_parity(oracle_mod, xyz, t.astype(np.int64), "after a refused call")
