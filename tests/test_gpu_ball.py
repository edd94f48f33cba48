"""Balls on both sides of the edge tables' limits (64, 256 and 2048 facets): points near a sphere,
then points near its centre, whose balls have about two facets per point of the sphere.  Exact
equality with the oracle."""
import numpy as np
import pytest

from synth import shell_points, uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)
from validators import check_invariants

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 34, 36, 129, 130, 131, 400, 1025, 1026, 1030, 1500])
@pytest.mark.parametrize("opts", [{}, dict(lanes_per_insert=16), dict(large_lanes=64), dict(index_bits=64)])
def test_ball_sizes(dtlib, oracle_mod, n, opts):
    say(f"ball of {2 * n - 4} facets, {opts}")
    sphere, centre = shell_points(n, 40 + n), 0.02 * (uniform_points(3, n) - 0.5)
    xyz = np.vstack([sphere, centre])
    with dtlib.Triangulation(**opts) as tri:
        tri.insert(sphere)
        tri.insert(centre[:1])
        tri.insert(centre[1:])
        t, nb = tri.tets()
    assert_parity(oracle_mod, xyz, t.astype(np.int64), f"{n} {opts}")
    check_invariants(xyz, t.astype(np.int64), nb, oracle_mod, expect_vertices=np.arange(len(xyz)))
