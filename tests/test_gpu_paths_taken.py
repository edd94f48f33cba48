"""That the paths which leave the result as it is are taken, seen by the rounds and the walk steps of
a call, and the places where one path hands over to another."""
import numpy as np
import pytest

from synth import shell_points, uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)
from validators import check_invariants

pytestmark = pytest.mark.gpu


def mesh(dtlib, oracle_mod, clouds, **opts):
    """Statistics of one call over the clouds, each compared with the oracle."""
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])]).astype(np.uint64)
    with dtlib.Triangulation(**opts) as tri:
        if len(clouds) == 1:
            tri.insert(clouds[0])
            assert_parity(oracle_mod, clouds[0], tri.tets()[0].astype(np.int64), f"{opts}")
        else:
            tri.insert_batch(np.vstack(clouds), off)
            for k, c in enumerate(clouds):
                assert_parity(oracle_mod, c, tri.tets_batch(k)[0].astype(np.int64), f"cloud {k} {opts}")
        return tri.stats()


# Without the first insertions in one block, a mesh of v vertices gains at most a third of them in a
# round (winners' cavities are disjoint, an insertion takes about 20 of the 6.7 v tetrahedra): 17
# rounds from 4 to 576 vertices, 15 to 340.  With them the 1024 ranks of up to 1024 points pass in
# windows of at least 128: 8 rounds, and a few for points that the block left out.
SEEDED = 12


@pytest.mark.parametrize("opts,seeded", [
    ({}, True), (dict(index_bits=64), True), (dict(timing=2), True), (dict(timing=1), False),
    (dict(round_size=4096), False), (dict(max_rounds=100000), False)])
def test_first_insertions_run(dtlib, oracle_mod, opts, seeded):
    say(f"first insertions: {opts}")
    st = mesh(dtlib, oracle_mod, [uniform_points(576, 951)], **opts)
    assert (st["rounds"] <= SEEDED) if seeded else (st["rounds"] >= 17), st["rounds"]


def test_first_insertions_without_room(dtlib, oracle_mod):
    """Three clouds of 340 points (2,200 tetrahedra each) and a pool of 4096 slots: two clouds keep
    their initial tetrahedron and go through the rounds."""
    say("first insertions: no room in the pool")
    clouds = [uniform_points(340, 952 + k) for k in range(3)]
    assert mesh(dtlib, oracle_mod, clouds)["rounds"] <= SEEDED
    assert mesh(dtlib, oracle_mod, clouds, capacity_tets=4096)["rounds"] >= 15


@pytest.mark.parametrize("parts", [[20000] + [2500] * 4, [3000] * 6])
def test_appended_walks_start_near(dtlib, oracle_mod, parts):
    """Walks of appended calls start at the nearest of four records around the point's place on the
    curve: a few tetrahedra away, whatever the mesh's size (6.7 steps a point measured at 300,007
    points in 6 calls, 77 from the call's own records)."""
    say(f"append: walk steps, {parts}")
    xyz = uniform_points(sum(parts), 955)
    cuts = np.cumsum(parts)
    with dtlib.Triangulation() as tri:
        tri.insert(xyz[:cuts[0]])
        first = tri.stats()["walk_steps"]
        for lo, hi in zip(cuts[:-1], cuts[1:]):
            tri.insert(xyz[lo:hi])
        steps = (tri.stats()["walk_steps"] - first) / (cuts[-1] - cuts[0])
        assert_parity(oracle_mod, xyz, tri.tets()[0].astype(np.int64), f"append {parts}")
    say(f"append: {steps:.2f} walk steps a point")
    assert steps < 20


@pytest.mark.parametrize("rounds", [(1 << 16) - 7, (5 << 16) - 7, (1 << 31) - 7])
def test_round_counter_wraps(dtlib, oracle_mod, rounds):
    """Claim stamps hold 16 bits of the round counter, the marks of lost attempts 31: across the
    wrap of the stamps alone, and of both."""
    say(f"round counter wrap at {rounds + 7}")
    xyz = uniform_points(30000, 957)
    with dtlib.Triangulation() as tri:
        tri.insert(uniform_points(3000, 956))  # claims left in the pool by earlier rounds
        tri.clear()
        dtlib.dt_debug_set_round_counter(tri.ctx, rounds)
        tri.insert(xyz)
        assert tri.stats()["rounds"] > 7
        assert_parity(oracle_mod, xyz, tri.tets()[0].astype(np.int64), f"across {rounds + 7}")


@pytest.mark.parametrize("n", [60, 70, 80, 90, 100, 107, 108, 109, 110])
@pytest.mark.parametrize("opts", [{}, dict(lanes_per_insert=16), dict(index_bits=64)])
def test_hand_over_to_the_rounds_for_large_cavities(dtlib, oracle_mod, n, opts):
    """Balls around the limits of the regular rounds: 128 cavity tetrahedra, 213 boundary facets, 256
    tetrahedra of both (points near a sphere and its centre: 2 n - 4 facets)."""
    say(f"hand-over: ball of {2 * n - 4} facets, {opts}")
    sphere, centre = shell_points(n, 60 + n), 0.02 * (uniform_points(2, n) - 0.5)
    xyz = np.vstack([sphere, centre])
    with dtlib.Triangulation(**opts) as tri:
        tri.insert(sphere)
        tri.insert(centre[:1])
        tri.insert(centre[1:])
        t, nb = tri.tets()
    assert_parity(oracle_mod, xyz, t.astype(np.int64), f"{n} {opts}")
    check_invariants(xyz, t.astype(np.int64), nb, oracle_mod, expect_vertices=np.arange(len(xyz)))


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_appended_walks_on_spread_scales(dtlib, oracle_mod, seed):
    """Points whose scales spread over 2^160: one cell of the first call's grid holds nearly all of
    its records, and those around a point's place are no start for its walk.  Exact orientations,
    most of the calls' time: 48,000 to 77,000 from the calls' own records, 139,000 to 431,000 from
    there."""
    say(f"append: spread scales, {seed}")
    rng = np.random.default_rng(seed)
    parts = [(rng.random((n, 3)) - 0.5) * 2.0 ** rng.integers(-60, 100, (n, 1)) for n in (1000, 500, 500, 500)]
    with dtlib.Triangulation() as tri:
        for p in parts:
            tri.insert(p)
        exact = tri.stats()["orient_exact"]
        assert_parity(oracle_mod, np.vstack(parts), tri.tets()[0].astype(np.int64), f"spread scales {seed}")
    say(f"append: {exact} exact orientations")
    assert exact < 110_000


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_appended_walks_beyond_the_grid(dtlib, oracle_mod, seed):
    """Points far beyond the earlier call's grid: records of its border, here nearly all on one line,
    are no start for them where a curve neighbour is inserted.  Exact orientations: 134,000 to
    151,000 with walks that start at the neighbour, 187,000 to 218,000 with walks from the border."""
    say(f"append: beyond the grid, {seed}")
    rng = np.random.default_rng(seed)
    line = np.outer(rng.random(1300), [1.0, 2.0, 3.0])
    line[:130] = rng.random((130, 3))
    parts = [line] + [(rng.random((n, 3)) - 0.5) * 2.0 ** rng.integers(-60, 100, (n, 1)) for n in (100, 900)]
    with dtlib.Triangulation() as tri:
        for p in parts:
            tri.insert(p)
        exact = tri.stats()["orient_exact"]
        assert_parity(oracle_mod, np.vstack(parts), tri.tets()[0].astype(np.int64), f"beyond the grid {seed}")
    say(f"append: beyond the grid: {exact} exact orientations")
    assert exact < 170_000
