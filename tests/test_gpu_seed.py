"""The first insertions in one block's LDS (csrc/dt_seed.hip), at the sizes and inputs where they
can go wrong: around the block's vertex limit, clouds whose tetrahedra outgrow its LDS (points
of the moment curve have O(n^2) of them), signs its filter cannot decide, duplicates, a pool
without room, 64-bit codes, the sub-determinant cache, clouds of a batch.  Exact equality with
the oracle throughout."""
import numpy as np
import pytest

from synth import lattice_points, shell_points, uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)
from validators import check_invariants

pytestmark = pytest.mark.gpu


def moment_curve(n, seed):
    t = np.sort(uniform_points(n, seed)[:, 0]) + 0.05
    return np.random.default_rng(seed).permutation(np.c_[t, t * t, t ** 3])


@pytest.mark.parametrize("case,opts", [
    (("uniform", 5), {}), (("uniform", 31), {}), (("uniform", 575), {}), (("uniform", 576), {}),
    (("uniform", 577), {}), (("uniform", 2100), {}), (("uniform", 800), dict(index_bits=64)),
    (("uniform", 900), dict(subdet_cache=True)), (("uniform", 3000), dict(capacity_tets=4096)),
    (("uniform", 1500), dict(seed=7, adaptive_curve=True)), (("moment", 300), {}), (("shell", 1200), {}),
    (("lattice", 700), {}), (("duplicates", 900), {})])
def test_seeded_mesh_matches_oracle(dtlib, oracle_mod, case, opts):
    kind, n = case
    say(f"seed {kind} {n} {opts}")
    xyz = {"uniform": lambda: uniform_points(n, 611 + n), "moment": lambda: moment_curve(n, 3),
           "shell": lambda: shell_points(n, 5), "lattice": lambda: lattice_points(n, 6, side=9),
           "duplicates": lambda: uniform_points(n // 3, 8)[np.random.default_rng(4).integers(0, n // 3, n)]}[kind]()
    xyz = np.ascontiguousarray(xyz)
    with dtlib.Triangulation(**opts) as tri:
        tri.insert(xyz)
        t, nb = tri.tets()
        st = tri.stats()
        assert_parity(oracle_mod, xyz, t.astype(np.int64), f"{kind} {n}")
        distinct = len(np.unique(xyz, axis=0))
        assert st["vertices"] == distinct and st["inserted"] == distinct - 4
        expect = np.sort(np.unique(xyz, axis=0, return_index=True)[1])
        check_invariants(xyz, t.astype(np.int64), nb, oracle_mod, expect_vertices=expect)
        tri.clear()
        tri.insert(xyz[::-1].copy())  # the context's second mesh, on used slots
        t, _ = tri.tets()
        assert_parity(oracle_mod, xyz[::-1], t.astype(np.int64), f"{kind} {n} again")


def test_seeded_clouds_of_a_batch(dtlib, oracle_mod):
    say("seed: batch of clouds below, at and above the block's limit")
    clouds = [uniform_points(n, 700 + n) + n for n in (4, 5, 40, 576, 577, 2500)] + [moment_curve(200, 9)]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])]).astype(np.uint64)
    with dtlib.Triangulation() as tri:
        tri.insert_batch(np.ascontiguousarray(np.vstack(clouds)), off)
        for k, c in enumerate(clouds):
            t, nb = tri.tets_batch(k)
            assert_parity(oracle_mod, c, t.astype(np.int64), f"cloud {k}")
            check_invariants(c, t.astype(np.int64), nb, oracle_mod, expect_vertices=np.arange(len(c)))


@pytest.mark.parametrize("clouds,points", [(64, 6), (65, 15), (65, 16), (1024, 18), (1025, 18)])
def test_batches_around_the_limits(dtlib, oracle_mod, clouds, points):
    """Both sides of the rule on the number of clouds and their mean size."""
    say(f"seed: {clouds} clouds of {points} points")
    xyz = uniform_points(clouds * points, 47 + clouds + points)
    off = np.arange(clouds + 1, dtype=np.uint64) * points
    with dtlib.Triangulation() as tri:
        tri.insert_batch(xyz, off)
        for k in sorted({0, 1, clouds // 2, clouds - 1}):
            c = xyz[k * points:(k + 1) * points]
            t, nb = tri.tets_batch(k)
            assert_parity(oracle_mod, c, t.astype(np.int64), f"cloud {k} of {clouds}")
            check_invariants(c, t.astype(np.int64), nb, oracle_mod, expect_vertices=np.arange(points))
