"""Errors that the kernels of a round raise reach the caller, also those of the DelaunayBall kernel,
which runs behind its round's snapshot of the counters: after the last round of a call, beside
a full pool, and where a limit of rounds ends the call.  The bits are raised around a round by
a hook of the library (dt_test_raise), no kernel fails."""
import ctypes

import numpy as np
import pytest

from synth import uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

ERR_WALK, ERR_POOL = 1, 16  # csrc/dt_internal.h


def raise_bits(dtlib, tri, before, behind):
    hook = dtlib.lib().dt_test_raise
    hook.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32]
    assert hook(tri.ctx, before, behind) == dtlib.DT_OK


def expect_internal(dtlib, tri, xyz):
    with pytest.raises(dtlib.DTError) as e:
        tri.insert(xyz)
    assert e.value.code == dtlib.DT_E_INTERNAL


OPTS = [{}, dict(graph_rounds=True), dict(index_bits=64)]


@pytest.mark.parametrize("opts", OPTS)
@pytest.mark.parametrize("before,points", [(0, 1), (ERR_POOL, 100)])
def test_errors_of_the_balls_are_reported(dtlib, oracle_mod, before, points, opts):
    say(f"error behind a round's snapshot, {points} points, {opts}")
    xyz = uniform_points(1000 + points, 931)
    with dtlib.Triangulation(**opts) as tri:
        tri.insert(xyz[:1000])
        raise_bits(dtlib, tri, before, ERR_WALK)
        expect_internal(dtlib, tri, xyz[1000:])
        tri.clear()  # the context can be used again
        tri.insert(xyz)
        t, _ = tri.tets()
        assert_parity(oracle_mod, xyz, t.astype(np.int64), "after the error")


@pytest.mark.parametrize("opts", OPTS)
def test_a_full_pool_alone_is_no_error(dtlib, oracle_mod, opts):
    say(f"full pool, {opts}")
    xyz = uniform_points(1300, 933)
    with dtlib.Triangulation(**opts) as tri:
        tri.insert(xyz[:1000])
        raise_bits(dtlib, tri, ERR_POOL, 0)
        tri.insert(xyz[1000:])
        t, _ = tri.tets()
        assert_parity(oracle_mod, xyz, t.astype(np.int64), "after a full pool")


def test_errors_beside_a_limit_of_rounds(dtlib):
    say("errors of the last round before the limit")
    xyz = uniform_points(400, 932)
    with dtlib.Triangulation(max_rounds=1) as tri:
        tri.insert(xyz[:5])
        raise_bits(dtlib, tri, 0, ERR_WALK)
        expect_internal(dtlib, tri, xyz[5:])


@pytest.mark.parametrize("points", [5, 300, 2000])
def test_errors_before_the_first_round(dtlib, points):
    """As the first insertions (csrc/dt_seed.hip) raise them, ahead of every round."""
    say(f"error ahead of the first round, {points} points")
    with dtlib.Triangulation() as tri:
        raise_bits(dtlib, tri, ERR_WALK, 0)
        expect_internal(dtlib, tri, uniform_points(points, 934))
