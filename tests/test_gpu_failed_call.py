"""A call that fails among its rounds leaves candidates in the lists; insertions are refused until
the context is cleared, and then work as in a new one."""
import numpy as np
import pytest

from synth import lattice_points, uniform_points
from test_gpu import assert_parity, dtlib, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def expect(dtlib, code, call, *args):
    with pytest.raises(dtlib.DTError) as e:
        call(*args)
    assert e.value.code == code


@pytest.mark.parametrize("case", ["rounds", "cavity"])
def test_insertions_after_a_failed_call_are_refused(dtlib, oracle_mod, case):
    say(f"after a failed call: {case}")
    if case == "rounds":  # the limit of rounds ends the call
        opts, xyz, code = dict(max_rounds=2), uniform_points(400, 961), dtlib.DT_E_INCOMPLETE
    else:  # a centre in a cospherical shell: a cavity beyond the whole buffer
        opts, code = dict(cavity_cap=1, round_size=1), dtlib.DT_E_CAPACITY
        xyz = np.vstack([lattice_points(27, 3, side=3), [[1.0 / 64, 1.0 / 128, 1.0 / 256]]])
    small = uniform_points(4, 962)
    with dtlib.Triangulation(**opts) as tri:
        expect(dtlib, code, tri.insert, xyz)
        for again in (small, uniform_points(700, 963)):
            expect(dtlib, dtlib.DT_E_ARG, tri.insert, again)
        expect(dtlib, dtlib.DT_E_ARG, tri.insert_batch, small, np.array([0, 4], np.uint64))
        assert tri.stats()["points"] == len(xyz)
        tri.clear()
        tri.insert(small)
        t, _ = tri.tets()
        assert_parity(oracle_mod, small, t.astype(np.int64), "after the clear")
