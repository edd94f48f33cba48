"""The cavity kernel's set holds as many tetrahedra with 64-bit adjacency codes as with 32-bit
ones: uniform points, whose insertions touch about 47 tetrahedra and up to a hundred and more,
do not overflow it more often."""
import pytest

from synth import uniform_points
from test_gpu import assert_parity, dtlib, gpu_dt, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes", [0, 16, 64])
def test_wide_set_does_not_overflow(dtlib, oracle_mod, lanes):
    say(f"64-bit codes, {lanes} lanes: overflows")
    xyz = uniform_points(60000, 71)
    tets, _, st = gpu_dt(dtlib, xyz, index_bits=64, lanes_per_insert=lanes)
    assert_parity(oracle_mod, xyz, tets, "wide set")
    _, _, narrow = gpu_dt(dtlib, xyz, index_bits=32, lanes_per_insert=lanes)
    assert st["overflows"] <= narrow["overflows"] + 20
