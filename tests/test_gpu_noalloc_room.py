"""The room of the entry point without allocation: points whose pool has to grow once and then
fills its static array to the last few hundred KiB.  Same tetrahedra as with allocation."""
import numpy as np
import pytest

from test_gpu import dtlib, say  # noqa: F401  (fixture)
from test_zz_no_alloc import _allocating

pytestmark = pytest.mark.gpu


def test_pool_grows_into_the_last_of_the_array(dtlib, oracle_mod):
    import torch
    n, m, rng = 44650, 800, np.random.default_rng(3)
    say(f"no-alloc: {n - m} uniform points and {m} of the moment curve")
    t = np.sort(rng.random(m)) + 0.05  # m^2 / 2 tetrahedra among themselves
    xyz = rng.permutation(np.vstack([rng.random((n - m, 3)), np.c_[t, t * t, t ** 3] + 3.0]))
    rows = 640_000
    d = torch.from_numpy(xyz).cuda()
    tets = torch.empty((rows, 4), dtype=torch.int32, device="cuda")
    nbrs = torch.empty((rows, 4), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    T = dtlib.dt_triangulate_noalloc(d, tets, nbrs, rows)
    assert T > 600_000
    got = oracle_mod.canonical(tets[:T].cpu().numpy().astype(np.int64))
    assert np.array_equal(got, _allocating(dtlib, oracle_mod, xyz))
