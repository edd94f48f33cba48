"""The winner rule of the insertion rounds by marks, checked on the CPU with the oracle's exact
predicates (no GPU code involved).

Attempts claim the tetrahedra of their cavities (stamp 2 r) and around them (2 r + 1) in any
interleaving; a claim word keeps the lowest.  A claim that finds a lower one it cannot share
loses its attempt, which may stop there; a claim that displaces a later attempt's cavity claim
marks that attempt.  The attempts that complete unmarked win.  Whatever the interleaving, the
winners' cavities must be disjoint and apart from each other's outer tetrahedra, and the first
attempt must win."""
import numpy as np
import pytest

from synth import lattice_points, uniform_points
from test_claim_protocol import _cavities


def _attempts(oracle_mod, case):
    if case == "uniform":
        xyz, n0 = uniform_points(1300, 931), 1000
        new = [i for i in range(n0, 1300) if np.all((xyz[i] > 0.15) & (xyz[i] < 0.85))]
    else:  # cospherical: large cavities that share many tetrahedra
        xyz, n0 = lattice_points(343, 17, side=7), 250
        lim = np.abs(xyz).max() * 0.8
        new = [i for i in range(n0, 343) if np.all(np.abs(xyz[i]) < lim)]
    rc, tets, nbrs, _ = oracle_mod.delaunay(xyz[:n0])
    assert rc == 0
    tets, nbrs = tets.astype(np.int64), nbrs.astype(np.int64)
    return [c for c in _cavities(oracle_mod, xyz, tets, nbrs, new) if c is not None]


def _play(att, rng, stop_share):
    """One round: the winners' positions in att (their order is the rank)."""
    order = [[(t, 0) for t in rng.permutation(list(c))] + [(t, 1) for t in rng.permutation(list(o))] for c, o in att]
    for o in order:
        rng.shuffle(o)
    word, lost, done = {}, set(), [0] * len(att)
    running = list(range(len(att)))
    while running:
        r = running[rng.integers(len(running))]
        t, kind = order[r][done[r]]
        t, stamp = int(t), 2 * r + int(kind)
        found = word.get(t, np.inf)
        word[t] = min(found, stamp)
        if 2 * r + 1 < found < np.inf and found % 2 == 0:
            lost.add(int(found) // 2)
        done[r] += 1
        if found < 2 * r and (kind == 0 or found % 2 == 0):
            lost.add(r)
            if rng.random() < stop_share:  # most attempts stop here, some a step later
                running.remove(r)
                continue
        if done[r] == len(order[r]):
            running.remove(r)
    return [r for r in range(len(att)) if r not in lost]


@pytest.mark.parametrize("case", ["uniform", "lattice"])
@pytest.mark.parametrize("stop_share", [0.0, 0.7, 1.0])
def test_unmarked_attempts_are_apart(oracle_mod, case, stop_share):
    att = _attempts(oracle_mod, case)
    assert len(att) > 20
    for seed in range(8):
        winners = _play(att, np.random.default_rng(seed), stop_share)
        assert winners[0] == 0 and 1 < len(winners) < len(att)
        for k, a in enumerate(winners):
            for b in winners[k + 1:]:
                (ca, oa), (cb, ob) = att[a], att[b]
                assert not (ca & cb) and not (ca & ob) and not (oa & cb)
