"""Open boxes of a batch are stepped in tiles, their sizes taken together,
beside subdomains in two passes: each gives its single drain bit for bit (odd
and periodic sizes, z-segments of unequal boxes, checkpoints and ghost planes of
a bisection)."""
import numpy as np
import pytest

import synth
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

CONV = dict(tol=1e-7, check_every=20, max_steps=60, bisect_rel=0.3)


def _open(nx, ny, nz, bc, probe):
    return Problem(nx=nx, ny=ny, nz=nz, bc=bc, z_front=nz // 4, rho_in_nw=2.02, probe=probe,
                   spheres=np.array([[0.5 * nx, 0.4 * ny, 0.6 * nz, 0.15 * nx], [nx - 1.0, 3.0, 1.0, 5.0]]))


RES = (BC_PERIODIC, BC_WALLS, BC_RESERVOIR)
ALL = (BC_PERIODIC,) * 3


@pytest.mark.parametrize("which", ["one", "several", "mixed"])
def test_open_boxes_equal_their_single_drains(which):
    from paper_1906_04722_amd import lbm
    wall = _open(127, 128, 140, RES, (5, 60, 100))
    turn = _open(96, 95, 77, ALL, (5, 50, 60))
    first = _open(128, 112, 33, RES, (100, 60, 3))  # its probe is invaded at once
    small = synth.small_throat_problem(n=24, seed=3)
    probs = {"one": [wall], "several": [turn, first, wall],
             "mixed": [small, first, turn, small, wall]}[which]
    pcs = np.tile(np.array([0.004, 0.008]), (len(probs), 1))
    outs, info = lbm.drain_batch(probs, pcs, **CONV)
    print(which, info)
    assert (info["tx"] > 0) == (which != "mixed")
    singles = {}
    for p, pc, b in zip(probs, pcs, outs):
        if id(p) not in singles:
            t = lbm.Throat(p)
            singles[id(p)] = t.drain(pc, **CONV)
            t.close()
        s = singles[id(p)]
        for k in ("S", "steps", "status"):
            assert np.array_equal(s[k], b[k]), k
        for k in ("pce", "pce_lo", "pce_hi"):
            assert np.array_equal(s[k], b[k], equal_nan=True), k
        for k in ("invaded_at", "n_bisect", "total_steps"):
            assert s[k] == b[k], k
    if which != "one":
        assert singles[id(first)]["n_bisect"] >= 1


def test_a_few_small_open_boxes_stay_in_two_passes():
    from paper_1906_04722_amd import lbm
    probs = [_open(64, 48, 40, RES, (5, 20, 30))] * 3
    outs, info = lbm.drain_batch(probs, np.array([[0.004, 0.008]] * 3), **CONV)
    assert info["tx"] == lbm.LBM_SCHED_NODE_LIST
    assert np.array_equal(outs[0]["S"], outs[2]["S"])
