"""The tiled step at every tile shape on a ragged box that is kept in bricks:
z-segments of one plane, of an odd count and longer than the box, columns cut
by both sides, solids across the periodic face.  Tolerance against the oracle:
1e-5 of each population's natural scale w_k rho, the bar of the other parity
tests; the shapes share their arithmetic, so they agree bit for bit."""
import numpy as np
import pytest

import oracle
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


def _box(bc):
    return Problem(nx=139, ny=131, nz=126, bc=bc,
                   spheres=np.array([[60.0, 65.0, 70.0, 25.0], [138.0, 20.0, 3.0, 9.0],
                                     [30.0, 130.0, 125.0, 11.0]]),
                   z_front=20, rho_in_nw=2.02)


@pytest.mark.parametrize("bc", [(BC_PERIODIC, BC_WALLS, BC_RESERVOIR),
                                (BC_WALLS, BC_PERIODIC, BC_PERIODIC)])
def test_every_tile_shape(bc):
    from paper_1906_04722_amd import lbm
    p = _box(bc)
    o, g = oracle.Oracle(p), lbm.Throat(p)
    assert g.schedule()[0] > 0  # kept in bricks
    o.step(7)
    g.step(7)
    live = o.types() != oracle.SOLID
    rho = g.density()
    a, b = g.f()[:, :, live], o.f()[:, :, live]
    err = float(np.max(np.abs(a - b) / (W[None, :, None] * b.sum(axis=1, keepdims=True))))
    print(bc, "max scaled err", err)
    assert err <= 1e-5
    g.close()
    for tx, ty in ((32, 4), (32, 8), (64, 4), (16, 4), (16, 8), (8, 8)):
        for lz in (1, 13, 200):
            g = lbm.Throat(p)
            g.set_schedule(tx, ty, lz)
            g.step(7)
            assert np.array_equal(g.density(), rho), (tx, ty, lz)
            g.close()
    g = lbm.Throat(p)
    g.set_schedule(lbm.LBM_SCHED_NODE_LIST)  # recorded; the default tiles run
    assert g.schedule()[0] == lbm.LBM_SCHED_NODE_LIST
    g.step(7)
    assert np.array_equal(g.density(), rho)
    g.close()


def test_stores_ahead_of_the_sums_equal_the_two_passes():
    """Boxes of more than 2^24 nodes store a plane before they sum the next
    one; a batch steps the same box in two passes, bit for bit alike."""
    from paper_1906_04722_amd import lbm
    p = Problem(nx=260, ny=257, nz=252, bc=(BC_PERIODIC, BC_WALLS, BC_RESERVOIR),
                spheres=np.array([[120.0, 130.0, 140.0, 40.0], [259.0, 20.0, 3.0, 9.0]]),
                z_front=20, rho_in_nw=2.02, probe=(5, 100, 100))
    assert p.nx * p.ny * p.nz > 1 << 24
    pcs = np.array([0.004, 0.008])
    conv = dict(tol=1e-7, check_every=10, max_steps=20, bisect_rel=0.5)
    one = lbm.Throat(p)
    assert one.schedule()[0] > 0
    ref = one.drain(pcs, **conv)
    one.close()
    out, _ = lbm.drain_batch([p], pcs[None, :], **conv)
    assert np.array_equal(out[0]["S"], ref["S"])
    assert out[0]["total_steps"] == ref["total_steps"]
