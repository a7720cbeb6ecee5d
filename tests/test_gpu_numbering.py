"""The node numberings and the two step paths at the sizes where they can go
wrong: rows around one wavefront (64) long, row groups around 32, periodic
wraps of the shortest axes, and a box large and open enough for the tiled step.

Tolerance against the oracle: 1e-5 of each population's natural scale w_k rho,
the bar of the other parity tests (FP32 storage, 30 steps).  The two step
paths and the batch share their arithmetic, so they agree bit for bit."""
import numpy as np
import pytest

import oracle
import synth
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


@pytest.mark.parametrize("shape,bc", [
    ((63, 31, 4), (BC_PERIODIC, BC_WALLS, BC_RESERVOIR)),
    ((64, 32, 3), (BC_PERIODIC, BC_PERIODIC, BC_PERIODIC)),
    ((65, 33, 5), (BC_WALLS, BC_PERIODIC, BC_RESERVOIR)),
    ((3, 65, 33), (BC_PERIODIC, BC_PERIODIC, BC_WALLS)),
    ((130, 3, 9), (BC_WALLS, BC_PERIODIC, BC_PERIODIC)),
])
def test_rows_and_groups_against_the_oracle(shape, bc):
    from paper_1906_04722_amd import lbm
    nx, ny, nz = shape
    sph = np.array([[0.4 * nx, 0.5 * ny, 0.5 * nz, 1.2], [nx - 1.0, 0.0, 0.0, 1.1],
                    [0.0, ny - 1.0, nz - 1.0, 0.6]])
    rho0 = synth.layered_density(nx, ny, nz, nz // 2, 2.0, 0.0609883, 11, 1e-3)
    p = Problem(nx=nx, ny=ny, nz=nz, bc=bc, spheres=sph, rho_init=rho0, rho_in_nw=2.02)
    o, g = oracle.Oracle(p), lbm.Throat(p)
    assert np.array_equal(g.types(), o.types())
    o.step(30)
    g.step(30)
    live = o.types() != oracle.SOLID
    a, b = g.f()[:, :, live], o.f()[:, :, live]
    err = float(np.max(np.abs(a - b) / (W[None, :, None] * b.sum(axis=1, keepdims=True))))
    mg, Sg = g.reduce()
    mo, So, _ = o.reduce()
    g.close()
    print(shape, "max scaled err", err)
    assert err <= 1e-5
    np.testing.assert_allclose(mg, mo, rtol=1e-6)
    assert abs(Sg - So) < 1e-6


def _open_box():
    """Large and open enough to be kept in bricks, with a solid and baths."""
    return Problem(nx=170, ny=169, nz=168, bc=(BC_PERIODIC, BC_WALLS, BC_RESERVOIR),
                   spheres=np.array([[80.0, 85.0, 90.0, 30.0]]), z_front=20, rho_in_nw=2.02,
                   probe=(5, 80, 100))


def test_tiled_step_equals_the_two_passes_and_the_batch(tmp_path):
    from paper_1906_04722_amd import lbm
    p = _open_box()
    tiles, lists = lbm.Throat(p), lbm.Throat(p)
    assert tiles.schedule()[0] > 0      # the tiled step is the default here
    lists.set_schedule(lbm.LBM_SCHED_NODE_LIST)
    tiles.step(21)
    lists.step(21)
    d = tiles.density()
    assert np.array_equal(d, lists.density())
    path = str(tmp_path / "open.lbm")
    tiles.save(path)
    lists.step(4)
    lists.load(path)
    assert np.array_equal(lists.density(), d)
    lists.close()
    tiles.close()
    # the batch keeps every subdomain in the compact numbering
    pcs = np.array([0.004, 0.008])
    conv = dict(tol=1e-7, check_every=20, max_steps=40, bisect_rel=0.5)
    one = lbm.Throat(p)
    ref = one.drain(pcs, **conv)
    one.close()
    out, _ = lbm.drain_batch([p], pcs[None, :], **conv)
    assert np.array_equal(out[0]["S"], ref["S"])
    assert out[0]["total_steps"] == ref["total_steps"]
