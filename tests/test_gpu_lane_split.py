"""The two passes with a lane per component, at the edges of a wavefront's half
(32 nodes), of an item (64) and of the rule's limits (32768, 65536 and 77824
nodes).  Tolerance
against the oracle: 1e-5 of each population's natural scale w_k rho, the bar
of the other parity tests."""
import numpy as np
import pytest

import oracle
import synth
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
BCS = {"p": BC_PERIODIC, "w": BC_WALLS, "r": BC_RESERVOIR}


@pytest.mark.parametrize("shape,bc", [((3, 3, 3), "ppp"), ((4, 4, 4), "wpr"), ((5, 13, 3), "wwr"),
                                      ((32, 32, 32), "pwr"), ((33, 31, 33), "wpp"),
                                      ((32, 33, 32), "pwr"), ((64, 32, 32), "ppp"),
                                      ((41, 40, 40), "pwp"), ((76, 32, 32), "ppp"),
                                      ((60, 40, 33), "wpr")])
def test_lane_split_against_the_oracle(shape, bc):
    from paper_1906_04722_amd import lbm
    nx, ny, nz = shape
    rho0 = synth.layered_density(nx, ny, nz, nz // 2, 2.0, 0.0609883, 3, 1e-3)
    sph = np.array([[0.0, 1.0, nz - 1.0, 1.1]]) if 4 < nx < 40 else np.zeros((0, 4))
    p = Problem(nx=nx, ny=ny, nz=nz, bc=tuple(BCS[c] for c in bc), spheres=sph, rho_init=rho0,
                rho_in_nw=2.02, tau=(1.0, 1.1))
    o, g = oracle.Oracle(p), lbm.Throat(p)
    o.step(12)
    g.step(12)
    live = o.types() != oracle.SOLID
    a, b = g.f()[:, :, live], o.f()[:, :, live]
    g.close()
    err = float(np.max(np.abs(a - b) / (W[None, :, None] * b.sum(axis=1, keepdims=True))))
    print(shape, int(live.sum()), "max scaled err", err)
    assert err <= 1e-5
