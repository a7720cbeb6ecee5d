"""The two ways the second pass stores populations, at both ends of the range
of sizes where it stores through the caches (165.6 k and 993.4 k stepped nodes):
boxes just below and just above each.  Tolerance: 1e-5 of each population's
natural scale w_k rho against the oracle, the bar of the other parity tests."""
import numpy as np
import pytest

import oracle
import synth
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


@pytest.mark.parametrize("shape", [(55, 55, 54), (56, 55, 55), (99, 100, 100), (100, 101, 100)])
def test_store_variants_against_the_oracle(shape):
    from paper_1906_04722_amd import lbm
    nx, ny, nz = shape
    rho0 = synth.layered_density(nx, ny, nz, nz // 2, 2.0, 0.0609883, 3, 1e-3)
    p = Problem(nx=nx, ny=ny, nz=nz, bc=(BC_PERIODIC, BC_WALLS, BC_RESERVOIR),
                spheres=np.array([[3.0, 0.0, 8.0, 2.2]]), rho_init=rho0, rho_in_nw=2.02)
    o, g = oracle.Oracle(p), lbm.Throat(p)
    g.set_schedule(lbm.LBM_SCHED_NODE_LIST)
    o.step(5)
    g.step(5)
    live = o.types() != oracle.SOLID
    a, b = g.f()[:, :, live], o.f()[:, :, live]
    g.close()
    err = float(np.max(np.abs(a - b) / (W[None, :, None] * b.sum(axis=1, keepdims=True))))
    print(shape, int(live.sum()), "max scaled err", err)
    assert err <= 1e-5
