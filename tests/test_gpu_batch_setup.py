"""The batch sets all its subdomains up at once: what a single subdomain
refuses is refused wherever it stands in a batch, and subdomains next to each
other in the shared blocks (odd sizes, one with a given initial state) give
the single drains' results bit for bit."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CONV = dict(tol=1e-6, check_every=20, max_steps=60, bisect_rel=0.2)


def _probs():
    out = [synth.small_throat_problem(n=n, seed=n) for n in (17, 25, 18)]
    out[0].rho_init = out[2].rho_init = None
    return out


def test_neighbours_in_the_shared_blocks_equal_single_drains():
    from paper_1906_04722_amd import lbm
    probs = _probs()
    pcs = np.array([[0.003, 0.006]] * 3)
    outs, _ = lbm.drain_batch(probs, pcs, **CONV)
    for p, pc, b in zip(probs, pcs, outs):
        t = lbm.Throat(p)
        s = t.drain(pc, **CONV)
        t.close()
        for k in ("S", "steps", "status"):
            assert np.array_equal(s[k], b[k])


@pytest.mark.parametrize("where", [0, 1, 2])
@pytest.mark.parametrize("what", ["outside", "solid", "bath", "rho_init", "tau"])
def test_a_bad_subdomain_is_refused(where, what):
    from paper_1906_04722_amd import lbm
    probs = _probs()
    p = probs[where]
    if what == "outside":
        q = dict(probe=(p.nx, 1, 1))
    elif what == "solid":
        types = lbm.Throat(p).types().reshape(p.nz, p.ny, p.nx)
        z, y, x = np.argwhere(types == 1)[0]
        q = dict(probe=(int(x), int(y), int(z)))
    elif what == "bath":
        q = dict(probe=(p.probe[0], p.probe[1], 0))
    elif what == "rho_init":
        q = dict(rho_init=np.full((2, p.nz, p.ny, p.nx), np.nan))
    else:
        q = dict(tau=(0.5, 1.0))
    probs[where] = dataclasses.replace(p, **q)
    with pytest.raises(lbm.LBMError):
        lbm.drain_batch(probs, np.array([[0.003, 0.006]] * 3), **CONV)
    with pytest.raises(lbm.LBMError):
        lbm.Throat(probs[where])
