"""Saving and loading a subdomain needs no device memory of its own: both still
work where none can be had."""
import pytest

from tests import hip_shim

pytestmark = pytest.mark.gpu

RUN = """
import synth
from paper_1906_04722_amd import lbm
path = sys.argv[3]
few = synth.Problem(nx=40, ny=40, nz=40, bc=(synth.BC_WALLS,) * 3,
                    spheres=np.array([[20.0, 20.0, 20.0, 33.0]]))
for p in (synth.c1_problem(seed=1), few):
    a, b = lbm.Throat(p), lbm.Throat(p)
    a.step(31)
    ref = a.f()
    deny.value = 1
    try:
        lbm.Throat(p)
        raise SystemExit("the allocations were not denied")
    except lbm.LBMError as e:
        assert e.code == lbm.LBM_ENOMEM
    a.save(path)
    b.load(path)
    deny.value = 0
    assert np.array_equal(b.f(), ref)
    a.step(9)
    b.step(9)
    assert np.array_equal(a.f(), b.f())
"""


def test_save_and_load_without_device_memory(tmp_path):
    hip_shim.run(tmp_path, RUN, str(tmp_path / "state.lbm"))
