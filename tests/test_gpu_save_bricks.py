"""Checkpoint files hold nodes only: a subdomain in bricks saves zeros in its
solid slots, its padding and, unless it is periodic in z, its ghost planes,
whatever its buffers hold there, so that two handles in one state save the
same bytes.  (The file's buffer is [nz + 2][ny / 4][nx / 8][38][4][8].)"""
import numpy as np
import pytest

from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

pytestmark = pytest.mark.gpu

NX, NY, NZ = 126, 127, 140   # large and open enough to be kept in bricks


@pytest.mark.parametrize("bc_z", [BC_RESERVOIR, BC_PERIODIC])
def test_a_saved_brick_box_is_zero_where_it_has_no_node(tmp_path, bc_z):
    from paper_1906_04722_amd import lbm
    p = Problem(nx=NX, ny=NY, nz=NZ, bc=(BC_PERIODIC, BC_WALLS, bc_z),
                spheres=np.array([[60.0, 65.0, 70.0, 25.0], [20.0, 30.0, 1.0, 9.0]]), z_front=20,
                rho_in_nw=2.02)
    a, b = lbm.Throat(p), lbm.Throat(p)
    assert a.schedule()[0] > 0
    solid = np.ones((NZ + 2, 128, 128), bool)
    solid[1:NZ + 1, :NY, :NX] = a.types().reshape(NZ, NY, NX) == lbm.LBM_NODE_SOLID
    if bc_z == BC_PERIODIC:
        solid[0], solid[-1] = solid[NZ], solid[1]
    none = solid.reshape(NZ + 2, 32, 4, 16, 8).transpose(0, 1, 3, 2, 4)[:, :, :, None]
    path = str(tmp_path / "a.lbm")
    a.step(4)
    a.save(path)
    raw = np.fromfile(path, np.uint8)
    buf = raw[raw.size - 4 * 38 * solid.size:].view(np.float32).reshape(NZ + 2, 32, 16, 38, 4, 8)
    kept = raw.copy()
    assert not np.any(buf * none)
    # a file that holds something there: it loads, and is not passed on
    np.copyto(buf, np.float32(7.0), where=none)
    assert not np.array_equal(raw, kept)
    raw.tofile(path)
    b.load(path)
    b.save(path)
    assert np.array_equal(np.fromfile(path, np.uint8), kept)
    a.step(3)
    b.step(3)
    assert np.array_equal(a.density(), b.density())
    a.close()
    b.close()
