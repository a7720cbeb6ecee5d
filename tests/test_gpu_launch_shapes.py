"""The launch shape that is asked for is the one that runs: tiles over bricks,
the two passes over the compact nodes, whichever of the two a subdomain was
set up in.  Its state, ramp and checkpoints move between the two bit for bit,
and a shape whose storage cannot be had leaves the subdomain as it was."""
import numpy as np
import pytest

import synth
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem
from tests import hip_shim

pytestmark = pytest.mark.gpu

LIST = (-1, 0, 0)


def _ragged(bc):
    return Problem(nx=37, ny=34, nz=19, bc=bc, tau=(0.9, 1.1), rho_in_nw=2.02, z_front=6,
                   spheres=np.array([[12.0, 14.0, 9.0, 7.5], [36.0, 2.0, 18.0, 3.2]]),
                   probe=(20, 25, 10))


# a compact box of which four fifths are solid
STORAGE = """
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem
from paper_1906_04722_amd import lbm
LIST = (-1, 0, 0)
sph = np.array([[x, y, z, 19.8] for x in (16, 48, 80) for y in (16, 48, 80) for z in (16, 48, 80)],
               float)
g = lbm.Throat(Problem(nx=97, ny=98, nz=96, bc=(BC_WALLS, BC_PERIODIC, BC_RESERVOIR), spheres=sph,
                       rho_in_nw=2.02, z_front=12))
nodes = int((g.types() != lbm.LBM_NODE_SOLID).sum())
assert nodes < 0.25 * g.N and g.schedule() == LIST
g.step(7)
f, compact = g.f(), live.value
more = 2 * 152 * (g.N - nodes)  # two buffers of every node of the box
g.set_schedule(32, 8, 16)
print("compact", compact, "bricks", live.value, "nodes add", more)
assert live.value - compact > 0.95 * more
assert g.schedule() == (32, 8, 16) and np.array_equal(g.f(), f)
g.set_schedule(*LIST)
assert live.value - compact < 0.01 * more
assert g.schedule() == LIST and np.array_equal(g.f(), f)
deny.value = 1
try:
    g.set_schedule(16, 8, 5)
    raise SystemExit("storage that cannot be had was not refused")
except lbm.LBMError as e:
    assert e.code == lbm.LBM_ENOMEM
deny.value = 0
assert g.schedule() == LIST and np.array_equal(g.f(), f)
g.step(2)
h = g.f()
g.close()
assert live.value == 0
"""


def test_tiles_and_two_passes_have_their_own_storage(tmp_path):
    hip_shim.run(tmp_path, STORAGE)


# buffers of 3 MB and more are denied: populations are, the index map is not
IN_PLACE = """
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem
from paper_1906_04722_amd import lbm
LIST = (-1, 0, 0)
pcs, conv = np.array([0.004, 0.02, 0.05]), dict(tol=1e-9, check_every=20, max_steps=40, bisect_rel=0.3)
for bc in ((BC_WALLS, BC_PERIODIC, BC_RESERVOIR), (BC_PERIODIC,) * 3):
    p = Problem(nx=37, ny=34, nz=19, bc=bc, tau=(0.9, 1.1), rho_in_nw=2.02, z_front=6,
                spheres=np.array([[12.0, 14.0, 9.0, 7.5], [36.0, 2.0, 18.0, 3.2]]),
                probe=(20, 25, 10))
    one = lbm.Throat(p)
    ref = one.drain(pcs, **conv)
    g = lbm.Throat(p)
    g.set_schedule(32, 8, 5)
    g.drain_begin(pcs, **conv)
    assert not g.drain_advance(20)
    f, held = g.f(), live.value
    deny.value = 3000000
    g.set_schedule(*LIST)
    assert abs(live.value - held) < 1000000
    try:
        g.set_schedule(32, 8, 5)
        raise SystemExit("storage that cannot be had was not refused")
    except lbm.LBMError as e:
        assert e.code == lbm.LBM_ENOMEM
    deny.value = 0
    assert g.schedule() == LIST and np.array_equal(g.f(), f)
    g.drain_advance(20)
    g.set_schedule(16, 8, 4)
    while not g.drain_advance(20):
        pass
    got = g.drain_get()
    assert all(np.array_equal(got[k], ref[k]) for k in ("S", "steps", "status"))
    assert got["n_bisect"] == ref["n_bisect"] and np.array_equal(g.f(), one.f())
    print(got["S"], got["n_bisect"])
    g.close()
    one.close()
assert live.value == 0
"""


def test_two_passes_take_the_buffers_of_the_tiles(tmp_path):
    hip_shim.run(tmp_path, IN_PLACE)


@pytest.mark.parametrize("bc", [(BC_WALLS, BC_PERIODIC, BC_RESERVOIR), (BC_PERIODIC,) * 3])
def test_the_state_moves_between_the_shapes(bc, tmp_path):
    from paper_1906_04722_amd import lbm
    p = _ragged(bc)
    a, b = lbm.Throat(p), lbm.Throat(p)
    for n, shape in ((3, (32, 4, 5)), (4, (8, 8, 2)), (1, LIST), (2, (64, 4, 40)), (5, LIST)):
        b.set_schedule(*shape)
        assert b.schedule() == shape
        assert np.array_equal(a.f(), b.f())
        a.step(n)
        b.step(n)
        assert np.array_equal(a.f(), b.f()) and a.probe_invaded() == b.probe_invaded()
        (ma, Sa), (mb, Sb) = a.reduce(), b.reduce()
        assert np.array_equal(ma, mb) and Sa == Sb
    # a file of either numbering is the same file
    b.set_schedule(16, 8, 3)
    a.save(str(tmp_path / "a"))
    b.save(str(tmp_path / "b"))
    assert (tmp_path / "a").read_bytes() == (tmp_path / "b").read_bytes()
    b.step(2)
    b.load(str(tmp_path / "a"))
    b.step(3)
    a.step(3)
    assert np.array_equal(a.f(), b.f())
    a.close()
    b.close()


def test_a_ramp_goes_on_in_another_shape():
    from paper_1906_04722_amd import lbm
    p = synth.c2_problem(n=40, mean_r=32.0 * 40 / 96, seed=11)
    r_ins, _ = synth.throat_incircle(p.spheres)
    pcs = synth.pc_ramp(synth.GAMMA_LAPLACE, r_ins, 5, 0.1, 0.9)
    conv = dict(tol=1e-5, check_every=100, max_steps=3000, bisect_rel=0.02)
    one = lbm.Throat(p)
    ref = one.drain(pcs, **conv)
    assert ref["n_bisect"] >= 1
    g = lbm.Throat(p)
    g.drain_begin(pcs, **conv)
    shapes = [(32, 8, 7), LIST, (16, 4, 40)]
    i = 0
    while not g.drain_advance(300):
        g.set_schedule(*shapes[i % 3])
        i += 1
    got = g.drain_get()
    assert i >= 6
    for k in ("S", "steps", "status"):
        assert np.array_equal(got[k], ref[k])
    for k in ("pce_lo", "pce_hi", "invaded_at", "n_bisect", "total_steps"):
        assert got[k] == ref[k]
    assert np.array_equal(g.f(), one.f())
    g.close()
    one.close()


def test_a_shape_beyond_the_budget_changes_nothing():
    from paper_1906_04722_amd import lbm
    p = _ragged((BC_PERIODIC,) * 3)
    a, b = lbm.Throat(p), lbm.Throat(p)
    a.step(3)
    b.step(3)
    lbm.set_memory_budget(1 << 20)
    try:
        with pytest.raises(lbm.LBMError) as e:
            b.set_schedule(32, 8, 4)
        assert e.value.code == lbm.LBM_ENOMEM
    finally:
        lbm.set_memory_budget(0)
    assert b.schedule() == LIST
    a.step(4)
    b.step(4)
    assert np.array_equal(a.f(), b.f())
    a.close()
    b.close()


@pytest.mark.parametrize("start", [None, LIST])
def test_autotuner_trials_leave_a_brick_box_as_it_was(start):
    from paper_1906_04722_amd import lbm
    p = Problem(nx=126, ny=127, nz=140, bc=(BC_PERIODIC,) * 3, z_front=60,
                spheres=np.array([[60.0, 65.0, 70.0, 25.0], [20.0, 30.0, 1.0, 9.0]]))
    a, b = lbm.Throat(p), lbm.Throat(p)
    a.step(5)
    b.step(5)
    if start:
        b.set_schedule(*start)
    shape = b.autotune(3)
    print("picked", shape)
    assert shape[0] > 0 and b.schedule() == shape
    assert np.array_equal(a.density(), b.density())
    a.step(6)
    b.step(6)
    assert np.array_equal(a.density(), b.density())
    a.close()
    b.close()


@pytest.mark.parametrize("shape,tiles", [((128, 128, 128), True), ((64, 64, 520), True),
                                         ((129, 129, 129), False), ((40, 40, 1400), False),
                                         ((33, 65, 1000), False), ((8, 8, 33000), False)])
def test_open_boxes_start_in_tiles_where_these_are_full(shape, tiles):
    from paper_1906_04722_amd import lbm
    nx, ny, nz = shape
    g = lbm.Throat(Problem(nx=nx, ny=ny, nz=nz, bc=(BC_PERIODIC,) * 3, z_front=nz // 2))
    assert (g.schedule()[0] > 0) == tiles
    g.close()
