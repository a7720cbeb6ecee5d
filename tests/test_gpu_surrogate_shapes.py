"""The surrogate's inference at the edges of its launch shapes: row tiles of 16
and 64, the host-visible buffers of small calls (512 rows) and the chunks of
large ones (32768 rows).  A row's answer does not depend on the call it is part
of: every shape evaluates the same products in the same order, so parts of a
call are bit-identical to the whole.  Against the FP64 reference the norm-wise
bar is the 2e-2 of the BF16 products used by the other surrogate tests."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu

N_ALL = 32769 + 70


def _model(members=3):
    from paper_1906_04722_amd import surrogate
    rng = np.random.default_rng(21)
    m = surrogate.Surrogate(members=members, seed=4)
    ws = [m.get_params(z).astype(np.float64) for z in range(members)]
    F = rng.normal(size=(N_ALL, 80)) * 1.5 + 0.2
    stats = (np.full(80, 0.2), np.full(80, 1.5), rng.normal(size=17), np.full(17, 0.3))
    m.set_stats(*stats)
    return m, ws, F, stats


@pytest.fixture(scope="module")
def whole():
    m, ws, F, stats = _model()
    return m, ws, F, stats, m.predict(F), m.forward(F)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 512, 513, 11000, 32768, 32769])
def test_parts_of_a_call_equal_the_whole(whole, n):
    m, ws, F, stats, (mean, std), y = whole
    a, b = m.predict(F[:n])
    assert np.array_equal(a, mean[:n]) and np.array_equal(b, std[:n])
    assert np.array_equal(m.forward(F[:n]), y[:, :n])


def test_whole_call_against_the_reference(whole):
    m, ws, F, (xm, xs, tm, ts), (mean, std), y = whole
    ref, _ = mlp.predict(ws, (xm, xs), (tm, ts), F[-200:])
    d = np.linalg.norm(mean[-200:] - ref) / np.linalg.norm(ref)
    print("relative error", d)
    assert d <= 2e-2


@pytest.mark.parametrize("n", [3, 600, 40])
def test_non_finite_rows_are_refused_and_outputs_left_alone(n):
    from paper_1906_04722_amd import lbm, surrogate
    m, ws, F, stats = _model(2)
    X = F[:n].copy()
    X[n - 1, 79] = np.inf if n == 40 else np.nan
    mean, std = np.full((n, 17), -7.0), np.full((n, 17), -7.0)
    rc = surrogate.lib().lbm_surrogate_predict(m.h, n, surrogate._d(X), surrogate._d(mean),
                                               surrogate._d(std))
    assert rc == lbm.LBM_ENONFINITE
    assert np.all(mean == -7.0) and np.all(std == -7.0)
    a, _ = m.predict(F[:n])          # the next call is not affected
    assert np.all(np.isfinite(a))
