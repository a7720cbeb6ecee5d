"""What a prediction keeps between calls is bounded, also after a call that was
refused."""
import pytest

from tests import hip_shim

pytestmark = pytest.mark.gpu

RUN = """
from paper_1906_04722_amd import lbm, surrogate
m = surrogate.Surrogate(members=2, seed=1)
m.set_stats(np.zeros(80), np.ones(80), np.zeros(17), np.ones(17))
X = np.random.default_rng(0).normal(size=(200000, 80))
m.predict(X[:100000])
kept = live.value
assert kept > 0
ref = m.predict(X)
assert live.value <= kept, (live.value, kept)
X[150000, 3] = np.nan
try:
    m.predict(X)
    raise SystemExit("a row that is not finite was accepted")
except lbm.LBMError as e:
    assert e.code == lbm.LBM_ENONFINITE
print("live", live.value, "kept", kept)
assert live.value <= kept, (live.value, kept)
again = m.predict(X[:100000])
assert np.array_equal(again[0], ref[0][:100000]) and np.array_equal(again[1], ref[1][:100000])
"""


def test_a_refused_prediction_gives_its_memory_back(tmp_path):
    hip_shim.run(tmp_path, RUN)
