"""The one-launch split and centre move at the edges of its 8, 16 and 32 column forms and of
its range, through builds whose bond cap sets the split's columns to twice
itself."""
import numpy as np
import pytest

from oracle import circuit as oc, mps
from tests import inputs
from tests.gpu_util import truncated_tolerance, get_rcs, to_complex, normwise_rel, oracle_state_from

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


# 6, 8 | 10, 16 | 18, 30, 32 columns; 34 go to the general split; 256 is exact,
# with 128 x 32 splits; 1 and the two-cycle build have rank-deficient matrices
@pytest.mark.parametrize("rows,cols,cyc,chi,eps", [
    (3, 4, 8, 1, 0.0), (3, 4, 8, 3, 0.0), (3, 4, 8, 4, 1e-6), (3, 4, 8, 5, 0.0), (3, 4, 8, 8, 1e-8),
    (3, 4, 8, 9, 0.0), (3, 4, 8, 15, 1e-7), (3, 5, 8, 16, 0.0), (3, 5, 8, 17, 0.0), (3, 5, 8, 256, 0.0),
    (4, 4, 2, 16, 0.0),
])
def test_small_split_build(env, rows, cols, cyc, chi, eps):
    """The bars of test_truncated_build_matches_oracle, and the spectra."""
    rcs, torch = env
    c = rcs.Circuit(rows, cols, cyc, 11)
    g = rcs.State.build(c, chi, eps, log_spectra=True)
    om = mps.build(oc.Circuit(rows, cols, cyc, 11), chi, eps)
    assert list(g.layout()[0]) == om.bond_dims()
    b = inputs.random_bitstrings(c.n, 500, seed=5)
    bits = torch.from_numpy(np.asarray(b).astype(np.int64)).cuda()
    amps = torch.zeros(len(b), 2, dtype=torch.float64, device="cuda")
    g.amplitudes(bits, amps)
    assert normwise_rel(to_complex(amps), om.amplitudes(b)) < truncated_tolerance(om)
    assert oracle_state_from(g.to_host()).canonical_residual() < 1e-12
    for rec in g.spectra():
        v = np.asarray(rec["values"])
        assert len(v) == rec["m"] and np.all(np.diff(v) <= 0.0) and np.all(np.isfinite(v))
