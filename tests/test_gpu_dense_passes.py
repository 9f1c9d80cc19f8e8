"""Pass planning of the dense state vector: vectors below, at and just above
one pass's 12 qubits, more gates than one launch carries, idle qubits, no
cycles, no final layer and general fSim angles, against the oracle's dense
simulator (1e-12 2^(-n/2) elementwise, the bar of the other dense tests)."""
import numpy as np
import pytest

from oracle import circuit as oc, dense
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


@pytest.mark.parametrize("rows,cols,cyc,kw", [
    (2, 2, 0, {}), (2, 2, 1, dict(final_1q_layer=False)), (2, 3, 0, dict(final_1q_layer=False)), (2, 6, 20, {}),
    (3, 4, 16, dict(pattern="A")), (2, 7, 9, dict(removed=(3,))), (2, 7, 12, dict(theta=0.7, phi=1.1)),
    (3, 5, 11, dict(removed=(0, 7, 14))), (3, 6, 9, dict(pattern="D")), (4, 4, 24, {}), (2, 9, 13, dict(theta=0.0))])
def test_dense_passes(env, rows, cols, cyc, kw):
    rcs, torch = env
    c = rcs.Circuit(rows, cols, cyc, 11, **kw)
    psi = torch.full((1 << c.n,), float("nan"), dtype=torch.complex128, device="cuda")
    rcs.dense_simulate(c, psi)
    okw = dict(kw)
    if "removed" in okw:
        okw["removed"] = list(okw["removed"])
    if "final_1q_layer" in okw:
        okw["final_layer"] = okw.pop("final_1q_layer")
    ref = dense.simulate(oc.Circuit(rows, cols, cyc, 11, **okw))
    assert np.abs(psi.cpu().numpy() - ref).max() <= 1e-12 * 2.0 ** (-c.n / 2)
