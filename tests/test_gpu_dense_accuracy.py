"""Accuracy of the dense state vector over long circuits: no further from an
extended-precision simulation of the same gates (80-bit floats, 64-bit
mantissa) than the gate-by-gate simulation in fp64 is."""
import numpy as np
import pytest

from oracle import circuit as oc, dense
from oracle.circuit import ONE_QUBIT_GATES
from tests.gpu_util import get_rcs, normwise_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


def _extended(circ):
    gates = [np.asarray(u).astype(np.clongdouble) for u in ONE_QUBIT_GATES]
    two = np.asarray(circ.gate2).astype(np.clongdouble)
    psi = np.zeros(1 << circ.n, dtype=np.clongdouble)
    psi[0] = 1
    for kind, data in circ.layers:
        if kind == "1q":
            for q in range(circ.n):
                psi = dense.apply_1q(psi, circ.n, q, gates[int(data[q])])
        else:
            for qa, qb in data:
                psi = dense.apply_2q(psi, circ.n, qa, qb, two)
    return psi


# the last two have fSim angles whose entries repeat other roundings
@pytest.mark.parametrize("rows,cols,cyc,kw", [(2, 5, 100, {}), (3, 4, 200, {}), (2, 4, 300, {}),
                                              (3, 4, 120, dict(theta=0.7, phi=1.1)),
                                              (2, 5, 150, dict(theta=0.3, phi=0.0))])
def test_long_circuits(env, rows, cols, cyc, kw):
    rcs, torch = env
    c = rcs.Circuit(rows, cols, cyc, 7, **kw)
    psi = torch.zeros(1 << c.n, dtype=torch.complex128, device="cuda")
    rcs.dense_simulate(c, psi)
    circ = oc.Circuit(rows, cols, cyc, 7, **kw)
    ref = _extended(circ)
    assert normwise_rel(psi.cpu().numpy(), ref) <= normwise_rel(dense.simulate(circ), ref)
