"""Dense state vector of circuits whose couplers never join some qubits to the
others: a pass may then run one pair's couplers to the end of a long circuit
before another pair's first."""
import pytest

from oracle import circuit as oc, dense
from tests.gpu_util import get_rcs, normwise_rel

pytestmark = pytest.mark.gpu


# 2, 3, 4, 6 disjoint pairs (couplers per layer), and pairs of two layers
@pytest.mark.parametrize("rows,cols,pattern", [(2, 2, "A"), (2, 3, "A"), (2, 4, "A"), (3, 4, "C"), (2, 3, "AC")])
def test_long_pairs(rows, cols, pattern):
    rcs, torch = get_rcs()
    cyc = 2500
    c = rcs.Circuit(rows, cols, cyc, 5, pattern=pattern)
    psi = torch.zeros(1 << c.n, dtype=torch.complex128, device="cuda")
    rcs.dense_simulate(c, psi)
    circ = oc.Circuit(rows, cols, cyc, 5, pattern=pattern)
    ref = dense.simulate(circ)
    # a coupler with its two rotations takes an amplitude through four steps of
    # at most four roundings each, with entries rounded once: 20 u, on either side
    steps = sum(len(d) for k, d in circ.layers if k == "2q") + 2 * c.n
    assert normwise_rel(psi.cpu().numpy(), ref) <= 2 * 20 * 1.11e-16 * steps
