"""Scale invariance of the fp64 Jacobi: a matrix times a power of two has the
same left singular vectors and the scaled singular values, bit for bit, also
where the squares of the squared column norms leave the fp64 range."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


def _svd(rcs, torch, M, shift):
    ln, cnt = M.shape
    x = torch.from_numpy(np.ascontiguousarray(np.ldexp(M.T.copy().view(np.float64), shift)).view(np.complex128)).cuda()
    s = torch.zeros(cnt, dtype=torch.float64, device="cuda")
    u = torch.zeros(cnt, ln, dtype=torch.complex128, device="cuda")
    rcs.svd_jacobi(x, s, u)
    return s.cpu().numpy(), u.cpu().numpy()


# one column pair block, and several with row-resident workgroups; 32-column
# blocks take the rotations from a product instead
@pytest.mark.parametrize("ln,cnt,block", [(40, 24, 16), (203, 131, 16), (130, 100, 32)])
@pytest.mark.parametrize("shift", [-400, -230, -149, 149, 260, 400])
def test_power_of_two_scaling(env, ln, cnt, block, shift):
    rcs, torch = env
    # singular values in groups of equal ones, so that equally long columns meet
    M = inputs.planted_matrix(ln, cnt, np.repeat([1.0, 0.5, 0.25], cnt)[:cnt * 3:3], seed=ln + cnt)
    try:
        rcs.tuning_set(4096, block, 1)
        s0, u0 = _svd(rcs, torch, M, 0)
        s, u = _svd(rcs, torch, M, shift)
    finally:
        rcs.tuning_clear()
    U = u0.T
    assert np.abs(U.conj().T @ U - np.eye(cnt)).max() <= 4 * 16 * 1.11e-16 * np.sqrt(ln)
    assert np.array_equal(np.ldexp(s, -shift), s0)
    assert np.array_equal(u, u0)
