"""Singular values against planted ones in extended precision.

A column takes part in about 15 (cnt - 1) rotations.  The rounding of its
entries averages out in its norm, to about sqrt(15 cnt / (2 len)) u, 2 to 3 u
here; what is rounded once for a whole column (cosines, scales) does not and
would add up to sqrt(15 cnt) u or more, 25 to 80 u.  The bar lies between."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu
U = 1.11e-16


def _orthonormal(n, k, seed):
    q = np.linalg.qr(inputs.random_complex((n, k), seed))[0].astype(np.clongdouble)
    return q @ (1.5 * np.eye(k, dtype=np.clongdouble) - 0.5 * (q.conj().T @ q))


@pytest.mark.parametrize("ln,cnt", [(60, 36), (68, 40), (118, 87), (203, 131), (300, 200)])
def test_singular_values_to_rounding(ln, cnt):
    rcs, torch = get_rcs()
    s = np.linspace(1.0, 0.1, cnt).astype(np.longdouble)
    x = (_orthonormal(ln, cnt, 1) * s) @ _orthonormal(cnt, cnt, 2).conj().T
    xd = torch.from_numpy(np.ascontiguousarray(x.T).astype(np.complex128)).cuda()
    sd = torch.zeros(cnt, dtype=torch.float64, device="cuda")
    rcs.svd_jacobi(xd, sd, torch.zeros_like(xd))
    got = sd.cpu().numpy()
    assert np.linalg.norm(got - s) <= 16 * U * np.linalg.norm(s)

