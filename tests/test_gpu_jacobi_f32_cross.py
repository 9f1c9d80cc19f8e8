"""Cross rounds of the fp32 Jacobi with one, two and three inner sweeps, at
the edges of its blocks and row chunks."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def env():
    return get_rcs()


# 49 columns are four blocks, 17 two (one launch a sweep); rows end within and
# at a 16-row tile and a 64-row chunk
@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("ln,cnt", [(33, 17), (64, 49), (65, 64), (127, 97)])
def test_f32_cross_rounds(env, ln, cnt, inner):
    """The singular-value bar of test_svd_jacobi_f32, and its orthonormality."""
    rcs, torch = env
    M = inputs.random_complex((ln, cnt), seed=ln + cnt)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    s = torch.zeros(cnt, dtype=torch.float64, device="cuda")
    u = torch.zeros(cnt, ln, dtype=torch.complex128, device="cuda")
    try:
        rcs.tuning_set(4096, 16, inner)
        rcs.svd_jacobi_f32(x, s, u)
    finally:
        rcs.tuning_clear()
    ref = np.linalg.svd(M, compute_uv=False)
    nb = -(-cnt // 16)
    bound = max(64 * U32 * np.sqrt(max(ln, cnt)), 8 * U32 * 10 * nb * inner) * ref[0]
    assert np.abs(s.cpu().numpy() - ref).max() <= bound
    keep = ref > 1e-2 * ref[0]
    U = u.cpu().numpy().T[:, keep]
    assert np.abs(U.conj().T @ U - np.eye(keep.sum())).max() < 1e-4
