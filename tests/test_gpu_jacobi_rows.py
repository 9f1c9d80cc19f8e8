"""Edges of the fp64 Jacobi's row-resident rotate pass and its Gram pass:
row counts around the workgroup sizes (64, 128, 256 and 512 rows, chosen by
the number of column pairs and rows), partly filled column blocks, and more
than one inner sweep per meeting."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


def _check(rcs, torch, ln, cnt):
    M = inputs.planted_matrix(ln, cnt, np.geomspace(1.0, 0.05, cnt), seed=ln + 7 * cnt)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    s = torch.zeros(cnt, dtype=torch.float64, device="cuda")
    u = torch.zeros(cnt, ln, dtype=torch.complex128, device="cuda")
    rcs.svd_jacobi(x, s, u)
    s, U = s.cpu().numpy(), u.cpu().numpy().T
    # values: the class of an fp64 SVD; vectors: columns orthogonal to the
    # iteration's relative tolerance 16 u sqrt(len), with a factor 4 for the
    # pairs rotated after they were last measured
    assert np.abs(s - np.geomspace(1.0, 0.05, cnt)).max() <= 1e-13 * np.sqrt(ln)
    tol = 4 * 16 * 1.11e-16 * np.sqrt(max(ln, 16))
    assert np.abs(U.conj().T @ U - np.eye(cnt)).max() <= tol
    assert np.linalg.norm(M - U @ (U.conj().T @ M)) <= tol * np.sqrt(cnt) * np.linalg.norm(M)


# 64-row workgroups up to 16 x 16 columns, then 128 (32 pairs, 520 rows), 256
# (32 pairs, 1,100 rows) and 512 (64 pairs)
@pytest.mark.parametrize("ln,cnt", [(33, 32), (64, 33), (65, 64), (63, 17), (130, 97), (520, 514), (1100, 1010),
                                    (1540, 1537)])
def test_row_workgroups(env, ln, cnt):
    _check(env[0], env[1], ln, cnt)


@pytest.mark.parametrize("ln,cnt,inner", [(40, 30, 2), (100, 90, 3)])
def test_inner_sweeps(env, ln, cnt, inner):
    rcs, torch = env
    try:
        rcs.tuning_set(4096, 16, inner)
        _check(rcs, torch, ln, cnt)
    finally:
        rcs.tuning_clear()


@pytest.mark.parametrize("fixed,free", [(64, 64), (96, 33), (16, 80)])
def test_blocks_that_never_rotate(env, fixed, free):
    """Column blocks orthogonal to everything are skipped from the second
    sweep on while the others go on: the Gram blocks carried between rounds
    have to follow both.  The bars of _check; the fixed columns are the
    largest, so they fill the first blocks."""
    rcs, torch = env
    ln = fixed + free + 9
    M = np.zeros((ln, fixed + free), dtype=np.complex128)
    M[np.arange(fixed), np.arange(fixed)] = np.linspace(3.0, 2.0, fixed)
    M[fixed:, fixed:] = inputs.planted_matrix(free + 9, free, np.geomspace(1.0, 1e-3, free), seed=free)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    s = torch.zeros(fixed + free, dtype=torch.float64, device="cuda")
    u = torch.zeros(fixed + free, ln, dtype=torch.complex128, device="cuda")
    rcs.svd_jacobi(x, s, u)
    s, U = s.cpu().numpy(), u.cpu().numpy().T
    ref = np.concatenate([np.linspace(3.0, 2.0, fixed), np.geomspace(1.0, 1e-3, free)])
    assert np.abs(s - ref).max() <= 1e-13 * np.sqrt(ln) * ref[0]
    tol = 4 * 16 * 1.11e-16 * np.sqrt(ln)
    assert np.abs(U.conj().T @ U - np.eye(fixed + free)).max() <= tol
