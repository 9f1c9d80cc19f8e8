"""Cholesky panels at the edges of their 64-column and 16-column blocks and
the Newton-Schulz step count, through the QR that uses both."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


# cond 1e1 needs one Newton-Schulz step, 1e4 two, 1e5 up to three
@pytest.mark.parametrize("cond", [1e1, 1e4, 1e5])
@pytest.mark.parametrize("ln,cnt", [(64, 64), (70, 65), (129, 80), (200, 127), (193, 129), (400, 193)])
def test_qr_edges(env, ln, cnt, cond):
    """The bars of test_cholqr_against_numpy_qr."""
    rcs, torch = env
    M = inputs.planted_matrix(ln, cnt, np.geomspace(1.0, 1.0 / cond, cnt), seed=ln + cnt)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    q = torch.zeros(cnt, ln, dtype=torch.complex128, device="cuda")
    r = torch.zeros(cnt, cnt, dtype=torch.complex128, device="cuda")
    rcs.cholqr(x, q, r)
    Q, R = q.cpu().numpy().T, r.cpu().numpy().T
    assert np.abs(Q.conj().T @ Q - np.eye(cnt)).max() < 1e-13
    assert np.linalg.norm(M - Q @ R) <= 1e-14 * np.linalg.norm(M) * np.sqrt(cnt)
    assert np.abs(np.tril(R, -1)).max() <= 1e-10 * np.abs(R).max()


def test_breakdown_is_reported(env):
    """A zero pivot in the last column of a partly filled block."""
    rcs, torch = env
    M = inputs.random_complex((150, 70), 3)
    M[:, 69] = M[:, 0]
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    q = torch.zeros(70, 150, dtype=torch.complex128, device="cuda")
    r = torch.zeros(70, 70, dtype=torch.complex128, device="cuda")
    with pytest.raises(rcs.RcsError) as ei:
        rcs.cholqr(x, q, r)
    assert ei.value.status == 5


@pytest.mark.parametrize("cond", [1e1, 1e4, 1e5])
def test_q_in_place_of_x(env, cond):
    """x is read while q is written: one buffer for both gives the same bytes."""
    rcs, torch = env
    M = inputs.planted_matrix(200, 127, np.geomspace(1.0, 1.0 / cond, 127), seed=9)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    q = torch.zeros(127, 200, dtype=torch.complex128, device="cuda")
    r = torch.zeros(127, 127, dtype=torch.complex128, device="cuda")
    r2 = torch.zeros_like(r)
    rcs.cholqr(x, q, r)
    rcs.cholqr(x, x, r2)
    assert torch.equal(q, x) and torch.equal(r, r2)


@pytest.mark.parametrize("ln,cnt", [(256, 64), (517, 65), (1030, 130), (2050, 64)])
def test_qr_split_products(env, ln, cnt):
    """K ranges of the split products that end within a 16-row stage, and the
    most ranges; the bars of test_qr_edges."""
    rcs, torch = env
    M = inputs.planted_matrix(ln, cnt, np.geomspace(1.0, 1e-3, cnt), seed=ln)
    x = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    q = torch.zeros(cnt, ln, dtype=torch.complex128, device="cuda")
    r = torch.zeros(cnt, cnt, dtype=torch.complex128, device="cuda")
    rcs.cholqr(x, q, r)
    Q, R = q.cpu().numpy().T, r.cpu().numpy().T
    assert np.abs(Q.conj().T @ Q - np.eye(cnt)).max() < 1e-13
    assert np.linalg.norm(M - Q @ R) <= 1e-14 * np.linalg.norm(M) * np.sqrt(cnt)
