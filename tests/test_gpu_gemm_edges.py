"""Edges of the fp64 tile GEMM: sizes around the 64-wide tile and the
16-deep stage, through the two-site contraction (both operands) and the
sampler's row-indirect product (amplitudes of a ragged state)."""
import numpy as np
import pytest

from oracle import circuit as oc, mps
from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


@pytest.mark.parametrize("dl,dm,dr", [(1, 1, 1), (64, 16, 64), (65, 17, 63), (63, 15, 129), (2, 33, 64),
                                      (128, 48, 1), (31, 200, 66)])
def test_contraction_edges(env, dl, dm, dr):
    """Elementwise forward bound of a complex inner product of dm terms (two
    roundings per real term, four real products) followed by the 4-term gate
    sum: (2 dm + 24) u (|G| (|A| |B|)), with |x| taken as |re| + |im|."""
    rcs, torch = env
    A = inputs.random_complex((dl, 2, dm), 11)
    B = inputs.random_complex((dm, 2, dr), 12)
    G = oc.fsim(np.pi / 2, np.pi / 6)
    st = mps.MPS(2, [0, 1])
    st.A = [A, B]
    ref, _, _ = st.two_site_matrix(0, G)
    ab = lambda z: (np.abs(z.real) + np.abs(z.imag)).astype(complex)   # noqa: E731
    st.A = [ab(A), ab(B)]
    mag, _, _ = st.two_site_matrix(0, ab(G))
    out = torch.zeros(2 * dr, 2 * dl, dtype=torch.complex128, device="cuda")
    rcs.two_site(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), G, out)
    assert np.all(np.abs(out.cpu().numpy().T - ref) <= (2 * dm + 24) * 2.0 ** -53 * 2 * mag.real)


@pytest.mark.parametrize("dims,m", [([1, 2, 4, 2, 1], 1), ([1, 2, 4, 8, 15, 31, 33, 17, 16, 8, 4, 2, 1], 65),
                                    ([1, 2, 4, 8, 16, 32, 64, 65, 63, 32, 16, 8, 4, 2, 1], 127)])
def test_row_indirect_edges(env, dims, m):
    rcs, torch = env
    A = inputs.random_site_tensors(dims, 5)
    n = len(A)
    snake = list(range(n))
    st = rcs.State.from_host(dims, snake, A, canonical=False)
    bits = inputs.random_bitstrings(n, m, 6)
    got = torch.zeros(m, dtype=torch.complex128, device="cuda")
    st.amplitudes(torch.from_numpy(bits.astype(np.int64)).cuda(), got)
    o = mps.MPS(n, snake)
    o.A = A
    ref = o.amplitudes(bits)
    o.A = [(np.abs(a.real) + np.abs(a.imag)).astype(complex) for a in A]
    mag = o.amplitudes(bits).real
    assert np.all(np.abs(got.cpu().numpy() - ref) <= sum(2 * d + 8 for d in dims) * 2.0 ** -53 * 2 * mag)


@pytest.mark.parametrize("precision", ["c64", "split_bf16"])
@pytest.mark.parametrize("dl,dm,dr", [(1, 1, 1), (33, 31, 65), (32, 33, 31), (40, 129, 32)])
def test_reduced_precision_edges(env, precision, dl, dm, dr):
    """Against the oracle's emulation of the same operand rounding; the bar is
    fp32 accumulation noise of dm terms of size about 2 (8 units of 2^-24
    times the root of the term count and the sum's size)."""
    from oracle import precision as prec
    rcs, torch = env
    A, B = inputs.random_complex((dl, 2, dm), 21), inputs.random_complex((dm, 2, dr), 22)
    G = oc.fsim(np.pi / 2, np.pi / 6)
    mm = prec.matmul_c64 if precision == "c64" else prec.matmul_split_bf16_complex
    T = np.array([[mm(A[:, s], B[:, t]) for t in range(2)] for s in range(2)])
    ref = np.einsum("xyst,stac->axyc", G.reshape(2, 2, 2, 2), T).transpose(1, 0, 2, 3).reshape(2 * dl, 2 * dr)
    out = torch.zeros(2 * dr, 2 * dl, dtype=torch.complex128, device="cuda")
    rcs.two_site(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), G, out, precision=precision)
    assert np.abs(out.cpu().numpy().T - ref).max() <= 8 * 2.0 ** -24 * np.sqrt(2 * dm) * 2.0 * np.sqrt(dm)
