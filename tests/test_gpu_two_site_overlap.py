"""Two-site contraction into memory that it reads from: many tiles of the output
are written while others are still computed, so an operand that shares memory
with the output has to be read as it was; the bytes equal those of a separate
output."""
import numpy as np
import pytest

from oracle import circuit as oc
from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


# a, b: the output lies exactly in that operand; offset: it starts inside A and
# goes past the end of B, which follows A; row: its last element is A's first
@pytest.mark.parametrize("precision", ["c128", "c64", "split_bf16"])
@pytest.mark.parametrize("dl,dm,dr,where", [(100, 140, 70, "a"), (70, 140, 100, "b"), (97, 130, 131, "offset"),
                                            (65, 33, 64, "row")])
def test_output_in_an_operand(env, dl, dm, dr, where, precision):
    rcs, torch = env
    G = oc.fsim(np.pi / 2, np.pi / 6)
    A = torch.from_numpy(inputs.random_complex((dl, 2, dm), 31)).cuda()
    B = torch.from_numpy(inputs.random_complex((dm, 2, dr), 32)).cuda()
    ref = torch.zeros(2 * dr, 2 * dl, dtype=torch.complex128, device="cuda")
    rcs.two_site(A, B, G, ref, precision=precision)
    n, na, nb = ref.numel(), A.numel(), B.numel()
    buf = torch.zeros(2 * n + na + nb, dtype=torch.complex128, device="cuda")
    a = buf[n:n + na].copy_(A.reshape(-1)).view(dl, 2, dm)
    b = buf[n + na:n + na + nb].copy_(B.reshape(-1)).view(dm, 2, dr)
    at = dict(a=n, b=n + na, offset=n + na // 2, row=1)[where]
    out = buf[at:at + n].view(2 * dr, 2 * dl)
    assert out.numel() == n
    rcs.two_site(a, b, G, out, precision=precision)
    assert torch.equal(torch.view_as_real(out), torch.view_as_real(ref))
