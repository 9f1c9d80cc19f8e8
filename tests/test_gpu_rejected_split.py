"""A randomized split that is rejected leaves the two-site matrix: the full
split that follows takes it from there instead of contracting again, in both
orientations, in every contraction precision."""
import numpy as np
import pytest

from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("contraction", ["c128", "c64", "split_bf16"])
@pytest.mark.parametrize("rows,cols,chi", [(4, 5, 16), (4, 5, 90)])
def test_one_contraction_an_update(rows, cols, chi, contraction):
    rcs, torch = get_rcs()
    c = rcs.Circuit(rows, cols, 8, 3)
    plain = rcs.State.build(c, chi, 1e-10, contraction=contraction)
    two_site = rcs.KERNEL_CLASSES.index("k_two_site")
    rcs.profile_enable(1)
    try:
        st = rcs.State.build(c, chi, 1e-10, contraction=contraction, rank_mode=2, fallback_tau=-1.0,
                             rsvd_oversample=2)
        launches = rcs.profile_read(two_site)["launches"]
    finally:
        rcs.profile_enable(0)
    assert st.info().n_fallbacks > 10
    assert launches == len(st.updates())
    a, b = plain.to_host()[2], st.to_host()[2]
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
