"""The Jacobi's captured sweeps (RCS_JACOBI_GRAPH=1, read once per process,
hence the child process): every matrix runs with its own thresholds, also after
one of the same shape in the same buffers.  The later matrices are the first
times 2^-60, whose columns all lie below the first one's zero level; scaling by
a power of two leaves every rounding alike, so the results scale exactly."""
import os
import subprocess
import sys

import pytest

from tests.conftest import ROOT
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu

SCRIPT = """
import numpy as np, torch
import paper_2512_07311_amd as rcs
from tests import inputs
M = inputs.planted_matrix(150, 130, np.geomspace(1.0, 0.05, 130), seed=5)
shifts = (0, 0, 0, 0, -60, -60, 20, 0)
xs = [torch.from_numpy(np.ascontiguousarray(M.T) * 2.0 ** k).cuda() for k in shifts]
s = torch.zeros(130, dtype=torch.float64, device="cuda")
u = torch.zeros(130, 150, dtype=torch.complex128, device="cuda")
ref = None
for x, k in zip(xs, shifts):
    rcs.svd_jacobi(x, s, u)
    got = s.cpu().numpy() * 2.0 ** -k, u.cpu().numpy()
    ref = ref or got
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]), k
assert np.abs(ref[0] - np.geomspace(1.0, 0.05, 130)).max() <= 1e-13 * np.sqrt(150)
print("graphs ok")
"""


def test_captured_sweeps_take_their_own_thresholds():
    get_rcs()
    env = dict(os.environ, RCS_JACOBI_GRAPH="1")
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "graphs ok" in r.stdout, r.stderr[-2000:]
