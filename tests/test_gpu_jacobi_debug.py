"""RCS_DEBUG_JACOBI=1 (read once per process, hence the child process) reports
every SVD of a build on stderr, those of small matrices too."""
import os
import re
import subprocess
import sys

import pytest

from tests.conftest import ROOT
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu

SCRIPT = """
import paper_2512_07311_amd as rcs
st = rcs.State.build(rcs.Circuit(2, 6, 8, 1), 64, 0.0)
print("updates", len(st.updates()))
"""


def test_every_split_is_reported():
    get_rcs()
    # CholeskyQR off: moves are SVDs as well
    env = dict(os.environ, RCS_DEBUG_JACOBI="1", RCS_CHOLQR_MOVES="0")
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    updates = int(r.stdout.split()[-1])
    small = re.findall(r"^jacobi (\d+)x(\d+) in one launch: \d+ sweeps", r.stderr, re.M)
    large = re.findall(r"^jacobi (\d+)x(\d+) sweep 1:", r.stderr, re.M)
    assert len(small) + len(large) >= updates
    assert all(int(a) <= 128 and int(b) <= 32 for a, b in small)
    assert all(int(b) > 32 or int(a) > 128 for a, b in large)
