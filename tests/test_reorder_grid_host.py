"""fs_cache_reorder cuts sources and heads into launches on the host: the cut
ends at the largest counts the call takes.  Run in a child process without a
GPU, where every launch fails and the call has to come back with that error."""
import subprocess
import sys

import pytest
import torch

CHILD = """
from paper_2106_04718_amd import _native as N
st = N.lib().fs_cache_reorder(1 << 40, None, 1 << 50, {B}, 1, {H}, 1, 1, 1, N.FS_F32, None)
assert st == N.FS_ERR_HIP, (st, N.last_error())
"""


# the largest source count; one that is a whole number of launches; the most heads
@pytest.mark.parametrize("B,H", [(2**31 - 1, 1), (65535 * 32768, 1), (1, 2**29 - 1)])
def test_the_cut_into_launches_ends(B, H):
    if torch.cuda.is_available():
        pytest.skip("the addresses are made up: only where no launch can run")
    subprocess.run([sys.executable, "-c", CHILD.format(B=B, H=H)], check=True, timeout=60)
