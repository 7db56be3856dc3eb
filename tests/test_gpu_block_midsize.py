"""Block convs on the rings whose key switches are fused (needs an MI355X), where all
rotations of all blocks go through them together.  Word for word against the oracle's block
conv: full and block-diagonal layers (output blocks with different zero diagonals), more
inputs than one ModUp takes, more jobs than one launch takes, one to several rotations, and
no rotation at all."""
import numpy as np
import pytest

import oracle.plans as PL

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.midsize import mid_workload  # noqa: E402
from tests.test_gpu_conv_variants import Rig, run_parity  # noqa: E402

RIGS = {}


def rig(log_n, alpha):
    if (log_n, alpha) not in RIGS:
        RIGS[log_n, alpha] = Rig(mid_workload(log_n, alpha), True)
    return RIGS[log_n, alpha]


@pytest.mark.parametrize("log_n,alpha,level,w0,c_in,c_out,depthwise", [
    (13, 4, 1, 24, 16, 24, False),   # 2 -> 3 blocks of 8 channels
    (13, 4, 3, 24, 8, 16, False),    # the last level with one key-switching digit
    (13, 4, 4, 24, 8, 16, False),    # two digits
    (13, 3, 2, 24, 66, 11, False),   # 9 -> 2 blocks of 8 channels
    (14, 4, 1, 24, 64, 32, False),   # 4 -> 2 blocks of 16: 12 babies, 6 giants
    (14, 8, 7, 12, 128, 128, False),  # 2 -> 2 blocks of 64
    (13, 3, 9, 24, 16, 16, False),   # four digits
    (13, 4, 2, 24, 16, 16, True),    # block-diagonal: every output block reads one input
    (15, 8, 1, 60, 16, 8, False),    # 2 -> 1 blocks
])
def test_block_conv_midsize(log_n, alpha, level, w0, c_in, c_out, depthwise):
    r, rng = rig(log_n, alpha), np.random.default_rng(log_n + level)
    img = rng.uniform(-1, 1, (c_in, w0, w0))
    if depthwise:
        taps = PL.taps_depthwise(rng.uniform(-1, 1, (c_in, 3, 3)))
    else:
        taps = PL.taps_same(rng.uniform(-1, 1, (c_out, c_in, 3, 3)))
    run_parity(r, img, taps, c_in, c_out, w0, fuse=True, level=level)


def test_block_conv_without_rotations():
    r, rng = rig(13, 4), np.random.default_rng(3)
    img = rng.uniform(-1, 1, (16, 24, 24))
    run_parity(r, img, PL.taps_depthwise(rng.uniform(-1, 1, (16, 3, 3))), 16, 16, 24, fuse=False, level=2)
