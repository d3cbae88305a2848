"""The wide 3x3 convolutions on the halo GEMM kernels (forward, data gradient) and the filter-row weight
gradient, node by node against the oracle (tests/nodecheck.py, its bar for bf16: e_2 <= 2e-2), at the
sizes where their tiles are ragged or their pixel mapping changes.  One sub-network: a plain 3x3, then
two with a BN prologue (activated ahead of the kernels), so every form meets 64- and 128-column
tiles.  A network whose sizes miss the kernels runs the same check through the general ones.

The host's choice needs at least 256 tiles of 256 pixels, else 128 of 128 x 128 for the short kernel
(which applies the prologue itself); the comments give M = batch * H * W."""
import numpy as np
import pytest

from pnn_synth import nets
from tests.test_gpu_nodes import _assert, check_net

pytestmark = pytest.mark.gpu


def _net(H, W, batch, widths, seeds):
    c0, c1, c2, c3 = widths
    b = nets._SegBuilder((H, W, c0))
    s = b.conv(0, c1, 3)
    s = b.conv(s, c2, 3, preact=True)
    fine = b.done(b.conv(s, c3, 3, preact=True))
    p = nets._SegBuilder((H, W, 3))
    pre = p.done(p.conv(0, c0, 1))
    net = nets.Net(f"wide3x3-{H}x{W}-b{batch}", "bf16", batch, (H, W, 3), 10, [pre], [fine], [], c3, seeds)
    net.bn_init = "random"
    return net


@pytest.mark.parametrize("H,W,batch,widths", [
    (60, 59, 19, (64, 128, 64, 128)),     # the widest flat map; M = 67260: the last tile has 188 of 256 pixels
    (5, 7, 1900, (64, 64, 128, 64)),      # many images per tile; M = 66500: 196 pixels in the last tile
    (3, 1, 21900, (64, 64, 64, 64)),      # one-pixel rows: every side tap is padding
    (64, 80, 13, (64, 128, 192, 64)),     # 16 x 16 patches; three 64-column tiles
    (16, 176, 24, (128, 64, 128, 128)),   # patches one row of patches high
    (61, 61, 18, (64, 64, 128, 64)),      # too wide for flat tiles, no patches: the general kernels
    (9, 10, 190, (64, 128, 64, 64)),      # M = 17100: weight gradient only (under 256 tiles)
    (13, 63, 21, (128, 64, 64, 128)),     # rows of 64 with the pad: stages are whole rows
    (35, 35, 14, (128, 256, 128, 256)),   # the short kernel's widest map; M = 17150: 126 of 128 pixels in the last tile
    (36, 36, 13, (128, 256, 128, 256)),   # too wide for it
    (8, 8, 129, (256, 256, 256, 256)),    # images end inside its tiles; M = 8256: 64 pixels in the last
    (3, 1, 5462, (64, 128, 128, 256)),    # one-pixel rows; M = 16386: two pixels in the last tile
    (6, 6, 114, (512, 512, 512, 256)),    # the most channels of a prologue; 33 x 4 tiles
    (6, 6, 60, (512, 512, 512, 256)),     # 17 x 4 tiles: the split GEMM
])
def test_wide_3x3_nodes(H, W, batch, widths):
    _assert(*check_net(_net(H, W, batch, widths, (H, W, batch)), sample=384))
