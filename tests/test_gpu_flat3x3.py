"""The flat tiles of narrow 3x3 convolutions (forward and data gradient: maps whose rows do not divide a tile,
and fp32), node by node against the oracle (tests/nodecheck.py and its bars), where their pixel mapping,
LDS layout or tile height changes; and next to them the sizes that stay with the halo and gathered
kernels.  One sub-network: a plain 3x3, then two with a BN prologue."""
import pytest

from pnn_synth import nets
from tests.test_gpu_nodes import _assert, check_net

pytestmark = pytest.mark.gpu


def _net(H, W, batch, widths, dtype):
    c0, c1, c2, c3 = widths
    b = nets._SegBuilder((H, W, c0))
    s = b.conv(0, c1, 3)
    s = b.conv(s, c2, 3, preact=True)
    fine = b.done(b.conv(s, c3, 3, preact=True))
    p = nets._SegBuilder((H, W, 3))
    pre = p.done(p.conv(0, c0, 1))
    net = nets.Net(f"flat3x3-{H}x{W}-b{batch}-{dtype}", dtype, batch, (H, W, 3), 10, [pre], [fine], [], c3,
                   (H, W, batch))
    net.bn_init = "random"
    return net


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,W,batch,widths", [
    (7, 5, 3, (16, 16, 32, 16)),        # 105 pixels: short tiles, the only one ragged
    (9, 13, 41, (16, 32, 64, 32)),      # images end inside tiles; short tiles
    (10, 10, 370, (32, 64, 32, 64)),    # 37000 pixels: tall 32-column tiles, 64 ragged
    (40, 40, 37, (16, 16, 16, 16)),     # tall 16-column tiles
    (1, 37, 30, (16, 32, 16, 64)),      # one-row images
    (21, 1, 40, (64, 16, 32, 16)),      # one-pixel rows
    (6, 64, 50, (16, 16, 32, 16)),      # fp32: 16 channels at the even chunk stride
    (4, 310, 9, (16, 64, 16, 32)),      # too wide for the flat tiles of most layers
    (32, 32, 4, (16, 16, 16, 16)),      # the halo tile's maps: bf16 stays there
    (5, 6, 20, (48, 80, 48, 16)),       # channel counts off the powers of two
])
def test_flat_3x3_nodes(H, W, batch, widths, dtype):
    _assert(*check_net(_net(H, W, batch, widths, dtype)))
