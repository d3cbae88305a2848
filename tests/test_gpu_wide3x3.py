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


SIZES = [
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
]


@pytest.mark.parametrize("H,W,batch,widths", SIZES)
def test_wide_3x3_nodes(H, W, batch, widths):
    _assert(*check_net(_net(H, W, batch, widths, (H, W, batch)), sample=384))


def _taps(H, W):
    """(r, s, outputs, their inputs) of the nine taps of a 3x3 / stride 1 / pad 1 convolution."""
    for r in range(3):
        for s in range(3):
            o = (slice(None), slice(max(0, 1 - r), H - max(0, r - 1)), slice(max(0, 1 - s), W - max(0, s - 1)))
            i = (slice(None), slice(max(0, r - 1), H - max(0, 1 - r)), slice(max(0, s - 1), W - max(0, 1 - s)))
            yield r, s, o, i


def _mm(a, b):
    return (a.reshape(-1, a.shape[3]) @ b).view(*a.shape[:3], b.shape[1])


def _conv(x, w):
    y = x.new_zeros(*x.shape[:3], w.shape[0])
    for r, s, o, i in _taps(*x.shape[1:3]):
        y[o] += _mm(x[i], w[:, r, s].t().contiguous())
    return y


def _conv_t(g, w):
    d = g.new_zeros(*g.shape[:3], w.shape[3])
    for r, s, o, i in _taps(*g.shape[1:3]):
        d[i] += _mm(g[o], w[:, r, s].contiguous())
    return d


def _wgrad(x, g):
    dw = x.new_zeros(g.shape[3], 3, 3, x.shape[3])
    for r, s, o, i in _taps(*x.shape[1:3]):
        dw[:, r, s] = g[o].reshape(-1, g.shape[3]).t().contiguous() @ x[i].reshape(-1, x.shape[3])
    return dw


def _every(name, got, ref, mag, K):
    """Every element of a stored bf16 tensor against 64 bits: half an ulp (2^-8 of the value) and the fp32 sum
    of its K products (2^-24 of the sum of their magnitudes for each addition)."""
    bad = ~((got - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -24 * mag)
    assert not bad.any(), (name, int(bad.sum()), bad.nonzero()[:4].tolist())


@pytest.mark.parametrize("H,W,batch,widths", SIZES)
def test_wide_3x3_every_element(H, W, batch, widths):
    """All of the three layers' outputs, data gradients and weight gradients, each from the inputs that the GPU
    itself stored: the pixels at the edges of images, patches and the last tile among them."""
    import torch
    import pnn_synth as S
    from tests.test_gpu_nodes import gpu_step
    net = _net(H, W, batch, widths, (H, W, batch))
    x, labels, params = S.make_all(net)
    g, dx_fine = gpu_step(net, params, x, labels)
    seg = net.fine[0]

    def ws(buf, what, k, c):
        off = g.plan.inspect(1, 0, what, k)
        return buf[off:off + batch * H * W * c * 2].view(torch.bfloat16).view(batch, H, W, c).double()

    shape = lambda t, c: t.view(batch, H, W, c).double()
    value = [shape(g.x[0], widths[0]), ws(g.saved, 0, 1, widths[1]), ws(g.saved, 0, 2, widths[2]),
             shape(g.y[0], widths[3])]
    grad = [shape(dx_fine[0], widths[0]), ws(g.scratch, 1, 1, widths[1]), ws(g.scratch, 1, 2, widths[2]),
            shape(g.D[0], widths[3])]
    grads = g.unpack_grads(1, 0)
    for i, n in enumerate(seg.nodes):
        assert (n.src, n.dst) == (i, i + 1)
        w = torch.from_numpy(np.asarray(params["fine"][0]["conv"][i], dtype=np.float64)).cuda()
        a, z = value[i], None
        if n.bn >= 0:
            off = g.plan.inspect(1, 0, 3, n.bn)
            st = g.saved[off:off + 16 * widths[i]].view(torch.float32).view(4, widths[i]).double()
            # the stored value's fused multiply-add with the stored scale and shift: one rounding to fp32, one to bf16
            z = (a * st[2] + st[3]).float()
            a = torch.relu(z).to(torch.bfloat16).double()
            margin = 2.0 ** -20 * ((value[i] * st[2]).abs() + st[3].abs())
        K = 9 * widths[i]
        _every(f"forward {i}", value[i + 1], _conv(a, w), _conv(a.abs(), w.abs()), K)
        K = 9 * widths[i + 1]
        got = grad[0] if i == 0 else ws(g.scratch, 2, n.bn, widths[i])
        ref, mag = _conv_t(grad[i + 1], w), _conv_t(grad[i + 1].abs(), w.abs())
        if z is not None:
            ref = ref * (z > 0)
            edge = z.abs().double() <= margin            # (at the mask's edge either value is right)
            got = torch.where(edge, ref, got)
        _every(f"data gradient {i}", got, ref, mag, K)
        ref = _wgrad(a, grad[i + 1])
        err = (torch.from_numpy(grads["conv"][i]).cuda() - ref).norm() / ref.norm()
        # fp32 sums over M pixels, 32 to an addition.  (A pixel left out is 1 / sqrt(M) >= 3.8e-3.)
        assert err <= max(1.0, batch * H * W / 32) * 2.0 ** -24 + 1e-6, (f"weight gradient {i}", float(err))
    g.plan.close()


@pytest.mark.parametrize("H,W,cin,cout,batches", [
    (40, 40, 128, 128, (11, 41)),       # gemm_conv_kernel (138 of its tiles), halo GEMM (257 of its own)
    (40, 40, 256, 128, (11, 41)),       # the order of the channel chunks
    (40, 40, 64, 64, (21, 41)),         # 64 columns
    (40, 40, 128, 64, (21, 41)),
    (16, 16, 128, 256, (64, 257)),      # short halo GEMM, halo GEMM
])
def test_wide_3x3_same_bits_whichever_kernel(H, W, cin, cout, batches):
    """An image's output and data gradient do not depend on the batch it is in, where the batch chooses the kernel
    (unsplit): the kernels add the products in one order."""
    import torch
    import pnn_synth as S
    from paper_2103_08802_amd import binding as B
    from paper_2103_08802_amd.step import ParaRealGPU
    out = []
    for batch in batches:
        b = nets._SegBuilder((H, W, cin))
        fine = b.done(b.conv(0, cout, 3))
        p = nets._SegBuilder((H, W, 3))
        net = nets.Net("wide3x3-bits", "bf16", batch, (H, W, 3), 10, [p.done(p.conv(0, cin, 1))], [fine], [], cout,
                       (1, 2, 3))
        g = ParaRealGPU(net, S.make_all(net)[2])
        gen = torch.Generator(device="cuda").manual_seed(H * W + cin)
        draw = lambda c: torch.stack([torch.randn(H, W, c, generator=gen, device="cuda") for _ in range(batch)])
        g.x[0].copy_(draw(cin))
        gen.manual_seed(H * W + cout)
        g.D[0].copy_(draw(cout))
        B.parareal_fine_fwd(g.plan, g.x, g.phi, g.y, g.saved, g.scratch, g.stream())
        B.parareal_fine_bwd(g.plan, g.D, g.x, g.phi, g.saved, g.dx, g.dphi, g.scratch, g.stream())
        torch.cuda.synchronize()
        out.append((g.y[0][:batches[0]].clone(), g.dx[0][:batches[0]].clone()))
        g.plan.close()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])
