"""The head (pnn_head_fwd_bwd) over the sizes where its batch-tiled kernels and the per-sample kernel
meet and where their tiles are ragged (16 samples, 16 / 64 classes, 32 / 64 channels), against the
oracle's head.  Bounds: the logits sum C <= 512 products in fp32 (relative rounding 2^-24 each, a few
of them in a row), the gradients likewise over K or the batch: 1e-6 of the largest value; D_N of a
bf16 network is rounded once (half an ulp: 2^-8 of the value, here of the largest)."""
import numpy as np
import pytest

from pnn_synth import nets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,hw,C,K", [
    (1, 1, 16, 255),        # per-sample kernel: W just under the line
    (1, 1, 16, 256),        # batch-tiled: one tile in every direction but the classes
    (17, 3, 272, 65),       # one past a tile in samples, channels and classes
    (16, 2, 48, 1000),      # 48 channels: half a channel tile
    (33, 7, 512, 1000),
    (3, 5, 528, 4096),      # the largest class count
    (5, 2, 24, 300),        # channels off the tile: per-sample kernel
])
def test_head_sizes(B, hw, C, K, dtype):
    import torch
    from oracle.net import ParaRealOracle
    from paper_2103_08802_amd import binding as bind
    C2 = C if C % 16 == 0 else 48
    net = nets.Net("head", dtype, B, (hw, hw, C2), K, [nets.Segment((hw, hw, C2))],
                   [nets.Segment((hw, hw, C2), [nets.Node("conv", 0, 1, k=1, cout=C2)], [], 1)], [], C2, (1, 2, 3))
    if C % 16 != 0:         # identity sub-network: any channel count
        net.in_shape = (hw, hw, C)
        net.pre = [nets.Segment((hw, hw, C))]
        net.fine = [nets.Segment((hw, hw, C))]
        net.head_cin = C
    p = bind.Plan(net)
    rng = np.random.default_rng(B * 1000 + K)
    sdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    yt = torch.from_numpy(rng.standard_normal((B, hw, hw, C)).astype(np.float32)).cuda().to(sdt)
    w = (rng.standard_normal((K, C)) * np.sqrt(2.0 / C)).astype(np.float32)
    b = (0.1 * rng.standard_normal(K)).astype(np.float32)
    labels = rng.integers(0, K, B).astype(np.int32)
    eps = torch.from_numpy(np.concatenate([w.ravel(), b])).cuda()
    f32 = dict(dtype=torch.float32, device="cuda")
    logits, loss = torch.full((B, K), 7.0, **f32), torch.full((1,), 7.0, **f32)
    D, deps = torch.full_like(yt, 7.0), torch.full((K * C + K,), 7.0, **f32)
    scratch = torch.zeros(p.workspace_size(bind.PNN_WS_SCRATCH), dtype=torch.uint8, device="cuda")
    bind.pnn_head_fwd_bwd(p, yt, eps, torch.from_numpy(labels).cuda(), logits, loss, D, deps, scratch,
                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    o = ParaRealOracle(net, {"head": {"w": w.astype(np.float64), "b": b.astype(np.float64)}}, bf16=False)
    ref = o.head(yt.float().cpu().numpy().astype(np.float64), labels)
    err = lambda a, r: np.abs(a - r).max() / np.abs(r).max()
    g = deps.cpu().numpy().astype(np.float64)
    assert err(logits.cpu().numpy(), ref["logits"]) <= 1e-6
    assert abs(loss.item() - ref["loss"]) <= 1e-6 * abs(ref["loss"]) + 1e-7
    assert err(g[:K * C].reshape(K, C), ref["dw"]) <= 1e-6
    assert err(g[K * C:], ref["db"]) <= 1e-6
    assert err(D.float().cpu().numpy(), ref["D_N"]) <= (2.0 ** -8 if dtype == "bf16" else 1e-6)
    p.close()
