"""Performance cases: what a user of this library runs, through its public entry points.

Three networks carry the library: the tiny fp32 network, VGG-16 (Table vgg) and the pre-activation
ResNet-1001 (Table resnet), torn into N sub-networks.  A training program calls whole steps; the
calls inside a step are entry points of their own (fine sub-networks, coarse chain, head, SGD), and
those are what most cases time, on networks of the same layers but few of them in a row: rounding
differences grow through dozens of BN / ReLU layers until the deep gradients of two correct
implementations have little in common, while a residual unit or a VGG block can be compared.

Kinds (``kind``):

* ``step``    forward, loss and backward of a whole network; bf16 networks then take the SGD step
              and return the updated weights, the fp32 network returns its gradients
* ``fine``    ``parareal_fine_fwd`` + ``parareal_fine_bwd``
* ``coarse``  every block's ``coarse_fwd`` and ``coarse_bwd`` (the chains over all blocks are in ``step``)
* ``head``    ``pnn_head_fwd_bwd``
* ``sgd``     ``pnn_sgd_step`` over the fine sub-networks' parameters, with fp32 master weights

``exact`` evaluates the same definitions in plain torch, in 64 bits: convolutions as one matrix
product per filter tap, everything else by autograd.  A bf16 network's stored tensors are bf16 by
definition (every layer output, every activation that feeds a matrix product, their gradients), so
those are rounded once where the interface stores them; all arithmetic between stays in 64 bits.
"""
import math

import torch

from paper_2103_08802_amd import binding as B
from paper_2103_08802_amd.step import ParaRealGPU
from pnn_synth import nets
from pnn_synth.gen import segment_shapes

DEV = "cuda"
LR, MU, WD = 1e-3, 0.9, 1e-4      # the first steps of a warm-up; momentum and weight decay of the ResNet runs


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------

VGG_BLOCKS = [[[64]], [[128, 128]], [[256, 256]], [[512, 512]], [[512, 512]]]   # one block per sub-network


def _fine_resnet(hw, batch, n_sub, dtype="bf16"):
    # one residual unit per sub-network, n_sub / 3 of them per stage
    return {"kind": "fine", "net": "resnet", "hw": hw, "batch": batch, "n_sub": n_sub, "units": n_sub // 3,
            "dtype": dtype, "coarse": "config", "classes": 100}


def _fine_vgg(hw, batch):
    return {"kind": "fine", "net": "vgg_blocks", "hw": hw, "batch": batch, "n_sub": len(VGG_BLOCKS), "units": 0,
            "dtype": "bf16", "coarse": "config", "classes": 10}


def _coarse(hw, batch, n_sub, coarse):
    # three residual units per sub-network: the interfaces X_j of the contiguous split
    return {"kind": "coarse", "net": "resnet", "hw": hw, "batch": batch, "n_sub": n_sub, "units": n_sub,
            "dtype": "bf16", "coarse": coarse, "classes": 100}


def _head(batch, hw, c, classes, dtype="bf16"):
    return {"kind": "head", "net": "head", "hw": hw, "batch": batch, "n_sub": 1, "units": c, "dtype": dtype,
            "coarse": "config", "classes": classes}


def _step(net, hw, batch, n_sub, units, classes, dtype, coarse="config"):
    return {"kind": "step", "net": net, "hw": hw, "batch": batch, "n_sub": n_sub, "units": units, "dtype": dtype,
            "coarse": coarse, "classes": classes}


def listed():
    def named(name, c):
        return {"name": name, **c}
    return [
        # the smallest call: one training step of the fp32 network (launch latency and host work)
        named("tiny_f32_step", _step("tiny", 32, 4, 2, 0, 10, "f32")),
        # one training step of the CIFAR-shaped VGG-16 in four sub-networks
        named("vgg16_step", _step("vgg", 32, 128, 4, 0, 10, "bf16")),
        # one training step of ResNet-1001 in sixteen sub-networks, the benchmark's workload
        named("resnet1001_step", _step("resnet", 32, 128, 16, 111, 100, "bf16")),
        # that workload's fine sub-networks at a depth level: five residual units per stage
        named("resnet_fine_32px", _fine_resnet(32, 128, 15)),
        # the 64x64-input form's units: the largest ResNet tensors
        named("resnet_fine_64px", _fine_resnet(64, 128, 9)),
        # an odd batch on maps that are no power of two, a sub-network per stage
        named("resnet_fine_ragged", _fine_resnet(40, 37, 3)),
        # the fp32 storage type
        named("resnet_fine_f32", _fine_resnet(32, 64, 6, "f32")),
        # VGG layers at ImageNet's resolution and the full batch, a block per sub-network: the largest
        named("vgg_fine_224px", _fine_vgg(224, 128)),
        # the same layers on a small odd batch of smaller images
        named("vgg_fine_96px", _fine_vgg(96, 9)),
        # the coarse blocks of the sixteen-way split (one bottleneck per interface), one call each
        named("coarse_blocks", _coarse(32, 128, 16, "config")),
        # the paper's own coarse blocks (two-3x3 residual units)
        named("coarse_paper", _coarse(32, 128, 12, "paper")),
        # the ImageNet-shaped head
        named("head_1000", _head(128, 7, 512, 1000)),
    ]


def _even(n_sub, units):
    """The sub-networks of the contiguous split into at most n_sub that all get a unit."""
    total = 3 * units
    return math.ceil(total / math.ceil(total / n_sub))


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["resnet", "resnet", "resnet", "vgg", "vgg", "coarse", "head", "tiny", "sgd"])
    if kind == "resnet":
        return _fine_resnet(4 * rng.randint(4, 16), _logint(rng, 2, 128), 3 * rng.randint(1, 6),
                            rng.choice(["bf16", "bf16", "bf16", "f32"]))
    if kind == "vgg":
        hw = 32 * rng.randint(1, 7)
        return _fine_vgg(hw, _logint(rng, 2, 128))
    if kind == "coarse":
        coarse = rng.choice(["config", "paper"])   # (paper: one residual unit per block from N = 12 on)
        return _coarse(4 * rng.randint(4, 12), _logint(rng, 4, 128), rng.randint(2 if coarse == "config" else 12, 16),
                       coarse)
    if kind == "head":
        return _head(_logint(rng, 1, 256), rng.randint(1, 16), 16 * rng.randint(1, 32), _logint(rng, 2, 1000),
                     rng.choice(["bf16", "bf16", "f32"]))
    if kind == "tiny":
        return _step("tiny", 4 * rng.randint(2, 16), _logint(rng, 1, 64), rng.randint(1, 4), 0, 10, "f32")
    if rng.random() < 0.5:
        return {**_step("vgg", 32, 128, 4, 0, 10, "bf16"), "kind": "sgd"}
    units = rng.randint(8, 111)
    return {**_step("resnet", 32, 16, _even(rng.randint(3, 16), units), units, 100, "bf16"), "kind": "sgd"}


# ------------------------------------------------------------------------------------------------
# networks, parameters and inputs (from the seed alone)
# ------------------------------------------------------------------------------------------------

def _net(case):
    hw, batch, n_sub, dtype = case["hw"], case["batch"], case["n_sub"], case["dtype"]
    if case["net"] == "tiny":
        return nets.tiny_parareal("tiny", batch, hw, 16, n_sub, case["classes"], dtype)
    if case["net"] == "vgg":
        return nets.vgg_parareal("vgg", batch, hw, case["classes"], dtype, (1, 2, 3), coarse=case["coarse"])
    if case["net"] == "vgg_blocks":
        return nets.vgg_parareal("vgg", batch, hw, case["classes"], dtype, (1, 2, 3), split=VGG_BLOCKS)
    if case["net"] == "head":
        shape = (hw, hw, case["units"])
        one = nets.Segment(shape, [nets.Node("conv", 0, 1, k=1, cout=case["units"])], [], 1)
        return nets.Net("head", dtype, batch, shape, case["classes"], [nets.Segment(shape)], [one], [], case["units"],
                        (1, 2, 3))
    per_stage = case["kind"] == "fine" and n_sub % 3 == 0 and case["units"] % (n_sub // 3) == 0
    return nets.resnet_parareal("resnet", batch, hw, n_sub, case["classes"], dtype, (1, 2, 3), coarse=case["coarse"],
                                units_per_stage=case["units"],
                                partition="per_stage" if per_stage else "contiguous")


def _align(n):
    return (n + 255) & ~255


def _layout(seg, es):
    """Byte offsets of the filters (None without one) and of the (gamma | beta) pairs in a parameter
    buffer (es: bytes of a filter element) or a gradient buffer (es = 4), and the buffer's size."""
    sh, at, conv, bn = segment_shapes(seg), 0, [], []
    for n in seg.nodes:
        if n.op != "conv":
            conv.append(None)
            continue
        conv.append(at)
        at = _align(at + n.cout * n.k * n.k * sh[n.src][2] * es)
    for s in seg.bns:
        bn.append(at)
        at = _align(at + sh[s][2] * 8)
    return conv, bn, at


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + 17)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)


def _params(case, net, g):
    """Per part and segment: [filters (storage type)], [(gamma, beta)].  A training step starts from
    gamma = 1, beta = 0; the single calls get parameters that training has moved."""
    sdt = torch.bfloat16 if net.dtype == "bf16" else torch.float32
    trained = case["kind"] != "step"
    parts = []
    for segs in (net.pre, net.fine, net.coarse):
        out = []
        for seg in segs:
            sh, conv, bn = segment_shapes(seg), [], []
            for n in seg.nodes:
                if n.op != "conv":
                    conv.append(None)
                    continue
                cin = sh[n.src][2]
                conv.append((_randn(g, n.cout, n.k, n.k, cin) * math.sqrt(2.0 / (cin * n.k * n.k))).to(sdt))
            for s in seg.bns:
                c = sh[s][2]
                if trained:
                    bn.append((torch.rand(c, generator=g, device=DEV) + 0.5, 0.2 * _randn(g, c)))
                else:
                    bn.append((torch.ones(c, device=DEV), torch.zeros(c, device=DEV)))
            out.append((conv, bn))
        parts.append(out)
    c, k = net.head_cin, net.classes
    head = torch.cat([(_randn(g, k, c) * math.sqrt(2.0 / c)).reshape(-1), 0.1 * _randn(g, k) * float(trained)])
    return parts, head


def _inputs(case, net, seed):
    """Everything a call reads, from the seed: parameters, then the tensors of the case's kind."""
    g = _gen(seed)
    sdt = torch.bfloat16 if net.dtype == "bf16" else torch.float32
    bt, kind = case["batch"], case["kind"]
    parts, head = _params(case, net, g)
    inp = {"parts": parts, "head": head}

    def act(shape, scale=1.0):
        return (scale * _randn(g, bt, *shape)).to(sdt)

    xs = [tuple(s.in_shape) for s in net.fine]
    ys = [segment_shapes(s)[s.out] for s in net.fine]
    if kind == "step":
        inp["image"] = act(net.in_shape)
    if kind == "fine":
        # the residual stream deep in a stage (a unit adds about 1 to its variance)
        inp["x"] = [act(s, 8.0) for s in xs]
        if net.fine[0].nodes[0].bn < 0:        # VGG: sub-networks read activations
            inp["x"] = [torch.relu(x) for x in inp["x"]]
        inp["dy"] = [act(s, 1e-3) for s in ys]
    if kind == "coarse":
        inp["rt"] = [act(s, 8.0) for s in ys[:-1]]
        inp["add"] = [act(s) for s in ys[1:]]
        inp["d"] = [act(s, 1e-3) for s in ys[1:]]
    if kind == "head":
        inp["ytilde"] = act(ys[-1])
    if kind in ("step", "head"):
        inp["labels"] = torch.randint(0, net.classes, (bt,), generator=g, device=DEV, dtype=torch.int32)
    if kind == "sgd":
        inp["grads"] = [_randn(g, _layout(s, 4)[2] // 4) * 1e-2 for s in net.fine]
        inp["mom"] = [_randn(g, _layout(s, 4)[2] // 4) * 1e-2 for s in net.fine]
    return inp


def _put(buf, seg, prm, es):
    conv, bn, _ = _layout(seg, es)
    for o, w in zip(conv, prm[0]):
        if o is not None:
            buf[o:o + w.numel() * w.element_size()] = w.reshape(-1).view(torch.uint8)
    for o, (ga, be) in zip(bn, prm[1]):
        buf[o:o + 8 * ga.numel()] = torch.cat([ga, be]).view(torch.uint8)


def _flat(bufs):
    """The buffers as views of one allocation (what an optimiser keeps its state in)."""
    flat = torch.zeros(sum(b.numel() for b in bufs), dtype=torch.uint8, device=DEV)
    out, at = [], 0
    for b in bufs:
        out.append(flat[at:at + b.numel()])
        at += b.numel()
    return flat, out


def _bn_tail(buf, seg, es):
    """The BN parameters of a parameter buffer, as floats."""
    _, bn, tot = _layout(seg, es)
    return buf[bn[0]:tot].view(torch.float32) if bn else None


class _State:
    pass


def prepare(case, seed):
    net = _net(case)
    inp = _inputs(case, net, seed)
    es = 2 if net.dtype == "bf16" else 4
    g = ParaRealGPU(net)
    g.overlap_bwd = True
    for bufs, segs, prm in zip((g.delta, g.phi, g.eta), (net.pre, net.fine, net.coarse), inp["parts"]):
        for b, seg, p in zip(bufs, segs, prm):
            _put(b, seg, p, es)
    g.eps.copy_(inp["head"])
    s = _State()
    s.kind, s.g, s.net = case["kind"], g, net
    n = net.n_sub
    if s.kind == "step":
        g.image.copy_(inp["image"])
        g.labels.copy_(inp["labels"])
        if es == 2:
            g.sgd_init()
            s.flat = []
            for part in range(3):
                if g.master[part]:
                    flat, g.master[part] = _flat(g.master[part])
                    s.flat.append(flat.view(torch.float32))
            s.out = {"logits": g.logits, "loss": g.loss, "master": s.flat, "head": g.eps,
                     "bn": [t for bufs, segs in ((g.phi, net.fine), (g.eta, net.coarse), (g.delta, net.pre))
                            for b, seg in zip(bufs, segs) for t in [_bn_tail(b, seg, es)] if t is not None]}
        else:
            s.out = {"logits": g.logits, "loss": g.loss, "ytilde": g.ytilde, "dx": g.dx, "head": g.deps,
                     "grads": [b.view(torch.float32) for b in g.ddelta + g.dphi + g.deta]}
    elif s.kind == "fine":
        for a, b in zip(g.x + g.D, inp["x"] + inp["dy"]):
            a.copy_(b)
        s.out = {"y": g.y, "dx": g.dx, "dphi": [b.view(torch.float32) for b in g.dphi]}
    elif s.kind == "coarse":
        s.rt, s.add, s.d = inp["rt"], inp["add"], inp["d"]
        s.out = {"rt": g.rt[1:] + [g.ytilde], "d": g.D[:n - 1], "deta": [b.view(torch.float32) for b in g.deta]}
    elif s.kind == "head":
        g.y[0].copy_(inp["ytilde"])
        g.labels.copy_(inp["labels"])
        s.out = {"logits": g.logits, "loss": g.loss, "d": g.D[0], "deps": g.deps}
    else:
        g.sgd_init()
        for a, b in zip(g.dphi + g.mom[1], inp["grads"] + inp["mom"]):
            a.view(torch.float32).copy_(b)
        flat, g.master[1] = _flat(g.master[1])
        s.out = {"master": flat.view(torch.float32), "mom": [m.view(torch.float32) for m in g.mom[1]],
                 "bn": [t for b, seg in zip(g.phi, net.fine) for t in [_bn_tail(b, seg, es)] if t is not None]}
    s.fresh = True
    return s


def run(state):
    g = state.g
    p, st = g.plan, g.stream()
    if state.kind == "step":
        g.step(st)
        if g.net.dtype == "bf16":
            g.sgd_step(LR, MU, WD, s=st)
    elif state.kind == "fine":
        B.parareal_fine_fwd(p, g.x, g.phi, g.y, g.saved, g.scratch, st)
        B.parareal_fine_bwd(p, g.D, g.x, g.phi, g.saved, g.dx, g.dphi, g.scratch, st)
    elif state.kind == "coarse":
        rt, d = state.out["rt"], state.out["d"]
        for j in range(len(rt)):
            B.coarse_fwd(p, j, state.rt[j], g.eta[j], state.add[j], rt[j], g.saved, g.scratch, st)
        for j in range(len(rt) - 1, -1, -1):
            B.coarse_bwd(p, j, state.d[j], state.rt[j], g.eta[j], g.saved, d[j], g.deta[j], g.scratch, st)
    elif state.kind == "head":
        B.pnn_head_fwd_bwd(p, g.ytilde, g.eps, g.labels, g.logits, g.loss, g.D[0], g.deps, g.scratch, st)
    else:
        B.pnn_sgd_step(p, 1, g.phi, g.dphi, g.mom[1], LR, MU, WD, True, st, master=g.master[1],
                       master_init=state.fresh)
        state.fresh = False
    return state.out


# ------------------------------------------------------------------------------------------------
# work and tolerances
# ------------------------------------------------------------------------------------------------

def _segment_work(seg, batch, es, part):
    """(bytes, flops) of one segment's forward and backward.  BN with batch statistics separates any
    two layers, so each layer's tensors count once per direction: forward input and output, backward
    output gradient, input and (where wanted) input gradient."""
    sh = segment_shapes(seg)
    by = fl = 0.0

    def size(shape):
        return batch * shape[0] * shape[1] * shape[2] * es

    for n in seg.nodes:
        i, o = size(sh[n.src]), size(sh[n.dst])
        dgrad = part != 0 or n.src != 0
        by += (i + o) + (o + i + (i if dgrad else 0)) * (n.op != "maxpool3")
        if n.op == "conv":
            w = n.cout * n.k * n.k * sh[n.src][2]
            by += 2 * w * es + 4 * w
            fl += 2.0 * batch * sh[n.dst][0] * sh[n.dst][1] * w * (3 if dgrad else 2)
    return by, fl


def work(case):
    net = _net(case)
    es = 2 if net.dtype == "bf16" else 4
    bt, kind = case["batch"], case["kind"]
    by = fl = 0.0
    ys = [segment_shapes(s)[s.out] for s in net.fine]
    parts = {"step": (net.pre, net.fine, net.coarse), "fine": ((), net.fine, ()), "coarse": ((), (), net.coarse)}
    for part, segs in enumerate(parts.get(kind, ())):
        for seg in segs:
            b, f = _segment_work(seg, bt, es, part)
            by, fl = by + b, fl + f
    if kind in ("step", "head"):
        h, w, c = ys[-1]
        by += 2.0 * bt * h * w * c * es + 8.0 * net.classes * (c + 1)
        fl += 6.0 * bt * c * net.classes + 2.0 * bt * h * w * c
    if kind == "step":       # the combine's differences, both directions
        by += sum(6.0 * bt * h * w * c * es for h, w, c in ys[:-1])
    if kind in ("step", "sgd") and es == 2:   # weight, master, momentum read and written, gradient read
        n = sum(sum(m.cout * m.k * m.k * segment_shapes(s)[m.src][2] for m in s.nodes if m.op == "conv")
                for part in (parts.get(kind) or ((), net.fine, ())) for s in part)
        by += 22.0 * n
        fl += 8.0 * n
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """Measured against ``exact`` and against the library's own paths that sum in another order.  A
    ReLU mask or a pooling choice that flips where rounding moves a value across its edge changes
    that element's gradient by its whole size, so "max" is of the order of a value in every kind
    that has one (fp32: 1e-7 without a flip, 1e-3 with one)."""
    if case["kind"] == "sgd":
        return {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "head":          # (f32: no rounded operand; bf16: the stored gradient)
        return {"rel": 2e-6, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 4e-3, "max": 2e-2}
    if case["dtype"] == "f32":
        return {"rel": 5e-3, "max": 0.9}
    if case["kind"] == "step":          # logits 2e-3, and 2e-2 on the second of two steps; weights 3e-4
        return {"rel": 3e-2, "max": 0.3}
    return {"rel": 3e-2, "max": 0.9}    # a residual unit, two VGG layers or a coarse block: 3e-3 .. 1e-2


# ------------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------------

def _taps(x, k, stride, pad, ho, wo):
    if pad:
        x = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    for r in range(k):
        for c in range(k):
            yield r, c, x[:, r:r + (ho - 1) * stride + 1:stride, c:c + (wo - 1) * stride + 1:stride]


class _Conv(torch.autograd.Function):
    """Cross-correlation of NHWC x with w [c_out][k][k][c_in], one matrix product per filter tap."""

    @staticmethod
    def forward(ctx, x, w, stride, pad):
        ctx.save_for_backward(x, w)
        ctx.geom = stride, pad
        k = w.shape[1]
        ho, wo = (x.shape[1] + 2 * pad - k) // stride + 1, (x.shape[2] + 2 * pad - k) // stride + 1
        y = None
        for r, c, t in _taps(x, k, stride, pad, ho, wo):
            z = t.reshape(-1, t.shape[3]) @ w[:, r, c].t().contiguous()
            y = z if y is None else y.add_(z)
        return y.view(x.shape[0], ho, wo, w.shape[0])

    @staticmethod
    def backward(ctx, g):
        x, w = ctx.saved_tensors
        stride, pad = ctx.geom
        k, ho, wo = w.shape[1], g.shape[1], g.shape[2]
        g2 = g.reshape(-1, g.shape[3])
        dx = torch.zeros(x.shape[0], x.shape[1] + 2 * pad, x.shape[2] + 2 * pad, x.shape[3], dtype=x.dtype,
                         device=x.device)
        dw = torch.empty_like(w)
        for r, c, t in _taps(x, k, stride, pad, ho, wo):
            dw[:, r, c] = g2.t().contiguous() @ t.reshape(-1, t.shape[3])
            if ctx.needs_input_grad[0]:
                dx[:, r:r + (ho - 1) * stride + 1:stride, c:c + (wo - 1) * stride + 1:stride] += \
                    (g2 @ w[:, r, c].contiguous()).view(t.shape)
        return dx[:, pad:dx.shape[1] - pad, pad:dx.shape[2] - pad], dw, None, None


class _Store(torch.autograd.Function):
    """A tensor of a bf16 network as it is stored: the value and / or its gradient rounded to bf16."""

    @staticmethod
    def forward(ctx, x, value, grad):
        ctx.grad = grad
        return x.to(torch.bfloat16).double() if value else x.clone()

    @staticmethod
    def backward(ctx, g):
        return g.to(torch.bfloat16).double() if ctx.grad else g, None, None


def _stored(x, bf16, value=True, grad=True):
    return _Store.apply(x, value, grad) if bf16 else x


def _bn_relu(x, ga, be):
    m = x.mean((0, 1, 2))
    v = (x - m).square().mean((0, 1, 2))
    return torch.relu((x - m) * torch.rsqrt(v + 1e-5) * ga + be)


def _pool(x, k, stride, pad):
    return torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), k, stride, pad).permute(0, 2, 3, 1)


def _segment(seg, prm, x, bf16, add=None):
    slots, acts = {0: _stored(x, bf16)}, {}
    for n, w in zip(seg.nodes, prm[0]):
        s = slots[n.src]
        if n.bn >= 0:
            if n.bn not in acts:
                acts[n.bn] = _stored(_bn_relu(s, *prm[1][n.bn]), bf16, value=False)
            s = acts[n.bn]
        if n.op == "conv":
            s = _Conv.apply(_stored(s, bf16, grad=False), w, n.stride, n.pad)
        elif n.op == "maxpool3":
            s = _pool(s, 3, 2, 1)
        elif n.pool == 2:
            s = _pool(s, 2, 2, 0)
        if n.res >= 0:
            s = s + slots[n.res]
        if add is not None and n.dst == seg.out:
            s = s + add
        slots[n.dst] = _stored(s, bf16)
    return slots[seg.out]


def _double(prm):
    return ([None if w is None else w.double().requires_grad_() for w in prm[0]],
            [(a.double().requires_grad_(), b.double().requires_grad_()) for a, b in prm[1]])


def _grad_buffer(seg, prm, values=lambda t: t.grad):
    conv, bn, tot = _layout(seg, 4)
    buf = torch.zeros(max(tot, 256) // 4, dtype=torch.float64, device=DEV)
    for o, w in zip(conv, prm[0]):
        if o is not None:
            buf[o // 4:o // 4 + w.numel()] = values(w).reshape(-1)
    for o, (a, b) in zip(bn, prm[1]):
        buf[o // 4:o // 4 + 2 * a.numel()] = torch.cat([values(a), values(b)])
    return buf


def _sgd(w, d, v=None):
    d = d + WD * w
    v = d if v is None else MU * v + d
    return w - LR * (d + MU * v), v


def _master(seg, prm, new):
    """Updated filters laid out like a gradient buffer (BN entries stay zero), updated BN tail."""
    filters = (prm[0], [])
    buf = _grad_buffer(seg, filters, new)
    full = torch.zeros(max(_layout(seg, 4)[2], 256) // 4, dtype=torch.float64, device=DEV)
    full[:buf.numel()] = buf[:full.numel()]
    conv, bn, tot = _layout(seg, 2)
    if not bn:
        return full, None
    tail = torch.zeros((tot - bn[0]) // 4, dtype=torch.float64, device=DEV)
    for o, (a, b) in zip(bn, prm[1]):
        at = (o - bn[0]) // 4
        tail[at:at + 2 * a.numel()] = torch.cat([new(a), new(b)])
    return full, tail


def _head64(y, eps, labels, classes):
    c = y.shape[3]
    w, b = eps[:classes * c].view(classes, c), eps[classes * c:]
    logits = y.mean((1, 2)) @ w.t() + b
    return logits, torch.nn.functional.cross_entropy(logits, labels.long())


def exact(case, seed):
    if case["kind"] == "step" and case["units"] > 32:
        return None                        # (about 25 s)
    net = _net(case)
    inp = _inputs(case, net, seed)
    kind, n, bf16 = case["kind"], net.n_sub, net.dtype == "bf16"
    if kind == "sgd":
        flat, mom, tails = [], [], []
        for seg, prm, gr, mo in zip(net.fine, inp["parts"][1], inp["grads"], inp["mom"]):
            conv, bn, tot = _layout(seg, 4)
            gr, mo = gr.double(), mo.double()
            new_v = mo.clone()
            master = torch.zeros(max(tot, 256) // 4, dtype=torch.float64, device=DEV)
            _, bn2, tot2 = _layout(seg, 2)
            tail = torch.zeros((tot2 - bn2[0]) // 4 if bn2 else 0, dtype=torch.float64, device=DEV)
            for o, w in zip(conv, prm[0]):
                if o is not None:
                    a, b = o // 4, o // 4 + w.numel()
                    master[a:b], new_v[a:b] = _sgd(w.double().reshape(-1), gr[a:b], mo[a:b])
            for o, o2, (ga, be) in zip(bn, bn2, prm[1]):
                a, b, t = o // 4, o // 4 + 2 * ga.numel(), (o2 - bn2[0]) // 4
                tail[t:t + b - a], new_v[a:b] = _sgd(torch.cat([ga, be]).double(), gr[a:b], mo[a:b])
            flat.append(master)
            mom.append(new_v)
            tails += [tail] if bn2 else []
        return {"master": torch.cat(flat), "mom": mom, "bn": tails}
    if kind == "head":
        y = inp["ytilde"].double().requires_grad_()
        eps = inp["head"].double().requires_grad_()
        logits, loss = _head64(y, eps, inp["labels"], net.classes)
        loss.backward()
        return {"logits": logits.detach(), "loss": loss.detach().view(1), "d": y.grad.contiguous(), "deps": eps.grad}
    if kind == "fine":
        out = {"y": [], "dx": [], "dphi": []}
        for seg, prm, x, dy in zip(net.fine, inp["parts"][1], inp["x"], inp["dy"]):
            prm, x = _double(prm), x.double().requires_grad_()
            y = _segment(seg, prm, x, bf16)
            y.backward(dy.double())
            out["y"].append(y.detach().contiguous())
            out["dx"].append(x.grad.contiguous())
            out["dphi"].append(_grad_buffer(seg, prm))
            del y, x, prm
        return out
    if kind == "coarse":
        out = {"rt": [], "d": [], "deta": []}
        for seg, prm, x, a, d in zip(net.coarse, inp["parts"][2], inp["rt"], inp["add"], inp["d"]):
            prm, x = _double(prm), x.double().requires_grad_()
            y = _segment(seg, prm, x, bf16, a.double())
            y.backward(d.double())
            out["rt"].append(y.detach().contiguous())
            out["d"].append(x.grad.contiguous())
            out["deta"].append(_grad_buffer(seg, prm))
        return out
    # the whole step: eqs. (xjyj), (rk), (tilderk), (tildey), the head and autograd
    prms = [[_double(p) for p in part] for part in inp["parts"]]
    eps = inp["head"].double().requires_grad_()
    image = inp["image"].double()
    xs = []
    for seg, prm in zip(net.pre, prms[0]):
        t = _segment(seg, prm, image, bf16)
        t = t if t.requires_grad else t.detach().clone().requires_grad_()
        t.retain_grad()
        xs.append(t)
    ys = [_segment(seg, prm, x, bf16) for seg, prm, x in zip(net.fine, prms[1], xs)]
    yt = ys[-1]
    if n > 1:
        rt = _stored(ys[0] - xs[1], bf16)
        for j in range(n - 1):
            add = _stored(ys[j + 1] - xs[j + 2], bf16) if j < n - 2 else ys[n - 1]
            rt = _segment(net.coarse[j], prms[2][j], rt, bf16, add)
        yt = rt
    logits, loss = _head64(yt, eps, inp["labels"], net.classes)
    loss.backward()
    out = {"logits": logits.detach(), "loss": loss.detach().view(1)}
    if net.dtype != "bf16":
        grads = [_grad_buffer(s, p) for segs, part in zip((net.pre, net.fine, net.coarse), prms)
                 for s, p in zip(segs, part)]
        return {**out, "ytilde": yt.detach().contiguous(), "dx": [x.grad.contiguous() for x in xs],
                "head": eps.grad, "grads": grads}
    with torch.no_grad():
        def new(t):
            return _sgd(t, t.grad)[0]
        masters, tails = [], {0: [], 1: [], 2: []}
        for part, (segs, prm) in enumerate(zip((net.pre, net.fine, net.coarse), prms)):
            got = [_master(s, p, new) for s, p in zip(segs, prm)]
            if got:
                masters.append(torch.cat([a for a, _ in got]))
            tails[part] = [b for _, b in got if b is not None]
        return {**out, "master": masters, "head": new(eps), "bn": tails[1] + tails[2] + tails[0]}
