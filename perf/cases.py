"""What the framework's speed is measured on.

Whole training steps and blocks go through a Plan (monet_plan_load / monet_step), single layers through the operator
entry points of the C ABI (`monet.call`).  Everything is fp32, activations N,H,W,C, filters K,R,S,C.  A layer case runs
the forward pass and both gradients of one layer, a block or step case one training step under its schedule.

Every gradient of a plan lands in one flat tensor per block, each parameter at a multiple of 64 floats (the gaps stay
zero), so that a network of 161 parameters comes back whole in a few outputs.
"""
import math

import torch

from paper_2010_14501_amd import monet
from workloads import graphs, schedules

DEV = "cuda:0"
RESIDUAL_GAIN = 0.2


# ---------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: four 16-channel blocks on 16x16 maps, 20 operators of a few microseconds each
        dict(name="step_tiny_chain", kind="chain", n=2, hw=16, c=16, blocks=4),
        # the framework's own benchmark: one training step of ResNet-50 at batch 184, block outputs kept, the rest recomputed
        dict(name="step_resnet50_b184", kind="resnet", n=184),
        # a bottleneck block of that network (1x1, 3x3, 1x1 with BatchNorm and ReLU, residual add) on its 14x14 maps
        dict(name="block_bottleneck_14x14", kind="bottleneck", n=184, h=14, w=14, c=1024, k=256),
        # an inverted-residual block of MobileNetV2 at batch 272 (1x1 expansion, depthwise 3x3, 1x1 projection, ReLU6)
        dict(name="block_inverted_56x56", kind="inverted", n=272, h=56, w=56, c=24, k=144),
        # expansion layer of ResNet-50's first stage: few channels on large maps
        dict(name="conv1x1_56x56_64_256", kind="conv", n=184, h=56, w=56, c=64, k=256, r=1, stride=1, pad=0),
        # the strided 3x3 layer between two stages
        dict(name="conv3x3s2_56x56_128", kind="conv", n=184, h=56, w=56, c=128, k=128, r=3, stride=2, pad=1),
        # 5x5 branch of an inception module: 24 input channels
        dict(name="conv5x5_14x14_24_64", kind="conv", n=320, h=14, w=14, c=24, k=64, r=5, stride=1, pad=2),
        # odd batch, odd maps, channels that fill no tile: what a user's own small network brings
        dict(name="conv3x3_ragged", kind="conv", n=3, h=13, w=17, c=60, k=92, r=3, stride=1, pad=1),
        # VGG-16's first fully connected layer: a filter matrix of 411 MB
        dict(name="fc_25088_4096", kind="conv", n=176, h=1, w=1, c=25088, k=4096, r=1, stride=1, pad=0),
        # first layer of ResNet-50: three input channels, no input gradient
        dict(name="stem7x7_224", kind="conv", n=184, h=224, w=224, c=3, k=64, r=7, stride=2, pad=3),
        # a 3x3 layer of VGG-16 through the Winograd implementations that its schedules choose
        dict(name="winograd_112x112_128", kind="winograd", n=176, h=112, w=112, c=128, k=128),
        # BatchNorm and ReLU with sign mask, forward and backward, on ResNet-50's widest maps
        dict(name="bn_relu_56x56_256", kind="bn_relu", n=184, h=56, w=56, c=256),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _channels(rng, lo, hi, step=4):
    c = _log(rng, lo, hi)
    return max(step, c // step * step)


def _fit(rng, per_image, budget, top):
    """A batch whose work stays within the budget."""
    return _log(rng, 1, max(1, min(top, int(budget / per_image))))


def draw(rng):
    kind = rng.choice(["conv"] * 6 + ["winograd"] * 2 + ["bottleneck", "bottleneck", "inverted", "inverted", "bn_relu", "resnet", "chain"])
    if kind == "chain":
        return dict(kind=kind, n=_log(rng, 1, 16), hw=rng.randint(8, 40), c=16 * rng.randint(1, 3), blocks=rng.randint(2, 6))
    if kind == "resnet":
        return dict(kind=kind, n=_log(rng, 16, 160))
    hw = _log(rng, 7, 112)
    h, w = hw, max(5, hw + rng.choice([0, 0, 0, -1, 3]))
    if kind == "bottleneck":
        k = _channels(rng, 32, 512, 16)
        return dict(kind=kind, n=_fit(rng, 34.0 * h * w * k * k, 3e11, 256), h=h, w=w, c=4 * k, k=k)
    if kind == "inverted":
        c = _channels(rng, 16, 160, 8)
        return dict(kind=kind, n=_fit(rng, h * w * c * 6.0, 1.2e8, 272), h=h, w=w, c=c, k=6 * c)
    if kind == "bn_relu":
        c = _channels(rng, 16, 2048)
        return dict(kind=kind, n=_fit(rng, h * w * c, 1.5e8, 320), h=h, w=w, c=c)
    if kind == "winograd":
        c, k = _channels(rng, 64, 512, 16), _channels(rng, 64, 512, 16)
        return dict(kind=kind, n=_fit(rng, 18.0 * h * w * c * k, 5e11, 176), h=h, w=w, c=c, k=k)
    r = rng.choice([1, 1, 1, 3, 3, 5])
    stride = rng.choice([1, 1, 1, 2])
    step = rng.choice([1, 4, 4, 8, 16, 16, 32])
    c, k = _channels(rng, 16, 1024 if r == 1 else 512, step), _channels(rng, 16, 1024 if r == 1 else 512, step)
    per = 2.0 * (h // stride + 1) * (w // stride + 1) * c * k * r * r
    return dict(kind=kind, n=_fit(rng, per, 2e11 if step > 1 else 5e10, 320), h=h, w=w, c=c, k=k, r=r, stride=stride, pad=r // 2)


# ---------------------------------------------------------------------- plans
def _graph(c):
    """(graph, schedule) as a user's program builds them."""
    if c["kind"] == "chain":
        g = graphs.tiny_chain(batch=c["n"], hw=c["hw"], channels=c["c"], blocks=c["blocks"])
        return g, schedules.tiny_chain_schedule(g, set(range(0, c["blocks"], 2)))
    if c["kind"] == "resnet":
        g = graphs.resnet50(batch=c["n"])
        return g, schedules.block_output_schedule(g)
    g = graphs.Graph()
    a = g.ext("x", "f32", (c["n"], c["h"], c["w"], c["c"]))

    def cbr(a, K, R, pad, name, six):
        return g.relu(g.bn(g.conv(a, K, R, pad=pad, name=name), name=name + ".bn"), six=six)

    # a block inside a network: a 1x1 layer before it, so that the block's own input gradient is computed
    g.begin_block("before")
    a = cbr(a, c["c"], 1, 0, "before", c["kind"] == "inverted")
    g.end_block()
    g.begin_block("block")
    if c["kind"] == "bottleneck":
        h = cbr(a, c["k"], 1, 0, "conv1", False)
        h = cbr(h, c["k"], 3, 1, "conv2", False)
        h = g.bn(g.conv(h, c["c"], 1, name="conv3"), name="conv3.bn")
        a = g.relu(g.add(h, a))
    else:
        h = cbr(a, c["k"], 1, 0, "expand", True)
        h = g.relu(g.bn(g.dwconv(h, 3, 1, 1, name="dw"), name="dw.bn"), six=True)
        h = g.bn(g.conv(h, c["c"], 1, name="project"), name="project.bn")
        a = g.relu(g.add(h, a), six=True)
    g.end_block()
    g.sumloss(a)
    return g, schedules.block_output_schedule(g)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _plan_inputs(g, seed):
    """(external tensors, parameters) of a graph: N(0,1) images, uniform labels, He-normal filters, random affine BatchNorm."""
    gen = _gen(seed)
    exts, params = [], []
    for _, _, dt, shp in g.exts:
        exts.append(torch.randn(shp, generator=gen, device=DEV) if dt == "f32"
                    else torch.randint(0, 1000, shp, generator=gen, device=DEV, dtype=torch.int32))
    for _, name, shp in g.params:
        if name.endswith(".gamma"):
            # the BatchNorm that closes a residual branch starts small, as is usual for such networks
            gain = RESIDUAL_GAIN if name.endswith(".bn3.gamma") else 1.0
            params.append(gain * (0.5 + torch.rand(shp, generator=gen, device=DEV)))
        elif name.endswith(".beta"):
            params.append(0.1 * torch.randn(shp, generator=gen, device=DEV))
        elif name.endswith(".b"):
            params.append(torch.zeros(shp, device=DEV))
        elif len(shp) == 4:
            params.append(torch.randn(shp, generator=gen, device=DEV) * math.sqrt(2.0 / (shp[1] * shp[2] * shp[3])))
        else:
            params.append(torch.randn(shp, generator=gen, device=DEV) * math.sqrt(1.0 / shp[1]))
    return exts, params


def _param_groups(g):
    """Parameter ids by block, in order."""
    out, seen = [], set()
    for _, nodes in g.blocks:
        pids = [p for i in nodes for p in g.nodes[i - 1].pars if p not in seen]
        seen.update(pids)
        if pids:
            out.append(pids)
    return out


def _place(g, groups):
    """Offset of every parameter in its block's flat tensor, and the lengths of those tensors."""
    offs, lens = {}, []
    for grp in groups:
        at = 0
        for p in grp:
            offs[p] = (len(lens), at)
            at += -(-graphs.numel(g.params[p][2]) // 64) * 64
        lens.append(at)
    return offs, lens


class PlanState:
    def __init__(self, case, seed):
        g, sch = _graph(case)
        self.exts, self.params = _plan_inputs(g, seed)
        self.plan = monet.Plan(g.text(), sch.text())
        offs, lens = _place(g, _param_groups(g))
        self.grads = [torch.zeros(n, device=DEV) for n in lens]
        self.loss = torch.zeros(1, device=DEV)
        self.arena = torch.empty(self.plan.arena_bytes + 256, dtype=torch.uint8, device=DEV)
        self.plan.bind_arena((self.arena.data_ptr() + 255) // 256 * 256, self.plan.arena_bytes)
        self.in_ptrs = [t.data_ptr() for t in self.exts]
        self.w_ptrs = [t.data_ptr() for t in self.params]
        self.g_ptrs = [self.grads[offs[p][0]].data_ptr() + 4 * offs[p][1] for p in range(len(self.params))]

    def run(self):
        self.plan.step(torch.cuda.current_stream().cuda_stream, self.in_ptrs, self.w_ptrs, self.g_ptrs, self.loss.data_ptr())
        return {"loss": self.loss, "grads": self.grads}


# ---------------------------------------------------------------------- layers
def _out_hw(c):
    return tuple((c[a] + 2 * c["pad"] - c["r"]) // c["stride"] + 1 for a in ("h", "w"))


def _conv_inputs(c, seed):
    """Input as a ReLU leaves it (the first layer: an image), He-normal filter, output gradient."""
    gen = _gen(seed)
    x = torch.randn((c["n"], c["h"], c["w"], c["c"]), generator=gen, device=DEV)
    if c["c"] > 3:
        x = x.relu_()
    w = torch.randn((c["k"], c["r"], c["r"], c["c"]), generator=gen, device=DEV) * math.sqrt(2.0 / (c["c"] * c["r"] ** 2))
    dy = torch.randn((c["n"],) + _out_hw(c) + (c["k"],), generator=gen, device=DEV) * 1e-3
    return x, w, dy


def _buffer(nbytes):
    return torch.empty(max(64, -(-nbytes // 4)), device=DEV)


class ConvState:
    """Forward, input gradient and filter gradient of one layer, with the reduction splits and workspaces that the graph
    builder gives such a layer."""

    def __init__(self, c, seed):
        self.x, self.w, self.dy = _conv_inputs(c, seed)
        P, Q = _out_hw(c)
        n, h, w, C, K, r, s = (c[a] for a in ("n", "h", "w", "c", "k", "r", "stride"))
        self.dims = (n, h, w, C, K, r, r, s, c["pad"])
        self.y, self.dw = torch.empty_like(self.dy), torch.empty_like(self.w)
        self.dx = torch.empty_like(self.x) if C > 3 else None
        self.fwd_splits, ws_f = graphs.conv_split_plan(n * P * Q, K, C * r * r)
        self.bwd_splits, ws_b = graphs.conv_split_plan(n * math.ceil(h / s) * math.ceil(w / s), C, max(1, r // s) ** 2 * K, s * s, n * h * w * C)
        self.w_splits = graphs.wgrad_split_count(n * P * Q, K, C * r * r)
        ws_w = self.w_splits * 4 * K * C * r * r if self.w_splits > 1 else 0
        self.ws_bytes = [ws_f, ws_b, ws_w]
        self.ws = _buffer(max(self.ws_bytes))

    def run(self):
        st = torch.cuda.current_stream().cuda_stream
        x, w, dy, ws = self.x.data_ptr(), self.w.data_ptr(), self.dy.data_ptr(), self.ws.data_ptr()
        f, b, g = self.ws_bytes
        monet.call("monet_conv_fwd", st, x, w, self.y.data_ptr(), *self.dims, self.fwd_splits, ws if f else None, f)
        if self.dx is not None:
            monet.call("monet_conv_dgrad", st, dy, w, self.dx.data_ptr(), *self.dims, 0, self.bwd_splits, ws if b else None, b)
        monet.call("monet_conv_wgrad", st, x, dy, self.dw.data_ptr(), *self.dims, self.w_splits, ws if g else None, g)
        return {"y": self.y, "dx": self.dx, "dw": self.dw} if self.dx is not None else {"y": self.y, "dw": self.dw}


class WinogradState:
    """The same three operators of a 3x3 / stride-1 layer through the Winograd forms: one kernel with the transformed
    filters as workspace for the forward pass and the input gradient, the transformed domain for the filter gradient."""

    def __init__(self, c, seed):
        full = dict(c, r=3, stride=1, pad=1)
        self.x, self.w, self.dy = _conv_inputs(full, seed)
        self.dims = tuple(c[a] for a in ("n", "h", "w", "c", "k"))
        self.y, self.dx, self.dw = torch.empty_like(self.dy), torch.empty_like(self.x), torch.empty_like(self.w)
        lib = monet.load_library()
        self.ws_bytes = [lib.monet_conv_winograd_fused_workspace_bytes(*self.dims, 0), lib.monet_conv_winograd_fused_workspace_bytes(*self.dims, 1),
                         lib.monet_conv_winograd_wgrad_workspace_bytes(*self.dims, 4)]
        self.ws = _buffer(max(self.ws_bytes))

    def run(self):
        st = torch.cuda.current_stream().cuda_stream
        x, w, dy, ws = self.x.data_ptr(), self.w.data_ptr(), self.dy.data_ptr(), self.ws.data_ptr()
        f, b, g = self.ws_bytes
        monet.call("monet_conv_winograd_fused", st, x, w, self.y.data_ptr(), *self.dims, 0, 0, ws, f)
        monet.call("monet_conv_winograd_fused", st, dy, w, self.dx.data_ptr(), *self.dims, 1, 0, ws, b)
        monet.call("monet_conv_winograd_wgrad", st, x, dy, self.dw.data_ptr(), *self.dims, 4, ws, g)
        return {"y": self.y, "dx": self.dx, "dw": self.dw}


def _bn_inputs(c, seed):
    gen = _gen(seed)
    shape = (c["n"], c["h"], c["w"], c["c"])
    x = torch.randn(shape, generator=gen, device=DEV) + 0.25
    dz = torch.randn(shape, generator=gen, device=DEV) * 1e-3
    gamma = 0.5 + torch.rand(c["c"], generator=gen, device=DEV)
    beta = 0.1 * torch.randn(c["c"], generator=gen, device=DEV)
    return x, dz, gamma, beta


class BnReluState:
    """BatchNorm (statistics, apply), ReLU with its 1-bit sign mask, and their backward operators from mask and output."""

    def __init__(self, c, seed):
        self.x, self.dz, self.gamma, self.beta = _bn_inputs(c, seed)
        self.rows, self.c = c["n"] * c["h"] * c["w"], c["c"]
        self.count = self.rows * self.c
        self.stats = torch.empty(2 * self.c, device=DEV)
        self.y, self.z, self.dy, self.dx = (torch.empty_like(self.x) for _ in range(4))
        self.mask = torch.empty((self.count + 63) // 64, dtype=torch.int64, device=DEV)
        self.dgamma, self.dbeta = torch.empty_like(self.gamma), torch.empty_like(self.beta)
        self.scratch = _buffer(96 << 20)

    def run(self):
        st = torch.cuda.current_stream().cuda_stream
        p = {k: getattr(self, k).data_ptr() for k in ("x", "dz", "gamma", "beta", "stats", "y", "z", "dy", "dx", "mask", "dgamma", "dbeta", "scratch")}
        size = self.scratch.numel() * 4
        monet.call("monet_bn_stats", st, p["x"], p["stats"], self.rows, self.c, 1e-5, p["scratch"], size)
        monet.call("monet_bn_apply", st, p["x"], p["y"], p["gamma"], p["beta"], p["stats"], self.rows, self.c)
        monet.call("monet_relu_fwd", st, p["y"], p["z"], p["mask"], self.count, 0)
        monet.call("monet_relu_bwd", st, p["dz"], p["mask"], 2, p["dy"], self.count, 0, 0)
        monet.call("monet_bn_bwd", st, p["dy"], p["y"], 1, p["gamma"], p["beta"], p["stats"], p["dx"], p["dgamma"], p["dbeta"], self.rows, self.c, 0,
                   p["scratch"], size)
        return {"z": self.z, "mask": self.mask, "stats": self.stats, "dx": self.dx, "dgamma": self.dgamma, "dbeta": self.dbeta}


PLANS = ("chain", "resnet", "bottleneck", "inverted")
STATES = dict(conv=ConvState, winograd=WinogradState, bn_relu=BnReluState, **{k: PlanState for k in PLANS})


def prepare(case, seed):
    return STATES[case["kind"]](case, seed)


def run(state):
    return state.run()


# ---------------------------------------------------------------------- work and tolerances
def _conv_flops(shape):
    n, p, q, k, taps, c = shape
    return 2.0 * n * p * q * k * taps * c


def work(case):
    c = case
    if c["kind"] in PLANS:
        g, _ = _graph(c)
        flops = 0.0
        for node in g.nodes:      # forward and both gradients of every contraction (a layer over the input: no input gradient)
            if node.op in ("conv", "linear", "dwconv"):
                wshape = g.params[node.pars[0]][2]
                taps_c = graphs.numel(wshape[1:])
                one = 2.0 * graphs.numel(node.shape) * taps_c
                flops += one * (2 if node.ins[0] <= 0 else 3)
        moved = sum(graphs.numel(e[3]) for e in g.exts) + 2 * sum(graphs.numel(p[2]) for p in g.params)
        # the tensors between two operators that no single kernel can hold: every convolution's and depthwise layer's output
        # is written and read forward, and its gradient written and read backward
        moved += sum(4 * graphs.numel(n.shape) for n in g.nodes if n.op in ("conv", "dwconv"))
        return {"bytes": 4.0 * moved, "flops": flops}
    if c["kind"] == "bn_relu":
        count = c["n"] * c["h"] * c["w"] * c["c"]
        # two dependent passes forward (statistics, apply) and backward (sums, apply): x twice, z; dz and y twice, dx; the mask
        return {"bytes": 4.0 * 8 * count + 3 * count / 8, "flops": 20.0 * count}
    full = dict(c, r=3, stride=1, pad=1) if c["kind"] == "winograd" else c
    P, Q = _out_hw(full)
    x, y, w = c["n"] * c["h"] * c["w"] * c["c"], c["n"] * P * Q * c["k"], c["k"] * c["c"] * full["r"] ** 2
    modes = 3 if c["c"] > 3 else 2
    # the direct form's multiply-adds; x, w and dy read, y, dx and dw written once
    return {"bytes": 4.0 * (x * (modes - 1) + 2 * y + 2 * w), "flops": modes * _conv_flops((c["n"], P, Q, c["k"], full["r"] ** 2, c["c"]))}


def tolerance(case):
    return TOLERANCES[case["kind"]]


TOLERANCES = {
    # 32-bit sums of one layer
    "conv": {"rel": 1e-5, "max": 1e-3},
    # F(4x4, 3x3) rounds about five times more coarsely than the direct form
    "winograd": {"rel": 3e-5, "max": 3e-3},
    "bn_relu": {"rel": 1e-5, "max": 1e-3, "differ": 1e-5},
    # A few layers deep; a ReLU sign that 32 bits cannot decide moves a gradient by about 1/sqrt(elements).  Two sets of
    # convolution implementations were seen 4.5e-4 to 2.3e-3 apart, single values 0.05 of the rms.
    "chain": {"rel": 1e-2, "max": 0.3},
    "bottleneck": {"rel": 1e-2, "max": 0.3},
    "inverted": {"rel": 1e-2, "max": 0.3},
    # 53 layers, each of which passes the signs before it on: 3.6e-3 to 6.2e-3 apart, single values up to 0.87
    "resnet": {"rel": 2e-2, "max": 0.99},
}


# ---------------------------------------------------------------------- the same in 64 bits
def _mm(a, b):
    return torch.mm(a.contiguous(), b.contiguous())


def _taps(x, r, stride, pad, P, Q):
    """For every filter tap the input positions under it, as rows."""
    if pad:
        x = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    for i in range(r):
        for j in range(r):
            yield i, j, x[:, i:i + (P - 1) * stride + 1:stride, j:j + (Q - 1) * stride + 1:stride, :]


def _conv64(x, w, stride, pad):
    n, h, wd, C = x.shape
    K, r = w.shape[:2]
    P, Q = (h + 2 * pad - r) // stride + 1, (wd + 2 * pad - r) // stride + 1
    y = torch.zeros(n * P * Q, K, dtype=torch.float64, device=x.device)
    for i, j, t in _taps(x, r, stride, pad, P, Q):
        y += _mm(t.reshape(-1, C), w[:, i, j, :].t())
    return y.view(n, P, Q, K)


def _conv64_grads(x, w, dy, stride, pad, want_dx):
    n, h, wd, C = x.shape
    K, r = w.shape[:2]
    P, Q = dy.shape[1:3]
    g = dy.reshape(-1, K)
    dw = torch.empty_like(w)
    for i, j, t in _taps(x, r, stride, pad, P, Q):
        dw[:, i, j, :] = _mm(g.t(), t.reshape(-1, C))
    if not want_dx:
        return None, dw
    dx = torch.zeros(n, h + 2 * pad, wd + 2 * pad, C, dtype=torch.float64, device=x.device)
    for i in range(r):
        for j in range(r):
            dx[:, i:i + (P - 1) * stride + 1:stride, j:j + (Q - 1) * stride + 1:stride, :] += _mm(g, w[:, i, j, :]).view(n, P, Q, C)
    return dx[:, pad:pad + h, pad:pad + wd, :].contiguous(), dw


class _Conv64(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, w, stride, pad):
        ctx.save_for_backward(x, w)
        ctx.how = stride, pad
        return _conv64(x, w, stride, pad)

    @staticmethod
    def backward(ctx, dy):
        x, w = ctx.saved_tensors
        dx, dw = _conv64_grads(x, w, dy, *ctx.how, want_dx=ctx.needs_input_grad[0])
        return dx, dw, None, None


def _bn64(x, gamma, beta):
    rows = x.reshape(-1, x.shape[-1])
    mean = rows.mean(0)
    var = ((rows - mean) ** 2).mean(0)
    return (x - mean) / torch.sqrt(var + 1e-5) * gamma + beta


def _depthwise64(x, w):
    n, h, wd, C = x.shape
    y = torch.zeros_like(x)
    for i, j, t in _taps(x, 3, 1, 1, h, wd):
        y = y + t * w[:, i, j, 0]
    return y


def _net64(case, exts, p):
    """The loss of a plan's network.  Parameters come in the order in which the layers take them."""
    p = iter(p)

    def cbr(a, stride=1, pad=0, act=torch.relu):
        y = _bn64(_Conv64.apply(a, next(p), stride, pad), next(p), next(p))
        return act(y) if act else y

    def six(v):
        return torch.clamp(v, 0, 6)

    a = exts[0]
    if case["kind"] == "chain":
        for _ in range(case["blocks"]):
            a = cbr(a, pad=1)
        return a.sum()
    if case["kind"] == "bottleneck":
        a = cbr(a)
        h = cbr(cbr(a), pad=1)
        return torch.relu(cbr(h, act=None) + a).sum()
    if case["kind"] == "inverted":
        a = cbr(a, act=six)
        h = cbr(a, act=six)
        h = six(_bn64(_depthwise64(h, next(p)), next(p), next(p)))
        return six(cbr(h, act=None) + a).sum()
    a = cbr(a, 2, 3)
    a = torch.nn.functional.max_pool2d(a.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1)
    for si, depth in enumerate((3, 4, 6, 3)):
        for b in range(depth):
            s = 2 if b == 0 and si > 0 else 1
            h = cbr(cbr(a), s, 1)
            h = cbr(h, act=None)
            a = torch.relu(h + (cbr(a, s, act=None) if b == 0 else a))
    logits = _mm(a.mean((1, 2)), next(p).t()) + next(p)
    return torch.nn.functional.cross_entropy(logits, exts[1].long())


def exact(case, seed):
    c = case
    if c["kind"] in PLANS:
        g, _ = _graph(c)
        exts, params = _plan_inputs(g, seed)
        exts = [e.double() if e.is_floating_point() else e for e in exts]
        groups = _param_groups(g)
        # Gradients only where the tensors are small: a pre-activation closer to zero than 32 bits resolve takes another
        # sign in 64 bits, and among the millions of a block or a network there are always some.
        if c["kind"] != "chain" or c["blocks"] * c["n"] * c["hw"] ** 2 * c["c"] > 50000:
            with torch.no_grad():
                return {"loss": _net64(c, exts, [q.double() for q in params]).reshape(1), "grads": [None] * len(groups)}
        leaves = [q.double().requires_grad_(True) for q in params]
        loss = _net64(c, exts, leaves)
        loss.backward()
        offs, lens = _place(g, groups)
        flat = [torch.zeros(n, dtype=torch.float64, device=DEV) for n in lens]
        for i, q in enumerate(leaves):
            b, at = offs[i]
            flat[b][at:at + q.numel()] = q.grad.reshape(-1)
        return {"loss": loss.detach().reshape(1), "grads": flat}
    if c["kind"] == "bn_relu":
        x, dz, gamma, beta = (t.double() for t in _bn_inputs(c, seed))
        C = c["c"]
        rows, g = x.reshape(-1, C), dz.reshape(-1, C)
        mean = rows.mean(0)
        inv = 1 / torch.sqrt(((rows - mean) ** 2).mean(0) + 1e-5)
        xhat = (rows - mean) * inv
        y = xhat * gamma + beta
        g = torch.where(y > 0, g, torch.zeros((), dtype=torch.float64, device=DEV))
        dbeta, dgamma = g.sum(0), (g * xhat).sum(0)
        dx = gamma * inv * (g - dbeta / len(rows) - xhat * (dgamma / len(rows)))
        # the mask is whole numbers: compared as they are
        return {"z": torch.relu(y).view(x.shape), "mask": None, "stats": torch.cat([mean, inv]), "dx": dx.view(x.shape), "dgamma": dgamma, "dbeta": dbeta}
    full = dict(c, r=3, stride=1, pad=1) if c["kind"] == "winograd" else c
    x, w, dy = (t.double() for t in _conv_inputs(full, seed))
    y = _conv64(x, w, full["stride"], full["pad"])
    dx, dw = _conv64_grads(x, w, dy, full["stride"], full["pad"], want_dx=c["c"] > 3)
    return {"y": y, "dx": dx, "dw": dw} if dx is not None else {"y": y, "dw": dw}
