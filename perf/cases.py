"""The calls that a user of this package makes, as cases that can be timed and
compared: stage forwards, stage backwards (reconstruction + VJP), whole stage
steps and a tick of the multi-stage schedule, through Stage and Net.

A case is one call on one shape.  Stage shapes are [n, h, w] with c channels
per stream (2 c in all) and, for bottleneck blocks, an inner width of c_mid.
Backwards and steps have one block, as in the per-layer split, where every
reversible block is a stage of its own: in 16 bits a longer chain of
reconstructions moves ReLU decisions, and two correct implementations then
differ by far more than the data type says.  Forwards have all their blocks.
"""
import math

import torch

from paper_2406_02052_amd import Net, Stage

EPS, BN_MOMENTUM = 1e-5, 0.1
# the schedule's rate is that of a warm-up; a single stage, whose gradient here is
# the same in every call, gets a smaller one so that its weights stay where they are
LR, STAGE_LR, MOMENTUM, DECAY = 0.01, 1e-3, 0.9, 5e-4
NET_WIDTHS, NET_CLASSES, NET_BATCHES = (64, 128, 256, 512), 10, 4


def _stage(name, call, kind, dtype, n, h, w, c, c_mid=0, blocks=1, k=1):
    return {"name": name, "call": call, "kind": kind, "dtype": dtype, "n": n, "h": h, "w": w,
            "c": c, "c_mid": c_mid, "blocks": blocks, "k": k}


def listed():
    return [
        # the smallest stage that is used: one fp32 block, every kernel a launch
        _stage("step_fp32_8x8x8", "step", "basic", "fp32", 8, 8, 8, 16),
        # one block of the CIFAR-shaped RevNet-18's first level, a training step
        _stage("step_cifar_128x32x32", "step", "basic", "bf16", 128, 32, 32, 32),
        # one block of the ImageNet32-shaped RevNet-34 stage, a training step
        _stage("step_imagenet32_256x16x16", "step", "basic", "bf16", 256, 16, 16, 128),
        # one block of the ImageNet-shaped RevNet-50's first level, a training step
        _stage("step_bottleneck_64x56x56", "step", "bottleneck", "bf16", 64, 56, 56, 128, 32),
        # forwards of whole stages: a small batch (evaluation, the first stages of
        # a pipeline with small micro-batches) and the two large ones
        _stage("forward_cifar_8x32x32", "forward", "basic", "bf16", 8, 32, 32, 32, blocks=2),
        _stage("forward_imagenet32_256x16x16", "forward", "basic", "bf16", 256, 16, 16, 128, blocks=6),
        _stage("forward_bottleneck_64x56x56", "forward", "bottleneck", "bf16", 64, 56, 56, 128, 32, blocks=3),
        # backwards with gradient accumulation: the third level of the CIFAR-shaped
        # RevNet-18, the second level of an ImageNet-shaped one (28 pixels wide), a
        # ragged bottleneck and the CIFAR shape held in fp32
        _stage("backward_128x8x8", "backward", "basic", "bf16", 128, 8, 8, 128, k=2),
        _stage("backward_64x28x28", "backward", "basic", "bf16", 64, 28, 28, 64, k=2),
        _stage("backward_bottleneck_37x23x23", "backward", "bottleneck", "bf16", 37, 23, 23, 128, 32, k=2),
        _stage("backward_fp32_32x32x32", "backward", "basic", "fp32", 32, 32, 32, 32, k=2),
        # one tick of the 4-stage RevNet-18 schedule in its steady state
        {"name": "tick_revnet18_128", "call": "tick", "dtype": "bf16", "n": 128, "h": 32, "w": 32, "blocks": 2},
    ]


def draw(rng):
    """Stage calls over the widths, image sizes and batches of such networks, odd
    sizes among them, and ticks of small schedules."""
    if rng.random() < 0.1:
        return {"call": "tick", "dtype": "bf16", "n": round(2 ** rng.uniform(3, 7)), "h": 32, "w": 32,
                "blocks": rng.choice((1, 2))}
    call = rng.choice(("forward", "backward", "step"))
    kind = rng.choice(("basic", "basic", "bottleneck"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "fp32"))
    if rng.random() < 0.6:
        h = w = rng.choice((7, 8, 14, 16, 28, 32, 56))
    else:
        h, w = (round(2 ** rng.uniform(2.3, 6)) for _ in range(2))
    c = rng.choice((32, 64, 128) if kind == "basic" else (64, 128))
    c_mid = 0 if kind == "basic" else rng.choice((c // 4, 32))
    blocks = rng.choice((1, 2, 3)) if call == "forward" else 1
    # pixels: from small to what the largest stage above holds, with room for the
    # wider taps of basic blocks and the bytes of fp32
    most = 200704 * 128 // c // (4 if kind == "basic" else 1) // (4 if dtype == "fp32" else 1)
    pixels = 2 ** rng.uniform(9, math.log2(most))
    n = max(2, min(256, round(pixels / (h * w))))
    return {"call": call, "kind": kind, "dtype": dtype, "n": n, "h": h, "w": w, "c": c,
            "c_mid": c_mid, "blocks": blocks, "k": 1 if call == "step" else 2}


# ---------------------------------------------------------------------------
# shapes, layouts and inputs
# ---------------------------------------------------------------------------

def _convs(case):
    """(c_out, taps per side, c_in) of the convs of one residual function."""
    c, m = case["c"], case["c_mid"]
    return [(c, 3, c), (c, 3, c)] if case["kind"] == "basic" else [(m, 1, c), (m, 3, m), (c, 1, m)]


def _net_stage(case, j):
    """The blocks of level j of the schedule, as a stage case."""
    return {"kind": "basic", "c": NET_WIDTHS[j] // 2, "c_mid": 0, "blocks": case["blocks"]}


def _store(case, t):
    return t.to(torch.bfloat16) if case["dtype"] == "bf16" else t.float()


class _Draw:
    """Seeded fp32 tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator("cuda").manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda") * std

    def bn(self, c, last=False):
        """gamma and beta of a network in training: gamma about 1, and small in the
        last BN of a residual function, where it starts at zero."""
        gamma = 0.5 + torch.rand(c, generator=self.g, device="cuda")
        return [gamma * 0.2 if last else gamma, self.normal(c, std=0.2)]

    def conv(self, o, r, i):
        """He-normal weights [c_out][r][s][c_in] that bf16 holds exactly."""
        return self.normal(o, r, r, i, std=math.sqrt(2.0 / (r * r * i))).bfloat16().float()


def _stage_params(case, d):
    """Canonical order: block, function F then G, conv: weight, gamma, beta."""
    convs = _convs(case)
    return [t for _ in range(2 * case["blocks"]) for l, (o, r, i) in enumerate(convs)
            for t in (d.conv(o, r, i), *d.bn(o, last=l + 1 == len(convs)))]


def _stage_tensors(case, d):
    shape = (case["n"], case["h"], case["w"], case["c"])
    x = [_store(case, d.normal(*shape).abs()) for _ in range(2)]
    # a stage's output: its input plus the normalised output of a residual function
    y = [_store(case, d.normal(*shape).abs() + d.normal(*shape, std=0.2)) for _ in range(2)]
    dy = [_store(case, d.normal(*shape, std=1e-3)) for _ in range(2)]
    return x, y, dy


def _net_params(case, d):
    out = []
    for j, w in enumerate(NET_WIDTHS):
        out += [d.conv(w, 3, 3) if j == 0 else d.conv(w, 1, NET_WIDTHS[j - 1]), *d.bn(w)]
        out += _stage_params(_net_stage(case, j), d)
    return out + [d.normal(NET_CLASSES, NET_WIDTHS[-1], std=math.sqrt(2.0 / NET_WIDTHS[-1])),
                  torch.zeros(NET_CLASSES, device="cuda")]


def _net_tensors(case, d):
    images = [_store(case, d.normal(case["n"], case["h"], case["w"], 3)) for _ in range(NET_BATCHES)]
    labels = [torch.randint(NET_CLASSES, (case["n"],), generator=d.g, device="cuda", dtype=torch.int32)
              for _ in range(NET_BATCHES)]
    return images, labels


def _warm_ticks():
    """Ticks until every stage runs a forward and a backward in each."""
    return 2 * len(NET_WIDTHS) - 1


class _State:
    pass


def prepare(case, seed):
    d, s = _Draw(seed), _State()
    s.call = case["call"]
    if s.call == "tick":
        s.net = Net(case["n"], case["h"], case["w"], 3, NET_WIDTHS, case["blocks"], NET_CLASSES,
                    case["dtype"], EPS, BN_MOMENTUM)
        s.net.set_params([t.cpu().numpy() for t in _net_params(case, d)])
        s.net.set_optimizer(LR, MOMENTUM, DECAY)
        s.images, s.labels = _net_tensors(case, d)
        for t in range(_warm_ticks()):
            s.net.tick(s.images[t % NET_BATCHES], s.labels[t % NET_BATCHES])
        s.t = _warm_ticks()
        return s
    s.stage = Stage(case["n"], case["h"], case["w"], case["c"], case["blocks"], case["kind"],
                    case["dtype"], case["c_mid"], EPS, BN_MOMENTUM)
    s.stage.set_params([t.cpu().numpy() for t in _stage_params(case, d)])
    s.stage.set_optimizer(STAGE_LR, MOMENTUM, DECAY, accum_k=case["k"])
    s.x, s.y, s.dy = _stage_tensors(case, d)
    s.out, s.back, s.dx = ([s.stage.act(), s.stage.act()] for _ in range(3))
    return s


def run(s):
    if s.call == "tick":
        i = s.t % NET_BATCHES
        s.t += 1
        s.net.tick(s.images[i], s.labels[i])
        return {"loss": s.net.loss, "params": s.net.params, "run_mean": s.net.run_mean, "run_var": s.net.run_var}
    st = s.stage
    if s.call == "forward":
        st.forward(*s.x, *s.out)
        return {"y": s.out}
    if s.call == "backward":
        st.reconstruct_backward(*s.y, *s.dy, *s.back, *s.dx)
        return {"x": s.back, "dx": s.dx, "grad": st.grad, "run_mean": st.run_mean, "run_var": st.run_var}
    st.step(*s.x, *s.out, *s.y, *s.dy, *s.back, *s.dx)
    return {"y": s.out, "x": s.back, "dx": s.dx, "params": st.params, "momentum": st.mom,
            "run_mean": st.run_mean, "run_var": st.run_var}


# ---------------------------------------------------------------------------
# what a call cannot do without
# ---------------------------------------------------------------------------

def _stage_work(case, n, h, w, call, esz):
    """A forward reads and writes both streams; a backward reads the outputs and
    their gradients and writes as much; a step does both and updates.  Between
    two functions of a block the streams, and between two convs of a function
    the normalised tensors, need all rows for their batch statistics: chip
    memory is not counted for them, since a small stage's could stay in caches."""
    m, convs = n * h * w, _convs(case)
    macs = m * 2 * case["blocks"] * sum(o * r * r * i for o, r, i in convs)
    params = 2 * case["blocks"] * sum(o * r * r * i + 2 * o for o, r, i in convs)
    act = 2 * m * case["c"] * esz
    fwd = {"bytes": 2 * act + 4 * params, "flops": 2 * macs}
    bwd = {"bytes": 4 * act + 8 * params, "flops": 6 * macs}
    if call == "forward":
        return fwd
    if call == "backward":
        return bwd
    return {"bytes": fwd["bytes"] + bwd["bytes"] + 16 * params, "flops": fwd["flops"] + bwd["flops"]}


def work(case):
    esz = 2 if case["dtype"] == "bf16" else 4
    if case["call"] != "tick":
        return _stage_work(case, case["n"], case["h"], case["w"], case["call"], esz)
    total = {"bytes": 0, "flops": 0}
    for j, wd in enumerate(NET_WIDTHS):
        h, w = case["h"] >> j, case["w"] >> j
        got = _stage_work(_net_stage(case, j), case["n"], h, w, "step", esz)
        macs = case["n"] * h * w * wd * (27 if j == 0 else NET_WIDTHS[j - 1])   # the front layer
        total["bytes"] += got["bytes"]
        total["flops"] += got["flops"] + 8 * macs
    return total


def tolerance(case):
    """About four times what the same calls differ by when their sums are taken in
    another order, with every tensor held in the case's storage type.  A last bit
    that moves a ReLU decision changes single gradients by about their size, which
    "max" allows for."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3} if case["call"] == "forward" else {"rel": 1e-3, "max": 0.5}
    if case["call"] in ("forward", "tick"):
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 3e-2, "max": 0.9}


# ---------------------------------------------------------------------------
# the same calls in plain torch, in 64 bits
# ---------------------------------------------------------------------------

def _conv(x, w, stride=1):
    """x [n][h][w][i], w [o][r][s][i], "same" padding."""
    r = w.shape[1]
    if r == 1:
        return x[:, ::stride, ::stride] @ w[:, 0, 0].T
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    h, wd = x.shape[1:3]
    return sum(p[:, i:i + h, j:j + wd] @ w[:, i, j].T for i in range(r) for j in range(r))


def _bn(h, gamma, beta, stats):
    mean = h.mean((0, 1, 2))
    var = (h - mean).square().mean((0, 1, 2))
    m = h[..., 0].numel()
    stats.append((mean.detach(), var.detach() * m / max(1, m - 1)))
    return (h - mean) / (var + EPS).sqrt() * gamma + beta


class _Math:
    """Sums in `dtype`; `store`, if any, rounds where the calls hold a tensor."""

    def __init__(self, dtype=torch.float64, store=None):
        self.dtype, self.store = dtype, store

    def hold(self, t):
        """Values as stored, straight through for gradients and stored there too."""
        return t if self.store is None else _Held.apply(t, self.store)

    def conv(self, x, w, stride=1):
        """With the weights rounded as the calls' compute copies are."""
        if self.store is not None:
            w = w + (w.to(self.store).to(w.dtype) - w).detach()
        return self.hold(_conv(x, w, stride))

    def fn(self, u, layers, stats):
        for i, (w, gamma, beta) in enumerate(layers):
            u = _bn(self.conv(u, w), gamma, beta, stats)
            if i + 1 < len(layers):
                u = self.hold(torch.relu(u))
        return u

    def forward(self, x1, x2, fns):
        with torch.no_grad():
            for b in range(0, len(fns), 2):
                x1 = self.hold(x1 + self.fn(x2, fns[b], []))
                x2 = self.hold(x2 + self.fn(x1, fns[b + 1], []))
        return x1, x2

    def backward(self, y1, y2, g1, g2, fns):
        """Rebuilds the input and takes the VJP; gradients and statistics by function."""
        grads, stats = [None] * len(fns), [[] for _ in fns]
        for b in reversed(range(len(fns))):
            # the function of u, added to v; g is the gradient of that sum
            u, v, g, rest = (y1, y2, g2, g1) if b % 2 else (y2, y1, g1, g2)
            u = u.detach().requires_grad_()
            leaves = [[t.detach().requires_grad_() for t in layer] for layer in fns[b]]
            f = self.fn(u, leaves, stats[b])
            du, *flat = torch.autograd.grad(f, [u] + [t for layer in leaves for t in layer], g)
            v, rest = self.hold(v - f.detach()), self.hold(rest + du)
            grads[b] = [flat[i:i + 3] for i in range(0, len(flat), 3)]
            (y1, y2, g1, g2) = (u, v, rest, g) if b % 2 else (v, u, g, rest)
        return [t.detach() for t in (y1, y2, g1, g2)], grads, stats


class _Held(torch.autograd.Function):
    @staticmethod
    def forward(ctx, t, store):
        ctx.store = store
        return t.to(store).to(t.dtype)

    @staticmethod
    def backward(ctx, g):
        return g.to(ctx.store).to(g.dtype), None


def _functions(params, nconv):
    layers = [params[i:i + 3] for i in range(0, len(params), 3)]
    return [layers[i:i + nconv] for i in range(0, len(layers), nconv)]


def _flat(fns):
    """All conv weights, then each BN's gamma and beta: the order of the flat buffers."""
    layers = [layer for f in fns for layer in f]
    return [w for w, _, _ in layers] + [t for _, g, b in layers for t in (g, b)]


def _cat(ts):
    return torch.cat([t.reshape(-1) for t in ts])


def _running(stats, mean, var):
    pairs = [p for f in stats for p in f]
    return ((1 - BN_MOMENTUM) * mean + BN_MOMENTUM * _cat([m for m, _ in pairs]),
            (1 - BN_MOMENTUM) * var + BN_MOMENTUM * _cat([v for _, v in pairs]))


def _sgd(lr, p, g, buf, decay):
    g = g + DECAY * p if decay else g
    buf = MOMENTUM * buf + g
    return p - lr * (g + MOMENTUM * buf), buf


def _exact_stage(case, seed, m):
    d = _Draw(seed)
    fns = _functions([t.to(m.dtype) for t in _stage_params(case, d)], len(_convs(case)))
    x, y, dy = ([t.to(m.dtype) for t in ts] for ts in _stage_tensors(case, d))
    if case["call"] == "forward":
        return {"y": list(m.forward(*x, fns))}
    (x1, x2, d1, d2), grads, stats = m.backward(*y, *dy, fns)
    mean, var = _running(stats, 0.0, 1.0)
    out = {"x": [x1, x2], "dx": [d1, d2], "run_mean": mean, "run_var": var}
    params, grad = _flat(fns), [g / case["k"] for g in _flat(grads)]
    if case["call"] == "backward":
        out["grad"] = _cat(grad)
        return out
    new = [_sgd(STAGE_LR, p, g, 0.0, p.dim() == 4) for p, g in zip(params, grad)]
    out.update(y=list(m.forward(*x, fns)), params=_cat([p for p, _ in new]), momentum=_cat([b for _, b in new]))
    return out


class _Level:
    """One stage of the schedule: a front layer, blocks and, in the last, the head."""

    def __init__(self, j, params, last, m):
        self.j, self.last, self.m = j, last, m
        self.front, rest = params[:3], params[3:]
        self.head, rest = (rest[-2:], rest[:-2]) if last else ([], rest)
        self.fns = _functions(rest, 2)
        self.buf = [torch.zeros_like(p) for p in self.leaves()]
        n = [sum(layer[1].numel() for f in self.fns for layer in f), self.front[1].numel()]
        self.stats = [[torch.zeros(c, device="cuda", dtype=m.dtype), torch.ones(c, device="cuda", dtype=m.dtype)] for c in n]
        self.inputs = {}

    def leaves(self):
        """[front weight][linear weight][blocks][front gamma, beta][linear bias]"""
        return self.front[:1] + self.head[:1] + _flat(self.fns) + self.front[1:] + self.head[1:]

    def run_front(self, x, front, stats):
        h = _bn(self.m.conv(x, front[0], 1 if self.j == 0 else 2), *front[1:], stats)
        return self.m.hold(torch.relu(h) if self.j == 0 else h)

    def forward(self, mb):
        with torch.no_grad():
            x = self.run_front(self.inputs[mb], self.front, [])
        return torch.cat(self.m.forward(*x.chunk(2, -1), self.fns), -1)

    def loss(self, y, labels):
        y = y.detach().requires_grad_()
        w, b = (t.detach().requires_grad_() for t in self.head)
        loss = torch.nn.functional.cross_entropy(y.mean((1, 2)) @ w.T + b, labels.long())
        g, *gh = torch.autograd.grad(loss, [y, w, b])
        return loss.detach(), self.m.hold(g), gh

    def backward(self, mb, y, g, head_grads):
        (_, _, d1, d2), grads, stats = self.m.backward(*y.chunk(2, -1), *g.chunk(2, -1), self.fns)
        x = self.inputs.pop(mb).detach().requires_grad_()
        front, fstats = [t.detach().requires_grad_() for t in self.front], []
        out = self.run_front(x, front, fstats)
        dx, *fg = torch.autograd.grad(out, [x] + front, torch.cat([d1, d2], -1))
        self.stats = [list(_running(stats, *self.stats[0])), list(_running([fstats], *self.stats[1]))]
        self.grads = fg[:1] + head_grads[:1] + _flat(grads) + fg[1:] + head_grads[1:]
        return self.m.hold(dx)

    def update(self):
        old = self.leaves()
        new = [_sgd(LR, p, g, b, p.dim() > 1) for p, g, b in zip(old, self.grads, self.buf)]
        self.buf = [b for _, b in new]
        at = {id(p): q for p, (q, _) in zip(old, new)}
        self.front = [at[id(p)] for p in self.front]
        self.head = [at[id(p)] for p in self.head]
        self.fns = [[[at[id(p)] for p in layer] for layer in f] for f in self.fns]


def _exact_tick(case, seed, m):
    d, levels = _Draw(seed), len(NET_WIDTHS)
    params = [t.to(m.dtype) for t in _net_params(case, d)]
    images, labels = _net_tensors(case, d)
    per = 3 + 12 * case["blocks"]
    st = [_Level(j, params[j * per:(j + 1) * per + (2 if j == levels - 1 else 0)], j == levels - 1, m) for j in range(levels)]
    grads_in, outs, loss = {}, {}, None
    for t in range(_warm_ticks() + 1):
        sent, arrived = {}, []
        st[0].inputs[t] = images[t % NET_BATCHES].to(m.dtype)
        for s in st:
            f, b = t - s.j, t - (2 * levels - 2 - s.j)
            if f >= 0:
                outs[s.j, f] = s.forward(f)
                if not s.last:
                    arrived.append((s.j + 1, f))
            if b >= 0:
                y, g, gh = outs.pop((s.j, b)), None, []
                if s.last:
                    loss, g, gh = s.loss(y, labels[b % NET_BATCHES])
                else:
                    g = grads_in[s.j]
                sent[s.j - 1] = s.backward(b, y, g, gh)
                s.update()
        for j, mb in arrived:   # one hop a tick
            st[j].inputs[mb] = outs[j - 1, mb]
        grads_in = sent
    return {"loss": loss.reshape(1), "params": _cat([p for s in st for p in s.leaves()]),
            "run_mean": _cat([t[0] for s in st for t in (s.stats[1], s.stats[0])]),
            "run_var": _cat([t[1] for s in st for t in (s.stats[1], s.stats[0])])}


def exact(case, seed):
    m = _Math()
    return _exact_tick(case, seed, m) if case["call"] == "tick" else _exact_stage(case, seed, m)
