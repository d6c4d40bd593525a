"""The calls whose speed matters to a user of the gradient compressor, as measurable cases.

A case names a network (its weight matrices), the entry point, and the options of one call; it is a dict of
plain values:

    net      "layer" (one rows x cols matrix), "resnet18", "resnet50", "vgg19" (the weight layers of those
             networks), "resnet50_all" (ResNet-50 with its normalisation and bias vectors and the side of each
             convolution kernel as that layer's neighbourhood side), "stack" (layers of many sizes from shape_seed)
    call     which entry point one pass goes through (see `run`)
    p, rho, alpha    neighbourhood side (Eq. 7), mean keep ratio, mixing weight (Eq. 8)

Inputs are drawn on the GPU: a gradient is noise plus a smooth field (neighbouring weights' gradients are
correlated), every layer on a scale of its own between 1e-5 and 1e-2; the carried residual (Eq. 12) is what
several earlier gradients add up to, without the entries so large that they would have been sent.  The plan's
workspace has seen a dozen calls, as in a running training: the first calls with a workspace are a start-up.
Nothing of the method's arithmetic is taken from the package: `exact` has its own, in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2312_17530_amd import binding, synth

DEVICE = "cuda:0"
WARM_CALLS = 12          # the first ten calls with a workspace sample their bounds


# ------------------------------------------------------------------ shapes
def _shapes(case):
    """[(rows, cols)], [p] of the case's layers."""
    net, p = case["net"], case["p"]
    if net == "layer":
        sh = [(case["rows"], case["cols"])]
    elif net == "resnet18":
        sh = synth.resnet18_shapes(case["classes"])
    elif net == "resnet50":
        sh = synth.resnet50_shapes(case["classes"])
    elif net == "vgg19":
        sh = synth.vgg19_shapes(case["classes"])
    elif net == "resnet50_all":
        # p follows the kernel's side (7 for conv1, 3 and 1 for the others); a scale and a shift vector per
        # convolution, a bias for the head
        sh, ps = [], []
        convs = synth.resnet50_shapes(case["classes"])
        in_block = 0
        for i, (r, c) in enumerate(convs):
            side = 1
            if i == 0:
                side = 7
            elif c % 9 == 0 and r * 9 == c:          # a 3x3 convolution keeps the number of channels
                side = 3
            sh.append((r, c))
            ps.append(side)
            last = i == len(convs) - 1
            for _ in range(1 if last else 2):
                sh.append((1, r))
                ps.append(1)
        return sh, ps
    elif net == "stack":
        rng = np.random.default_rng(case["shape_seed"])
        sh = []
        for _ in range(case["n_layers"]):
            r, c = (int(round(2.0 ** x)) for x in rng.uniform(4.0, 10.5, size=2))
            sh.append((r, c))
    else:
        raise ValueError(net)
    return sh, [p] * len(sh)


def _ratios(case, shapes):
    """One ratio for all layers, or ratios scattered around rho as the per-epoch refresh leaves them (Eq. 5)."""
    if not case.get("spread"):
        return [case["rho"]] * len(shapes)
    return synth.dynamic_ratios(shapes, case["rho"], 4)


# ------------------------------------------------------------------- cases
def _case(name, net, call, p, rho, alpha=0.5, classes=45, **more):
    c = {"net": net, "call": call, "p": p, "rho": rho, "alpha": alpha, "classes": classes}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small layer: what a call costs before any data moves
        _case("layer_512x512", "layer", "compress", 3, 0.02, rows=512, cols=512),
        # a small network, one ratio for all layers
        _case("resnet18", "resnet18", "compress", 3, 0.01),
        # an ordinary network of many layers with per-layer ratios
        _case("resnet50", "resnet50", "compress", 3, 0.02, spread=True),
        # every parameter of that network, odd head, p after the kernel's side (Section III-C), centre lists wanted
        _case("resnet50_all_centres", "resnet50_all", "compress", 3, 0.02, classes=21, spread=True, centres=True),
        # the benchmark's network
        _case("vgg19", "vgg19", "compress", 3, 0.02, spread=True),
        # ... with Eq. 12 in full, as the paper trains (momentum 0.9)
        _case("vgg19_momentum", "vgg19", "momentum", 3, 0.02, spread=True),
        # ... where memory allows one residual arena only
        _case("vgg19_in_place", "vgg19", "in_place", 3, 0.02, spread=True),
        # ... in the block reading of the method
        _case("vgg19_blocks", "vgg19", "blocks", 3, 0.02, spread=True),
        # one very large layer, strong compression, heavy tails, wide neighbourhoods
        _case("fc_25088x4096_p5", "layer", "compress", 5, 0.001, rows=25088, cols=4096, heavy=True),
        # the receiving side: one message back to a dense gradient
        _case("vgg19_decompress", "vgg19", "decompress", 3, 0.02, spread=True),
        # ... and the update of the weights from the messages of eight nodes
        _case("vgg19_apply8", "vgg19", "apply", 3, 0.02, spread=True, n_msgs=8),
        # the per-epoch step: keep ratios from the weights (Eqs. 3-5)
        _case("vgg19_ratios", "vgg19", "ratios", 3, 0.02),
    ]


def draw(rng):
    call = rng.choice(["compress", "compress", "compress", "momentum", "in_place", "blocks", "blocks_momentum",
                       "decompress", "apply", "ratios"])
    rho = 10.0 ** rng.uniform(-3.0, math.log10(0.05))
    alpha = rng.choice([0.5, 0.5, 0.25, 1.0])
    p = rng.choice([3, 3, 3, 5, 7, 1])
    more = {}
    if call == "compress" and rng.random() < 0.3:
        more["centres"] = True
    if call == "apply":
        more["n_msgs"] = rng.choice([1, 2, 4, 8])
    net = rng.choice(["layer", "layer", "stack", "resnet18", "resnet50", "resnet50_all", "vgg19"])
    if net == "layer":
        while True:
            r, c = (int(round(2.0 ** rng.uniform(4.0, 14.5))) for _ in range(2))
            if 2048 <= r * c <= 60_000_000:
                break
        return _case("", net, call, p, rho, alpha, rows=r, cols=c, heavy=rng.random() < 0.3, **more)
    if net == "stack":
        return _case("", net, call, p, rho, alpha, n_layers=rng.randint(3, 120), shape_seed=rng.randrange(1 << 20),
                     spread=rng.random() < 0.5, **more)
    classes = rng.randint(2, 400)
    if net == "vgg19":                         # (no larger than the listed ones)
        p, rho, classes = 3, min(rho, 0.02), min(classes, 45)
    return _case("", net, call, p, rho, alpha, classes=classes, spread=rng.random() < 0.5, **more)


# ------------------------------------------------------------------ inputs
def _gen(seed, salt):
    return torch.Generator(device=DEVICE).manual_seed((int(seed) * 1000003 + salt) & 0x7fffffff)


def _field(shape, g, heavy):
    """Noise plus a smooth field, both of standard deviation one (t-distributed noise when heavy)."""
    R, C = shape
    z = torch.randn(R, C, device=DEVICE, generator=g)
    if heavy:                                  # Student t with 3 degrees of freedom
        chi = torch.zeros_like(z)
        for _ in range(3):
            chi.add_(torch.randn(R, C, device=DEVICE, generator=g).square_())
        z.div_(chi.div_(3.0).sqrt_().add_(1e-6))
    coarse = torch.randn(1, 1, R // 8 + 2, C // 8 + 2, device=DEVICE, generator=g)
    b = torch.nn.functional.interpolate(coarse, size=(R, C), mode="bilinear", align_corners=False)[0, 0]
    return z.add_(b, alpha=1.5)                # (bilinear interpolation leaves two thirds of the deviation)


def _layout(shapes):
    """Arena offsets: every layer starts at a multiple of 64 elements."""
    offs, o = [], 0
    for r, c in shapes:
        offs.append(o)
        o += (r * c + 63) // 64 * 64
    return offs, o


def _scales(n, seed):
    rng = np.random.default_rng([int(seed), 77])
    return [float(x) for x in 10.0 ** rng.uniform(-5.0, -2.0, size=n)]


def _arenas(case, seed, shapes):
    """(gradient, residual, momentum) arenas of one node."""
    offs, total = _layout(shapes)
    scales = _scales(len(shapes), seed)
    heavy = bool(case.get("heavy"))
    want_u = case["call"] in ("momentum", "blocks_momentum")
    g = torch.zeros(total, device=DEVICE)
    r = torch.zeros(total, device=DEVICE)
    u = torch.zeros(total, device=DEVICE) if want_u else None
    gen = _gen(seed, 1)
    for (R, C), o, s in zip(shapes, offs, scales):
        n = R * C
        g[o:o + n] = _field((R, C), gen, heavy).mul_(s).reshape(-1)
        old = _field((R, C), gen, heavy).mul_(2.0 * s).reshape(-1)       # four earlier gradients' sum ...
        old[old.abs() > 5.0 * s] = 0.0                                   # ... without what has been sent
        r[o:o + n] = old
        if want_u:
            u[o:o + n] = _field((R, C), gen, heavy).mul_(2.0 * s).reshape(-1)
    return g, r, u


def _weights(seed, shapes):
    offs, total = _layout(shapes)
    w = torch.zeros(total, device=DEVICE)
    gen = _gen(seed, 2)
    for (R, C), o in zip(shapes, offs):
        n = R * C
        w[o:o + n] = torch.randn(n, device=DEVICE, generator=gen).mul_(math.sqrt(2.0 / max(1, C)))
    return w


ETA, MOMENTUM = 0.1, 0.9


class _State:
    pass


def prepare(case, seed):
    shapes, ps = _shapes(case)
    ratios = _ratios(case, shapes)
    call = case["call"]
    s = _State()
    s.call, s.case = call, case
    if call in ("blocks", "blocks_momentum"):
        s.plan = binding.rsdgc_plan_blocks(shapes, 3, case["alpha"], ratios, ps)
    else:
        s.plan = binding.rsdgc_plan(shapes, 3, case["alpha"], ratios, ps)
    plan = s.plan
    s.workspace = torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device=DEVICE)
    if call == "ratios":
        s.weights = _weights(seed, shapes)
        return s
    n_pairs, n_centres = max(1, plan.out_capacity), max(1, plan.centre_capacity)
    plan_is_blocks = call in ("blocks", "blocks_momentum")
    s.want_centres = bool(case.get("centres")) and not plan_is_blocks

    def outputs():
        idx = torch.zeros(n_centres if plan_is_blocks else n_pairs, dtype=torch.int32, device=DEVICE)
        return idx, torch.zeros(n_pairs, device=DEVICE), torch.zeros(len(shapes), dtype=torch.int32, device=DEVICE)

    s.centre_idx = torch.zeros(n_centres, dtype=torch.int32, device=DEVICE) if s.want_centres else None
    s.centre_counts = torch.zeros(len(shapes), dtype=torch.int32, device=DEVICE) if s.want_centres else None
    if call in ("decompress", "apply"):
        # the messages that came in: each node compressed its own gradient
        s.messages = []
        for k in range(case.get("n_msgs", 1)):
            g, r, _ = _arenas(case, seed + 7919 * k, shapes)
            msg = outputs()
            binding.rsdgc_compress(plan, g, r, torch.empty_like(r), *msg, s.workspace)
            s.messages.append(msg)
        if call == "apply":
            s.weights = _weights(seed, shapes)
        else:
            s.dense = torch.zeros_like(r)
        return s
    s.grad, s.residual, s.momentum = _arenas(case, seed, shapes)
    s.out = outputs()
    s.residual_out = torch.zeros_like(s.residual)
    s.momentum_out = torch.zeros_like(s.momentum) if s.momentum is not None else None
    in_place, s.call = call == "in_place", "compress" if call == "in_place" else call
    for _ in range(WARM_CALLS):
        run(s)
    s.call = call
    if in_place:
        s.residual_out = None
    return s


# -------------------------------------------------------------------- runs
def run(s):
    """One call, as a training step (or a receiving node, or the per-epoch refresh) makes it.  With two arenas the
    caller would swap them afterwards; here the same step is taken again.  In place the residual goes on from pass to
    pass, as do the weights that messages are applied to."""
    call = s.call
    if call == "compress":
        binding.rsdgc_compress(s.plan, s.grad, s.residual, s.residual_out, *s.out, s.workspace, s.centre_idx, s.centre_counts)
        return (*s.out, s.residual_out) + ((s.centre_idx, s.centre_counts) if s.want_centres else ())
    if call == "in_place":
        binding.rsdgc_compress(s.plan, s.grad, s.residual, s.residual, *s.out, s.workspace)
        return (*s.out, s.residual)
    if call == "momentum":
        binding.rsdgc_compress_momentum(s.plan, s.grad, s.momentum, s.momentum_out, MOMENTUM, s.residual, s.residual_out,
                                        *s.out, s.workspace)
        return (*s.out, s.residual_out, s.momentum_out)
    if call == "blocks":
        binding.rsdgc_compress_blocks(s.plan, s.grad, s.residual, s.residual_out, *s.out, s.workspace)
        return (*s.out, s.residual_out)
    if call == "blocks_momentum":
        binding.rsdgc_compress_blocks_momentum(s.plan, s.grad, s.momentum, s.momentum_out, MOMENTUM, s.residual,
                                               s.residual_out, *s.out, s.workspace)
        return (*s.out, s.residual_out, s.momentum_out)
    if call == "decompress":
        binding.rsdgc_decompress(s.plan, *s.messages[0], s.dense, False, s.workspace)
        return s.dense
    if call == "apply":
        binding.rsdgc_apply(s.plan, s.messages, s.weights, ETA, s.workspace)
        return s.weights
    return np.array(binding.rsdgc_dynamic_ratios(s.plan, s.weights, s.case["rho"], s.workspace))


def _keep(G, p, rho):
    return max(0, min(G, math.ceil((G / (p * p)) * rho)))


def work(case):
    """Bytes: each arena that the call reads or writes once, the message once.  Operations: the three window sums
    (rows, then columns) and the score of every neighbourhood."""
    shapes, ps = _shapes(case)
    ratios = _ratios(case, shapes)
    G = sum(r * c for r, c in shapes)
    ks = [_keep(r * c, p, rho) for (r, c), p, rho in zip(shapes, ps, ratios)]
    pairs = sum(min(k * p * p, r * c) for k, p, (r, c) in zip(ks, ps, shapes))
    call = case["call"]
    nsi_flops = sum(r * c * (6 * (p - 1) + 12) for (r, c), p in zip(shapes, ps))
    if call in ("compress", "in_place"):
        return {"bytes": 12 * G + 8 * pairs + (4 * sum(ks) if case.get("centres") else 0), "flops": nsi_flops}
    if call == "momentum":
        return {"bytes": 20 * G + 8 * pairs, "flops": nsi_flops}
    if call in ("blocks", "blocks_momentum"):
        msg = sum(k * (4 + 4 * p * p) for k, p in zip(ks, ps))
        return {"bytes": (20 if call == "blocks_momentum" else 12) * G + msg, "flops": 5 * G}
    if call == "decompress":
        return {"bytes": 4 * G + 8 * pairs, "flops": 0}
    if call == "apply":
        n = case["n_msgs"]
        named = sum((r * c) * (1.0 - (1.0 - min(1.0, k * p * p / (r * c))) ** n) for k, p, (r, c) in zip(ks, ps, shapes))
        return {"bytes": 8 * n * pairs + 8 * int(named), "flops": n * pairs + 2 * int(named)}
    return {"bytes": 4 * G, "flops": 0}


def tolerance(case):
    """Values and residuals are copies of the float32 sum r + g, indices and counts are whole numbers, and sums of
    messages have their order laid down: all of it comes out the same to the bit."""
    return "exact"


# ------------------------------------------------------------------- exact
def _scores(v, p, alpha):
    """Eqs. 8-10 at every element, zero outside the matrix, in 64 bits, rounded once to the float32 they are ranked as."""
    R, C = v.shape
    h, n = (p - 1) // 2, float(p * p)
    pad = torch.nn.functional.pad(v.double()[None, None], (h, h, h, h))[0, 0]
    sa = torch.zeros(R, C, dtype=torch.float64, device=v.device)
    ss = torch.zeros_like(sa)
    for dx in range(p):
        for dy in range(p):
            w = pad[dx:dx + R, dy:dy + C]
            sa += w.abs()
            ss += w
    m = ss / n
    ss.zero_()
    for dx in range(p):
        for dy in range(p):
            ss += (pad[dx:dx + R, dy:dy + C] - m).square_()
    return (alpha * (sa / n) + (1.0 - alpha) * (ss / n).sqrt()).float()


def _block_scores(v, p, alpha):
    R, C = v.shape
    BR, BC = -(-R // p), -(-C // p)
    w = torch.nn.functional.pad(v.double()[None, None], (0, BC * p - C, 0, BR * p - R))[0, 0]
    w = w.reshape(BR, p, BC, p).permute(0, 2, 1, 3).reshape(BR, BC, p * p)
    m = w.mean(-1, keepdim=True)
    return (alpha * w.abs().mean(-1) + (1.0 - alpha) * (w - m).square().mean(-1).sqrt()).float()


def _top(scores, k):
    """The k best scores as a mask, equal scores by the lower index."""
    bits = scores.reshape(-1).view(torch.int32)
    if k <= 0:
        return torch.zeros_like(bits, dtype=torch.bool)
    lo, hi = 0, 0x7f800000                     # lo: at least k scores reach it
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if int((bits >= mid).sum()) >= k:
            lo = mid
        else:
            hi = mid
    sel = bits > lo
    tied = (bits == lo).nonzero().reshape(-1)[:k - int(sel.sum())]
    sel[tied] = True
    return sel


def _dilate(sel, R, C, p):
    h = (p - 1) // 2
    pad = torch.nn.functional.pad(sel.reshape(1, 1, R, C).to(torch.uint8), (h, h, h, h))[0, 0]
    out = torch.zeros(R, C, dtype=torch.uint8, device=sel.device)
    for dx in range(p):
        for dy in range(p):
            out |= pad[dx:dx + R, dy:dy + C]
    return out.bool()


def _exact_node(case, seed, shapes, ps, ratios):
    """Per layer: v in 64 bits, kept elements (or blocks), selected centres; and the new momentum arena."""
    g, r, u = _arenas(case, seed, shapes)
    offs, _ = _layout(shapes)
    v64, v32, u64 = r.double() + g.double(), r + g, None
    if u is not None:
        m = torch.tensor(MOMENTUM, dtype=torch.float32)
        u32 = u * m.to(DEVICE) + g
        u64 = u.double() * float(m) + g.double()
        v64, v32 = r.double() + u64, r + u32
    out = []
    for (R, C), p, o, rho in zip(shapes, ps, offs, ratios):
        n = R * C
        v = v32[o:o + n].reshape(R, C)
        k = _keep(n, p, rho)
        if case["call"].startswith("blocks"):
            out.append(_top(_block_scores(v, p, case["alpha"]), k).nonzero().reshape(-1))
        else:
            sel = _top(_scores(v, p, case["alpha"]), k)
            out.append((_dilate(sel, R, C, p).reshape(-1).nonzero().reshape(-1), sel.nonzero().reshape(-1)))
    return v64, u64, out


def exact(case, seed):
    shapes, ps = _shapes(case)
    ratios = _ratios(case, shapes)
    offs, total = _layout(shapes)
    ks = [_keep(r * c, p, rho) for (r, c), p, rho in zip(shapes, ps, ratios)]
    call = case["call"]
    if call == "ratios":
        w = _weights(seed, shapes).abs()
        real = torch.cat([w[o:o + r * c] for (r, c), o in zip(shapes, offs)])
        keep = _top(real, math.ceil(case["rho"] * real.numel()))
        got, at = [], 0
        for r, c in shapes:
            got.append(int(keep[at:at + r * c].sum()) / (r * c))
            at += r * c
        return np.array(got)
    if call == "decompress":
        v64, _, kept = _exact_node(case, seed, shapes, ps, ratios)
        dense = torch.zeros(total, dtype=torch.float64, device=DEVICE)
        for (idx, _), o in zip(kept, offs):
            dense[o + idx] = v64[o + idx]
        return dense
    if call == "apply":
        acc = torch.zeros(total, dtype=torch.float64, device=DEVICE)
        for k in range(case["n_msgs"]):
            v64, _, kept = _exact_node(case, seed + 7919 * k, shapes, ps, ratios)
            for (idx, _), o in zip(kept, offs):
                acc[o + idx] += v64[o + idx]
        return _weights(seed, shapes).double() - ETA * acc
    v64, u64, kept = _exact_node(case, seed, shapes, ps, ratios)
    if call.startswith("blocks"):
        caps = [k * p * p for k, p in zip(ks, ps)]
        idx_out = torch.zeros(max(1, sum(ks)), dtype=torch.int32, device=DEVICE)
        val_out = torch.zeros(max(1, sum(caps)), dtype=torch.float64, device=DEVICE)
        counts, ko, vo = [], 0, 0
        for (R, C), p, o, k, cap, blk in zip(shapes, ps, offs, ks, caps, kept):
            BC = -(-C // p)
            d = torch.arange(p, device=DEVICE)
            x = (blk // BC * p)[:, None, None] + d[None, :, None]
            y = (blk % BC * p)[:, None, None] + d[None, None, :]
            inside = ((x < R) & (y < C)).reshape(-1)
            at = (o + x * C + y).reshape(-1)
            idx_out[ko:ko + k] = blk.to(torch.int32)
            val_out[vo:vo + cap][inside] = v64[at[inside]]
            v64[at[inside]] = 0.0
            if u64 is not None:
                u64[at[inside]] = 0.0
            counts.append(int(blk.numel()))
            ko += k
            vo += cap
        res = [idx_out, val_out, torch.tensor(counts, dtype=torch.int32), v64]
        return tuple(res + ([u64] if u64 is not None else []))
    caps = [min(k * p * p, r * c) for k, p, (r, c) in zip(ks, ps, shapes)]
    idx_out = torch.zeros(max(1, sum(caps)), dtype=torch.int32, device=DEVICE)
    val_out = torch.zeros(max(1, sum(caps)), dtype=torch.float64, device=DEVICE)
    cidx = torch.zeros(max(1, sum(ks)), dtype=torch.int32, device=DEVICE)
    counts, at, ko = [], 0, 0
    for o, k, cap, (idx, sel) in zip(offs, ks, caps, kept):
        n = int(idx.numel())
        idx_out[at:at + n] = idx.to(torch.int32)
        val_out[at:at + n] = v64[o + idx]
        v64[o + idx] = 0.0
        if u64 is not None:
            u64[o + idx] = 0.0
        cidx[ko:ko + k] = sel.to(torch.int32)
        counts.append(n)
        at += cap
        ko += k
    res = [idx_out, val_out, torch.tensor(counts, dtype=torch.int32), v64]
    if u64 is not None:
        res.append(u64)
    if case.get("centres"):
        res += [cidx, torch.tensor(ks, dtype=torch.int32)]
    return tuple(res)
