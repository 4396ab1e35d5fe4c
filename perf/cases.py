"""The workloads whose time this framework is judged by: one pass of each is what a program that trains with D-PSGD
does once per iteration, through the public binding (``Dpsgd.step``, ``grad``, ``mix_step*``, ``mean``).

``listed()`` names them, ``draw(rng)`` gives further ones of the same ranges, ``prepare`` makes what such a program has in
hand (replicas that disagree a little, as they do after the first iteration, and one minibatch per worker), ``run`` is
one pass, ``exact`` is the same pass in plain 64-bit torch, without the bf16 operand rounding of the bf16 models.

A case is a dict of plain values:
  model     "lsq", "softmax", "mlp", "cnn" or "none" (the caller has its own gradient and only mixes)
  widths    the model's widths, "3072-1024-10"; for "none" the number of parameters per worker
  n, batch  workers, samples per worker
  topo      "ring", "torus:RxC", "ring_chord", "complete", "hypercube" (CSR) or "graph" (CSR, unequal degrees)
  bf16      bf16 inputs and bf16 matrix operands
  call      "step" (one call per iteration), "grad_mix" (two calls), and without a model "mix", "mix_swapped",
            "mix_momentum", "mix_static"; the last four are followed by the node average when ``mean`` is set
  in_place  whether the mix overwrites its input (calls without a model)
  tight     rows of d floats without padding, what Dpsgd(n, d, ...) takes by default; else the recommended stride
  shadow    the "bf16_shadow" option
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1705_09056_amd import binding as B

GAMMA = 0.01      # the later step length of the paper's schedule; training stays bounded over any number of passes
MU = 0.9


def _case(name, model, widths, n, batch, topo, bf16, call, in_place=True, tight=False, shadow=False, mean=False):
    c = dict(model=model, widths=widths, n=n, batch=batch, topo=topo, bf16=bf16, call=call, in_place=in_place, tight=tight,
             shadow=shadow, mean=mean)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model on a small ring: launches and latency are all there is
        _case("lsq_ring8", "lsq", "64", 8, 32, "ring", False, "step"),
        # multi-class linear model in fp32
        _case("softmax_ring16", "softmax", "3072-10", 16, 128, "ring", False, "step"),
        # one hidden layer, the larger minibatch
        _case("mlp2_ring32", "mlp", "3072-1024-10", 32, 128, "ring", True, "step"),
        # the flagship: 29 million parameters for each of 64 workers (7.5 GB of replicas), the largest case
        _case("mlp3_ring64", "mlp", "3072-4096-4096-10", 64, 32, "ring", True, "step"),
        # the same on a grid
        _case("mlp3_torus8x8", "mlp", "3072-4096-4096-10", 64, 32, "torus:8x8", True, "step"),
        # the 16-machine runs of the paper's supplement: a ring with a link to the farthest node
        _case("mlp3_chord16", "mlp", "3072-4096-4096-10", 16, 32, "ring_chord", True, "step"),
        # the same kind of network in fp32 arithmetic, gradient and mix called separately
        _case("mlp2_f32_ring16", "mlp", "3072-1024-10", 16, 64, "ring", False, "grad_mix"),
        # 28 x 28 inputs and layer widths that no tile divides, rows without padding, an irregular graph
        _case("mlp3_ragged_graph12", "mlp", "784-500-300-10", 12, 50, "graph", True, "step", tight=True),
        # few workers with a large minibatch each, everyone averages with everyone: products, not weight streaming
        _case("mlp2_batch512_complete8", "mlp", "3072-1024-10", 8, 512, "complete", True, "grad_mix"),
        # the paper's convolutional network on 32 x 32 images at its largest scale
        _case("resnet20_ring112", "cnn", "3-32-32-16-3-10", 112, 32, "ring", True, "grad_mix"),
        # the same kind of network on 28 x 28 grey images: 28, 14 and 7 pixel rows
        _case("cnn28_chord16", "cnn", "1-28-28-16-2-10", 16, 32, "ring_chord", True, "step"),
        # a program with its own gradient: momentum mix over an irregular graph, odd length, then the node average
        _case("mix_momentum_graph24", "none", "1250003", 24, 0, "graph", False, "mix_momentum", mean=True),
    ]


# --------------------------------------------------------------------------------------------------- sizes
def _widths(case):
    return [int(v) for v in case["widths"].split("-")]


def _layout(case):
    """[(kind, offset, shape, fan_in)] of one worker's parameters, layer by layer, each weight followed by its bias."""
    w, out, off = _widths(case), [], 0

    def add(kind, shape, fan):
        nonlocal off
        out.append((kind, off, tuple(shape), fan))
        off += int(np.prod(shape))

    if case["model"] in ("lsq", "none"):
        add("x", (w[0],), 0)
    elif case["model"] in ("softmax", "mlp"):
        for i, o in zip(w[:-1], w[1:]):
            add("w", (o, i), i)
            add("b", (o,), 0)
    else:
        cin, _h, _w, base, blocks, classes = w
        add("w", (base, cin, 3, 3), 9 * cin)
        add("b", (1,), 0)
        prev = base
        for s in range(3):
            c = base << s
            for _ in range(blocks):
                add("w", (c, prev, 3, 3), 9 * prev)
                add("b", (1,), 0)
                add("w2", (c, c, 3, 3), 9 * c)
                add("b", (1,), 0)
                prev = c
        add("w", (classes, prev), prev)
        add("b", (classes,), 0)
    return out, off


def _dim(case):
    return _layout(case)[1]


def _features(case):
    w = _widths(case)
    return w[0] * w[1] * w[2] if case["model"] == "cnn" else w[0]


def _macs(case):
    """(multiply-adds of the forward pass per sample, those of the first layer)."""
    w = _widths(case)
    if case["model"] == "none":
        return 0, 0
    if case["model"] != "cnn":
        parts = [w[0]] if case["model"] == "lsq" else [i * o for i, o in zip(w[:-1], w[1:])]
        return sum(parts), parts[0]
    cin, h, wd, base, blocks, classes = w
    first = 9 * cin * base * h * wd
    total, prev = first, base
    for s in range(3):
        c = base << s
        for j in range(blocks):
            if s and j == 0:
                h, wd = (h + 1) // 2, (wd + 1) // 2
            total += 9 * (prev + c) * c * h * wd
            prev = c
    return total + prev * classes, first


def work(case):
    """What a pass cannot do without: replicas (and gradient, velocity) read once, the results written once, the
    minibatch read once; multiply-adds of forward, data gradient and weight gradient, and of the mix."""
    n, d = case["n"], _dim(case)
    per = {"step": 2, "grad_mix": 4, "mix": 3, "mix_swapped": 3, "mix_static": 3, "mix_momentum": 5}[case["call"]]
    b = 4.0 * per * n * d
    if case["in_place"] and case["call"] == "grad_mix":
        b -= 4.0 * n * d      # G is an output, X an input and an output
    total, first = _macs(case)
    b += n * case["batch"] * (_features(case) * (2.0 if case["bf16"] else 4.0) + 4.0)
    flops = 2.0 * (3 * total - first) * n * case["batch"]
    nnz = len(_weights(case["topo"], n)[1])
    flops += 2.0 * (nnz + n) * d
    if case["mean"]:
        b += 4.0 * d
        flops += float(n) * d
    return {"bytes": b, "flops": flops}


# ------------------------------------------------------------------------------------------ the weight matrix
def _weights(topo, n):
    """(rowptr, colidx, vals) of W: symmetric, doubly stochastic, ascending columns, fp32 values."""
    rows = [dict() for _ in range(n)]
    if topo in ("ring", "ring_chord") or topo.startswith("torus"):
        w = {"ring": 1.0 / 3.0, "ring_chord": 0.25}.get(topo, 1.0 / 5.0)
        if topo.startswith("torus"):
            R, C = (int(v) for v in topo[6:].split("x"))
        for i in range(n):
            if topo.startswith("torus"):
                r, c = divmod(i, C)
                js = (i, (r + 1) % R * C + c, (r - 1) % R * C + c, r * C + (c + 1) % C, r * C + (c - 1) % C)
            else:
                js = (i, (i + 1) % n, (i - 1) % n) + (((i + n // 2) % n,) if topo == "ring_chord" else ())
            for j in js:
                rows[i][j] = rows[i].get(j, 0.0) + w
    elif topo == "complete":
        rows = [{j: 1.0 / n for j in range(n)} for _ in range(n)]
    elif topo == "hypercube":
        k = n.bit_length() - 1
        rows = [{j: 1.0 / (k + 1) for j in [i] + [i ^ (1 << b) for b in range(k)]} for i in range(n)]
    else:      # a ring whose every third node also knows the node two fifths of the way round; Metropolis weights
        links = [set() for _ in range(n)]
        for i in range(n):
            for j in [(i + 1) % n] + ([(i + 2 * n // 5) % n] if i % 3 == 0 else []):
                if j != i:
                    links[i].add(j)
                    links[j].add(i)
        for i in range(n):
            for j in links[i]:
                rows[i][j] = float(np.float32(1.0 / (1 + max(len(links[i]), len(links[j])))))
            rows[i][i] = 1.0 - sum(rows[i].values())
    ptr, col, val = [0], [], []
    for r in rows:
        for j in sorted(r):
            col.append(j)
            val.append(r[j])
        ptr.append(len(col))
    return np.array(ptr, np.int32), np.array(col, np.int32), np.array(val, np.float32)


def _topology(case):
    t, n = case["topo"], case["n"]
    if t.startswith("torus"):
        return B.Topology.torus(*(int(v) for v in t[6:].split("x")))
    if t in ("ring", "ring_chord", "complete"):
        return getattr(B.Topology, t)()
    return B.Topology.csr(*_weights(t, n))


# --------------------------------------------------------------------------------------------------- inputs
def _stride(case):
    d = _dim(case)
    return d if case["tight"] else B.recommended_ld(d, _topology(case))


def _tensors(case, seed, ld):
    """Replicas around one Kaiming-normal starting point, one minibatch per worker labelled by a random linear teacher
    (least squares: y = A x* + noise); without a model a given gradient and velocity.  All on the GPU from the seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    n, d, batch, feat = case["n"], _dim(case), case["batch"], _features(case)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    t = {"X": torch.zeros(n, ld, device="cuda")}
    X = t["X"]
    layout, _ = _layout(case)
    residual_blocks = 3 * _widths(case)[4] if case["model"] == "cnn" else 0
    x0, spread = torch.empty(d, device="cuda"), torch.empty(d, device="cuda")
    for kind, off, shape, fan in layout:
        size = int(np.prod(shape))
        std = math.sqrt(2.0 / fan) if fan else (1.0 if case["model"] == "none" else 0.1)
        if kind == "w2":      # no normalisation layers: keeps the residual sums at unit scale
            std /= math.sqrt(2.0 * residual_blocks)
        x0[off:off + size] = std * normal(size)
        spread[off:off + size] = 0.05 * std
    for i in range(n):
        X[i, :d] = x0 + spread * normal(d)
    if case["model"] == "none":
        t["G"] = torch.zeros(n, ld, device="cuda")
        t["G"][:, :d] = normal(n, d)
        if case["call"] == "mix_momentum":
            t["V"] = torch.zeros(n, ld, device="cuda")
            t["V"][:, :d] = normal(n, d)
        return t
    a = normal(n, batch, feat)
    if case["bf16"]:
        a = a.to(torch.bfloat16)
    t["inputs"] = a
    if case["model"] == "lsq":
        t["targets"] = (a @ normal(feat) + 0.1 * normal(n, batch)).contiguous()
    else:
        classes = _widths(case)[-1]
        teacher = normal(feat, classes)
        t["targets"] = torch.stack([(a[i].float() @ teacher).argmax(dim=1) for i in range(n)]).to(torch.int32)
    return t


def prepare(case, seed):
    d, ld, topo = _dim(case), _stride(case), _topology(case)
    s = dict(_tensors(case, seed, ld), case=case, d=d, ld=ld, topo=topo)
    n = case["n"]
    s["consensus"] = torch.zeros(1, device="cuda")
    if case["mean"]:
        s["xbar"] = torch.zeros(d, device="cuda")
    if not case["in_place"]:
        s["X_out"] = torch.zeros(n, ld, device="cuda")
    s["ctx"] = B.Dpsgd(n, d, topo, GAMMA, ld=ld)
    if case["model"] != "none":
        kind = {"lsq": B.MODEL_LSQ, "softmax": B.MODEL_SOFTMAX, "mlp": B.MODEL_MLP, "cnn": B.MODEL_RESNET20}[case["model"]]
        s["model"] = B.Model(kind, _widths(case), compute_bf16=case["bf16"])
        s["G"] = torch.zeros(n, ld, device="cuda")
        s["loss"] = torch.zeros(n, device="cuda")
        if case["shadow"]:
            s["ctx"].set_option("bf16_shadow", 1)
    return s


# ----------------------------------------------------------------------------------------------------- a pass
def run(s):
    case, ctx, d, X = s["case"], s["ctx"], s["d"], s["X"]
    call = case["call"]
    if call == "step":
        ctx.step(s["model"], X, s["inputs"], s["targets"], case["batch"], s["G"], s["loss"], s["consensus"],
                 input_is_bf16=case["bf16"])
        return {"X": X[:, :d], "loss": s["loss"], "consensus": s["consensus"]}
    if call == "grad_mix":
        ctx.grad(s["model"], X, s["inputs"], s["targets"], case["batch"], s["G"], s["loss"], input_is_bf16=case["bf16"])
        ctx.mix_step(X, s["G"], X, s["consensus"])
        return {"X": X[:, :d], "G": s["G"][:, :d], "loss": s["loss"], "consensus": s["consensus"]}
    out = X if case["in_place"] else s["X_out"]
    got = {"X": out[:, :d], "consensus": s["consensus"]}
    if call == "mix_momentum":
        ctx.mix_step_momentum(X, s["G"], s["V"], MU, out, s["consensus"])
        got["V"] = s["V"][:, :d]
    elif call == "mix_static":
        B.mix_step_static(case["n"], d, s["topo"], GAMMA, X, s["G"], out, s["consensus"], ld=s["ld"])
    else:
        ctx.mix_step(X, s["G"], out, s["consensus"], swapped=call == "mix_swapped")
    if case["mean"]:
        ctx.mean(out, s["xbar"])
        got["xbar"] = s["xbar"]
    return got


# -------------------------------------------------------------------------------------------- the same in 64 bits
def _dense_grad(case, x, a, y):
    """Loss and gradient of one worker's least squares, softmax regression or ReLU network."""
    w, batch = _widths(case), a.shape[0]
    if case["model"] == "lsq":
        r = a @ x - y
        return 0.5 * (r * r).mean(), a.t() @ r / batch
    acts, off, mats = [a], 0, []
    for l, (i, o) in enumerate(zip(w[:-1], w[1:])):
        m, b = x[off:off + o * i].view(o, i), x[off + o * i:off + o * i + o]
        mats.append((off, m))
        off += o * i + o
        z = acts[-1] @ m.t() + b
        acts.append(z.clamp_min(0) if l < len(w) - 2 else z)
    logp = torch.log_softmax(acts[-1], dim=1)
    pick = torch.nn.functional.one_hot(y.long(), w[-1]).to(logp.dtype)
    loss = -(logp * pick).sum(1).mean()
    g = torch.empty_like(x)
    dz = (logp.exp() - pick) / batch
    for l in range(len(mats) - 1, -1, -1):
        off, m = mats[l]
        o, i = m.shape
        g[off:off + o * i] = (dz.t() @ acts[l]).reshape(-1)
        g[off + o * i:off + o * i + o] = dz.sum(0)
        if l:
            dz = (dz @ m) * (acts[l] > 0)
    return loss, g


def _conv(a, wt, bias, stride):
    h, w = ((s + 2 - 3) // stride + 1 for s in a.shape[2:])
    cols = torch.nn.functional.unfold(a, 3, padding=1, stride=stride)
    return (wt.reshape(wt.shape[0], -1) @ cols).view(a.shape[0], wt.shape[0], h, w) + bias


def _cnn_grad(case, x, a, y):
    cin, h, w, base, blocks, _classes = _widths(case)
    x = x.detach().clone().requires_grad_(True)
    p = [x[off:off + int(np.prod(shape))].view(shape) for _, off, shape, _ in _layout(case)[0]]
    act = _conv(a.view(-1, cin, h, w), p[0], p[1], 1).relu()
    k = 2
    for s in range(3):
        for j in range(blocks):
            stride = 2 if s and j == 0 else 1
            u = _conv(act, p[k], p[k + 1], stride).relu()
            skip = act[:, :, ::stride, ::stride]
            if skip.shape[1] < u.shape[1]:
                skip = torch.cat([skip, torch.zeros_like(u[:, skip.shape[1]:])], dim=1)
            act = (_conv(u, p[k + 2], p[k + 3], 1) + skip).relu()
            k += 4
    logits = act.mean((2, 3)) @ p[k].t() + p[k + 1]
    loss = -torch.log_softmax(logits, dim=1).gather(1, y.long()[:, None]).mean()
    (g,) = torch.autograd.grad(loss, x)
    return loss.detach(), g


def exact(case, seed):
    n, d = case["n"], _dim(case)
    t = _tensors(case, seed, _stride(case))
    X = t.pop("X")[:, :d]
    ptr, col, val = _weights(case["topo"], n)
    W = torch.zeros(n, n, dtype=torch.float64)
    for i in range(n):
        W[i, torch.from_numpy(col[ptr[i]:ptr[i + 1]].astype(np.int64))] = torch.from_numpy(val[ptr[i]:ptr[i + 1]]).double()
    W = W.cuda()
    gamma, mu = float(np.float32(GAMMA)), float(np.float32(MU))
    got = {}
    if case["model"] == "none":
        G = t["G"][:, :d].double()
        if case["call"] == "mix_momentum":
            G = mu * t["V"][:, :d].double() + G
            got["V"] = G
    else:
        G = torch.empty(n, d, dtype=torch.float64, device="cuda")
        loss = torch.empty(n, dtype=torch.float64, device="cuda")
        one = _cnn_grad if case["model"] == "cnn" else _dense_grad
        for i in range(n):
            loss[i], G[i] = one(case, X[i].double(), t["inputs"][i].double(),
                                t["targets"][i].double() if case["model"] == "lsq" else t["targets"][i])
        got["loss"] = loss
        if case["call"] == "grad_mix":
            got["G"] = G
    Xn, step = torch.empty(n, d, dtype=torch.float64, device="cuda"), 1 << 22
    xbar, spread = torch.empty(d, dtype=torch.float64, device="cuda"), 0.0
    for c in range(0, d, step):
        x, g = X[:, c:c + step].double(), G[:, c:c + step]
        m = W @ (x - gamma * g) if case["call"] == "mix_swapped" else W @ x - gamma * g
        Xn[:, c:c + step] = m
        xbar[c:c + step] = m.mean(0)
        spread += float((m - m.mean(0)).square().sum())
    got["X"] = Xn
    got["consensus"] = torch.tensor([spread / n], dtype=torch.float64)
    if case["mean"]:
        got["xbar"] = xbar
    return got


def tolerance(case):
    """Two correct implementations differ by the order of their fp32 sums (1e-7, a few 1e-7 for long sums).  In a ReLU
    network such a difference now and then turns one unit's sign or one bf16 rounding around, which moves the gradient
    by up to 7e-4 of its norm in fp32, 2e-3 in bf16, 6e-3 in the deep bf16 CNN (measured against sums in 64 bits) and one
    of its elements by up to half their root mean square.  An iterate feels that times gamma |G| / |X|, about 4e-3;
    on the complete graph the consensus distance consists of gradients alone."""
    grad, cnn = case["call"] == "grad_mix", case["model"] == "cnn"
    if case["model"] in ("lsq", "none") or (case["model"] == "softmax" and not case["bf16"]):
        return {"rel": 2e-6, "max": 2e-5}
    if case["model"] == "softmax":
        t = {"rel": 1e-3, "max": 0.1} if grad else {"rel": 1e-5, "max": 1e-3}
    elif not case["bf16"]:
        t = {"rel": 3e-3, "max": 0.9} if grad else {"rel": 1.3e-5, "max": 4e-3}
    elif grad:
        t = {"rel": 2e-2 if cnn else 1e-2, "max": 0.9}
    else:
        t = {"rel": 1e-4 if cnn else 4e-5, "max": 2e-2}
    if case["topo"] == "complete":
        t["rel"] = max(t["rel"], 1e-3)
    return t


# ------------------------------------------------------------------------------------------------ further cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _topo(rng, most, least=3):
    t = rng.choice(["ring", "ring", "ring", "torus", "ring_chord", "complete", "hypercube", "graph"])
    n = max(least, _log(rng, least, most))
    if t == "torus":
        r, c = max(3, round(math.sqrt(n))), 3 + rng.randrange(6)
        r = max(3, min(r, most // c))
        return "torus:%dx%d" % (r, c), r * c
    if t == "ring_chord":
        n = max(4, n // 2 * 2)
    if t == "hypercube":
        n = 1 << max(2, n.bit_length() - 1)
    if t == "graph":
        n = max(5, n)
    return t, n


def _width(rng, lo, hi):
    w = _log(rng, lo, hi)
    m = rng.choice([1, 1, 32, 256])
    return max(lo, w // m * m)


def _draw(rng):
    family = rng.choice(["lsq", "softmax", "mlp", "mlp", "mlp", "mlp_f32", "cnn", "cnn", "none", "none"])
    tight = rng.random() < 0.25
    if family == "lsq":
        topo, n = _topo(rng, 64)
        return _case(None, "lsq", str(_log(rng, 16, 4096)), n, _log(rng, 8, 256), topo, False,
                     rng.choice(["step", "grad_mix"]), tight=tight)
    if family == "softmax":
        topo, n = _topo(rng, 64)
        return _case(None, "softmax", "%d-%d" % (_width(rng, 64, 4096), rng.choice([2, 5, 10, 10, 10, 26])), n,
                     _log(rng, 16, 256), topo, rng.random() < 0.3, rng.choice(["step", "grad_mix"]), tight=tight)
    if family in ("mlp", "mlp_f32"):
        bf16 = family == "mlp"
        topo, n = _topo(rng, 64)
        hidden = [_width(rng, 64, 4096) for _ in range(rng.choice([1, 1, 2, 2, 3]))]
        widths = [rng.choice([784, 1024, 3072, 3072, _width(rng, 64, 4096)])] + hidden + [rng.choice([2, 10, 10, 10, 26])]
        batch = rng.choice([32, 32, 64, 128, _log(rng, 8, 512)])
        shadow = bf16 and topo == "ring" and rng.random() < 0.25
        # (the gradient itself is an output only where one sample's ReLU decision cannot move an element by its own size)
        call = "step" if shadow or batch < 64 else rng.choice(["step", "grad_mix"])
        return _case(None, "mlp", "-".join(str(w) for w in widths), n, batch, topo, bf16, call, tight=tight, shadow=shadow)
    if family == "cnn":
        topo, n = _topo(rng, 112)
        side = rng.choice([(32, 32), (32, 32), (28, 28), (_log(rng, 8, 48), _log(rng, 8, 48))])
        widths = [rng.choice([1, 3, 3]), side[0], side[1], rng.choice([8, 16, 16, 16, 24]), rng.choice([1, 2, 3, 3]), 10]
        return _case(None, "cnn", "-".join(str(w) for w in widths), n, _log(rng, 8, 64), topo, True,
                     rng.choice(["step", "grad_mix"]), tight=tight)
    topo, n = _topo(rng, 256)
    call = rng.choice(["mix", "mix_momentum", "mix_momentum", "mix_swapped"] +
                      (["mix_static"] if topo == "ring" or topo.startswith("torus") else []))
    return _case(None, "none", str(_log(rng, 1000, 8000000)), n, 0, topo, False, call, in_place=rng.random() < 0.7,
                 tight=tight, mean=rng.random() < 0.5)


# the largest listed cases: bytes of mlp3_ring64, multiply-adds of resnet20_ring112; fp32 arithmetic has a sixteenth of
# the matrix rate, and a network off the tuned sizes a fraction of it
_MOST_BYTES, _MOST_FLOPS = 15e9, 860e9


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        flops = w["flops"] if c["bf16"] and c["model"] == "mlp" else 3 * w["flops"] if c["model"] == "cnn" else 8 * w["flops"]
        if w["bytes"] <= _MOST_BYTES and (c["model"] == "none" or flops <= _MOST_FLOPS):
            return c
