"""The bounding calls that programs built on this framework make, as timed cases.

A verifier holds a network with its root bounds, a set of cuts and a pool of
branch-and-bound domains, and calls the bounding step over and over: bounds of
a batch of domains, their gradients, the 20-iteration projected ascent, the
certifying pass, and once per property the intermediate bounds.  Networks and
sizes are those of `workloads/` and `bench.py`; the drawn cases vary domains,
spec rows, cuts, splits, precision and (for fully connected nets) depth and
width, odd sizes among them.

`exact` evaluates Theorem 3.1 and the ascent of Appendix C.1 in 64-bit torch,
from the inputs alone.
"""
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2208_05740_amd import binding
from workloads import gen

OPT = dict(iters=20, lr_alpha=0.1, lr_mult=0.02, decay=0.9, b1=0.9, b2=0.999, adam_eps=1e-8)
MODES = {"fp32": binding.GCP_MODE_FP32, "bf16": binding.GCP_MODE_BF16}


def _case(name, call, net, B, S=9, cuts=0, K=0, dtype="fp32", **kw):
    c = dict(name=name, call=call, net=net, B=B, S=S, cuts=cuts, K=K, dtype=dtype)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one domain of a toy net, bound and gradients; launches and latency
        _case("grad_mlp8", "grad", "mlp8", 1, S=2, cuts=8),
        # the root of a property: one domain, no splits and no cuts yet, the whole ascent; latency of ~300 launches
        _case("optimize_mlp784_root", "optimize", "mlp784", 1, iters=20),
        # a solver's own ascent step over an early, ragged batch of domains, in the fast precision
        _case("grad_mlp784_ragged_bf16", "grad", "mlp784", 37, cuts=200, K=8, dtype="bf16"),
        # one bounding step of a full branch-and-bound batch (the benchmark's configuration), both precisions
        _case("optimize_mlp784", "optimize", "mlp784", 1024, cuts=200, K=8, iters=20),
        _case("optimize_mlp784_bf16", "optimize", "mlp784", 1024, cuts=200, K=8, dtype="bf16", iters=20),
        # re-certifying a large pool of stored domains with outward rounding: the bound pass alone
        _case("certify_mlp784_outward", "bound", "mlp784", 4096, cuts=200, K=8, outward=True),
        # uneven instances verified side by side
        _case("optimize_batch_mlp", "batch", "batch", 256, cuts=100, K=8, instances=8, iters=20),
        # convolutional nets: gradients of a small batch, the full benchmark batch, ...
        _case("grad_cnn", "grad", "cnn", 128, cuts=500, K=8),
        _case("optimize_cnn", "optimize", "cnn", 2048, cuts=500, K=8, iters=20),
        # ... and residual nets, where the convolutions are most of the work
        _case("grad_resnet", "grad", "resnet", 1024, cuts=1000, K=8),
        _case("optimize_resnet_bf16", "optimize", "resnet", 512, cuts=1000, K=8, dtype="bf16", iters=20),
        # intermediate bounds of a new property, layer by layer
        _case("crown_cnn", "crown", "cnn", 1, S=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["grad", "grad", "bound", "optimize", "optimize", "batch", "crown"])
    dtype = rng.choice(["fp32", "fp32", "bf16"])
    if call == "batch":
        return _case(None, "batch", "batch", _log(rng, 16, 256), S=rng.randint(1, 9), cuts=rng.randint(1, 200), K=8,
                     instances=rng.randint(2, 8), iters=20, draw=rng.randrange(1 << 20))
    net = rng.choice(["mlp", "mlp784", "cnn", "resnet"]) if call != "crown" else rng.choice(["mlp", "mlp784", "cnn"])
    c = _case(None, call, net, 1, dtype=dtype)
    if net == "mlp":
        c.update(d0=rng.choice([784, 3072]), width=_log(rng, 33, 700), depth=rng.randint(2, 7))
    if call == "crown":
        c.update(dtype="fp32", S=1, draw=rng.randrange(1 << 20))
        return c
    top = {"mlp": 1024, "mlp784": 1024, "cnn": 1024, "resnet": 512 if call != "optimize" else 128}[net]
    c.update(B=_log(rng, 1, top), S=rng.randint(1, 9), cuts=rng.choice([0, _log(rng, 1, 1000), 200]),
             K=rng.choice([0, rng.randint(1, 12), 8]))
    if call == "optimize":
        c["iters"] = 20
        if net == "mlp":      # interval bounds: too loose for an ascent in the fast precision
            c["dtype"] = "fp32"
    if call == "bound":
        c["outward"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------ inputs
@lru_cache(maxsize=None)
def _stored(name):
    """A workload's network with its stored CROWN root bounds: the model a program has loaded."""
    net, x0, eps = gen.workload_net(name)
    return net, x0, eps, gen.load_root_bounds(name, 0, net, x0, eps)


@lru_cache(maxsize=8)
def _mlp(dims, eps, w_var, tag):
    """A fully connected network of a case with interval root bounds; like a stored one it belongs to the case, and
    the seed gives the property and the domains on it."""
    rng = np.random.default_rng([11, tag])
    net = gen.mlp_net(rng, list(dims), w_var_num=w_var)
    x0 = rng.random(dims[0]).astype(np.float32).astype(np.float64)
    return net, x0, eps, gen.ibp_bounds(net, x0, eps)


def _spec(net, S, rng):
    """A property: up to S rows e_y - e_j of one class y against others, in any order."""
    d = net.nodes[-1].size
    y, *others = rng.permutation(d)
    C = np.zeros((min(S, d - 1), d))
    C[:, y] = 1.0
    C[np.arange(C.shape[0]), others[:C.shape[0]]] = -1.0
    return C


class _Inputs:
    """One problem (network, root bounds, box, spec rows, splits, cuts) and its starting multipliers."""

    def __init__(self, net, lu, x0, eps, C, B, K, n_cuts, root, rng):
        self.net, self.lu, self.x0, self.eps, self.C = net, lu, x0, float(eps), C
        rel = net.relu_nodes
        self.splits = _splits(rng, lu, rel, B, K)
        self.cuts = gen.make_cuts(rng, lu, rel, n_cuts, 2, 6) if n_cuts else gen.Cuts.empty()
        self.B, self.S, self.K, self.N = B, C.shape[0], K, self.cuts.n
        M, S = B * C.shape[0], C.shape[0]
        used = np.repeat(self.splits.node >= 0, S, axis=0)
        f32 = np.float32
        self.beta = rng.random((M, K), dtype=f32) * used.astype(f32)
        crown = gen.crown_alpha_init(lu).astype(f32)
        if root:        # the start of a property: CROWN-adaptive slopes, no cut active yet
            self.alpha = np.broadcast_to(crown, (M, crown.size))
            self.gamma = np.zeros((M, self.N), f32)
        else:           # inside an ascent, or a child that starts from its parent's: about half of the cuts active
            self.alpha = np.broadcast_to(crown, (M, crown.size)) * f32(0.4) + rng.random((M, crown.size), dtype=f32) * f32(0.6)
            self.gamma = np.maximum(rng.random((M, self.N), dtype=f32) * f32(0.8) - f32(0.4), f32(0))

    def on(self, dev):
        return (torch.tensor(np.ascontiguousarray(a), device=dev) for a in (self.alpha, self.beta, self.gamma))


def _splits(rng, lu, relu_nodes, B, K):
    """Each domain splits 1..K distinct root-unstable neurons, on a random side."""
    node = np.concatenate([np.full(int(((l < 0) & (u > 0)).sum()), p, np.int32) for p, (l, u) in zip(relu_nodes, lu)])
    neuron = np.concatenate([np.nonzero((l < 0) & (u > 0))[0] for l, u in lu]).astype(np.int32)
    K = min(K, neuron.size)
    if K == 0:
        return gen.Splits(np.zeros((B, 0), np.int32), np.zeros((B, 0), np.int32), np.zeros((B, 0), np.int8))
    step = max(1, neuron.size // K)          # one neuron out of each of K strides: distinct without a search
    pick = np.arange(K)[None, :] * step + rng.integers(0, step, (B, K))
    live = np.arange(K)[None, :] < rng.integers(1, K + 1, (B, 1))
    sign = np.where(rng.random((B, K)) < 0.5, 1, -1)
    return gen.Splits(np.where(live, node[pick], -1).astype(np.int32), np.where(live, neuron[pick], 0).astype(np.int32),
                      np.where(live, sign, 0).astype(np.int8))


def _instances(case):
    """Width, depth and domains of each network of a batch."""
    shape = np.random.default_rng([7, case.get("draw", 0)])
    out = []
    for _ in range(case["instances"]):
        width, depth = int(shape.integers(64, 513)), int(shape.integers(2, 6))
        lo, hi = math.log(max(1, case["B"] // 16)), math.log(case["B"])
        out.append((width, depth, max(1, int(round(math.exp(shape.uniform(lo, hi)))))))
    return out


def _model(case):
    """Network, centre, radius and root bounds of a case with one network."""
    if case["net"] == "mlp8":
        return _mlp((8, 16, 16, 3), 0.05, 1.0, 8)
    if case["net"] == "mlp":
        d0 = case["d0"]
        return _mlp((d0,) + (case["width"],) * case["depth"] + (10,), 0.015 if d0 == 784 else 2.0 / 255.0, 2.0, d0)
    return _stored(case["net"])


def _inputs(case, seed):
    """The problems of a case, from the seed alone (one; several for a batch)."""
    rng = np.random.default_rng([seed, case.get("draw", 0)])
    root = case["call"] == "crown" or (case["call"] == "optimize" and case["B"] == 1)
    if case["net"] == "batch":
        models = [(_mlp((784,) + (w,) * n + (10,), 0.015, 2.0, i), B) for i, (w, n, B) in enumerate(_instances(case))]
    else:
        models = [(_model(case), case["B"])]
    out = []
    for (net, x0, eps, lu), B in models:
        if case["call"] == "crown":          # a new property: another centre
            x0 = rng.random(x0.size).astype(np.float32).astype(np.float64)
        out.append(_Inputs(net, lu, x0, eps, _spec(net, case["S"], rng), B, case["K"], case["cuts"], root, rng))
    return out


class _Held:
    """What a program holds on the device for one problem."""

    def __init__(self, inp, dev, mode, ascent, iters):
        self.net = binding.Net(inp.net, inp.lu)
        self.cuts = binding.Cuts(self.net, inp.cuts) if inp.N else None
        self.splits = binding.Splits(self.net, inp.splits)
        self.x0 = torch.tensor(inp.x0, dtype=torch.float64, device=dev)
        self.C = torch.tensor(inp.C, dtype=torch.float64, device=dev)
        self.eps, self.S = inp.eps, inp.S
        self.start = tuple(inp.on(dev))
        if ascent:
            M = inp.B * inp.S
            self.alpha, self.beta, self.gamma = (torch.empty_like(t) for t in self.start)
            self.state = torch.zeros(binding.adam_state_size(M, self.net.n_I, inp.splits.K, inp.N), device=dev)
            self.bound = torch.empty(M, dtype=torch.float64, device=dev)
            self.verified = torch.empty(M, dtype=torch.uint8, device=dev)
        binding.prepare(self.net, self.S, self.splits, self.cuts, iters=iters, mode=mode)

    def restart(self):
        """A new ascent over these domains: starting multipliers, fresh Adam moments."""
        for t, s in zip((self.alpha, self.beta, self.gamma), self.start):
            t.copy_(s)
        self.state.zero_()

    def results(self):
        return self.bound, self.verified, self.alpha, self.beta, self.gamma


def prepare(case, seed):
    inputs = _inputs(case, seed)
    mode = MODES[case["dtype"]]
    st = dict(call=case["call"], mode=mode, iters=case.get("iters", 0))
    if case["call"] == "crown":
        st.update(net=inputs[0].net, eps=inputs[0].eps,
                  x0=torch.tensor(inputs[0].x0, dtype=torch.float64, device="cuda"))
        return st
    if case.get("outward"):
        st["mode"] = mode | binding.GCP_FLAG_OUTWARD
    held = [_Held(i, "cuda", mode, case["call"] in ("optimize", "batch"), st["iters"]) for i in inputs]
    st["held"] = held
    if case["call"] == "batch":
        st["items"] = [dict(P=h, alpha=h.alpha, beta=h.beta, gamma=h.gamma, state=h.state, bound=h.bound,
                            verified=h.verified) for h in held]
    return st


def run(state):
    call = state["call"]
    if call == "crown":
        return [a for pair in binding.crown_bounds(state["net"], state["x0"], state["eps"]) for a in pair]
    if call == "batch":
        for h in state["held"]:
            h.restart()
        binding.optimize_batch(state["items"], mode=state["mode"], **dict(OPT, iters=state["iters"]))
        return [h.results() for h in state["held"]]
    h = state["held"][0]
    if call == "optimize":
        h.restart()
        binding.optimize(h.net, h.x0, h.eps, h.C, h.splits, h.cuts, h.alpha, h.beta, h.gamma, h.state,
                         mode=state["mode"], bound_out=h.bound, verified_out=h.verified,
                         **dict(OPT, iters=state["iters"]))
        return h.results()
    out, ver, grads = binding.bound(h.net, h.x0, h.eps, h.C, h.splits, h.cuts, *h.start, mode=state["mode"],
                                    grads=call == "grad", verified=True)
    return (out, ver) + (grads or ())


# ------------------------------------------------------------------ work
def _macs(net):
    """Multiply-adds of one row through every edge but the output's (folded into the spec rows)."""
    total = 0
    for n in net.nodes[:-1]:
        for e in n.edges:
            if e.kind == "dense":
                total += e.W.size
            elif e.kind == "conv":
                total += e.W.size * n.shape[1] * n.shape[2]
    return total


def _params(net):
    return sum(e.W.size for n in net.nodes for e in n.edges if e.W is not None)


def work(case):
    call, it = case["call"], case.get("iters", 0)
    if case["net"] == "batch":
        tot = dict(bytes=0.0, flops=0.0)
        for width, depth, B in _instances(case):
            w = work(dict(case, net="mlp", d0=784, width=width, depth=depth, B=B, call="optimize"))
            tot = {k: tot[k] + w[k] for k in tot}
        return tot
    if case["net"] in ("mlp", "mlp8"):
        d0, w, depth = (8, 16, 2) if case["net"] == "mlp8" else (case["d0"], case["width"], case["depth"])
        macs = d0 * w + (depth - 1) * w * w
        n_par, n_un = macs + 10 * w, int(0.9 * w * depth)     # interval bounds leave about 0.9 of the neurons unstable
        sizes = [d0] + [w] * depth
        dense = [d0 * w] + [w * w] * (depth - 1)
    else:
        net, _, _, lu = _stored(case["net"])
        macs, n_par, n_un = _macs(net), _params(net), sum(int(((l < 0) & (u > 0)).sum()) for l, u in lu)
        sizes = [net.in_size] + [n.size for n in net.nodes[:-1]]
        dense = [sum(e.W.size * (n.shape[1] * n.shape[2] if e.kind == "conv" else 1) for e in n.edges if e.W is not None)
                 for n in net.nodes[:-1]]
    if call == "crown":      # node k: 2 d_k rows through every edge up to its own
        flops = sum(2.0 * 2 * sizes[k + 1] * sum(dense[:k]) for k in range(len(dense)))
        return dict(bytes=4.0 * n_par + 8 * sizes[0] + 16 * sum(sizes[1:]), flops=flops + 2.0 * dense[0])
    M = case["B"] * case["S"]
    row = 4.0 * (n_un + case["K"] + case["cuts"])
    fixed = 4.0 * n_par + 8 * sizes[0] + 9.0 * M
    if call == "bound":
        return dict(bytes=fixed + M * row, flops=2.0 * M * macs)
    if call == "grad":
        return dict(bytes=fixed + 2 * M * row, flops=4.0 * M * macs)
    return dict(bytes=fixed + 4 * M * row, flops=(2 * it + 1) * 2.0 * M * macs)   # moments written too


# ------------------------------------------------------------------ 64-bit values
def _t(a, dev):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)


class _Dual:
    """The dual objective of Theorem 3.1 in 64 bits for any set of rows."""

    def __init__(self, inp, dev):
        self.inp, self.dev = inp, dev
        net = inp.net
        self.rel = net.relu_nodes
        self.W = {(i, k): _t(e.W, dev) for i, n in enumerate(net.nodes) for k, e in enumerate(n.edges)
                  if e.W is not None}
        self.bias = [_t(n.bias, dev) for n in net.nodes]
        self.l = {p: _t(l, dev) for p, (l, u) in zip(self.rel, inp.lu)}
        self.u = {p: _t(u, dev) for p, (l, u) in zip(self.rel, inp.lu)}
        self.cols, off = {}, 0
        for p in self.rel:
            c = torch.nonzero((self.l[p] < 0) & (self.u[p] > 0)).flatten()
            self.cols[p] = (c, off)
            off += c.numel()
        cu = inp.cuts
        self.cut = {}
        for p in self.rel:
            for kind in (0, 1, 2):
                s = (cu.node == p) & (cu.kind == kind)
                if s.any():
                    self.cut[p, kind] = (torch.as_tensor(cu.cut[s].astype(np.int64), device=dev),
                                         torch.as_tensor(cu.neuron[s].astype(np.int64), device=dev), _t(cu.coef[s], dev))
        self.d = _t(cu.d, dev)
        self.x0, self.C = _t(inp.x0, dev), _t(inp.C, dev)

    def back(self, i, k, e, lam):
        """lam times the matrix of edge k of node i."""
        if e.kind == "identity":
            return lam
        if e.kind == "dense":
            return lam @ self.W[i, k]
        net = self.inp.net
        (co, ho, wo), (ci, hi, wi) = net.nodes[i].shape, net.shape_of(e.src)
        cols = self.W[i, k].reshape(co, -1).T @ lam.reshape(-1, co, ho * wo)
        return torch.nn.functional.fold(cols, (hi, wi), e.W.shape[2:], padding=e.pad, stride=e.stride).flatten(1)

    def cut_sum(self, p, kind, gamma, size):
        out = torch.zeros(gamma.shape[0], size, dtype=torch.float64, device=self.dev)
        if (p, kind) not in self.cut:
            return out
        k, j, c = self.cut[p, kind]
        return out.index_add(1, j, gamma[:, k] * c)

    def value(self, rows, alpha, beta, gamma):
        inp, net = self.inp, self.inp.net
        dom = torch.div(rows, inp.S, rounding_mode="floor")
        sp = inp.splits
        lam = self.C[rows % inp.S]
        g = lam @ self.bias[-1] - gamma @ self.d
        acc = {}

        def push(i, lam):
            for k, e in enumerate(net.nodes[i].edges):
                t = self.back(i, k, e, lam)
                acc[e.src] = acc[e.src] + t if e.src in acc else t

        push(len(net.nodes) - 1, lam)
        for p in reversed(self.rel):
            size, l, u = net.nodes[p].size, self.l[p], self.u[p]
            ah = acc.pop(p) + self.cut_sum(p, 1, gamma, size)
            t, s = self.cut_sum(p, 0, gamma, size), self.cut_sum(p, 2, gamma, size)
            cls = torch.where(l >= 0, 1, torch.where(u <= 0, 0, 2)).expand(rows.numel(), size)
            if sp.K and (sp.node == p).any():
                cls = cls.clone()
                node = torch.as_tensor(sp.node, device=self.dev)[dom]
                r, k = torch.nonzero(node == p, as_tuple=True)
                j = torch.as_tensor(sp.neuron.astype(np.int64), device=self.dev)[dom][r, k]
                sg = torch.as_tensor(sp.sign.astype(np.int64), device=self.dev)[dom][r, k]
                cls[r, j] = (sg > 0).long()
                t = t.index_put((r, j), -sg.double() * beta[r, k], accumulate=True)
            cols, off = self.cols[p]
            a = torch.zeros_like(ah).index_copy(1, cols, alpha[:, off:off + cols.numel()])
            n, pos = torch.relu(-ah), torch.relu(ah)
            zero = s >= u * n
            full = ~zero & (s <= l * n)
            mid = (u * n - s) / torch.where(u > l, u - l, torch.ones_like(u))
            none = torch.zeros_like(n)
            pi = torch.where(zero, none, torch.where(full, n, mid))
            h = torch.where(zero, none, torch.where(full, s, l * mid))
            lam = torch.where(cls == 1, ah, torch.where(cls == 0, none, a * pos - pi))
            # cut coefficients on x and the split terms enter every class
            lam = lam + t
            g = g + lam @ self.bias[p] + torch.where(cls == 1, s, torch.where(cls == 2, h, none)).sum(1)
            push(p, lam)
        v = acc[-1]
        return g + v @ self.x0 - inp.eps * v.abs().sum(1)

    def evaluate(self, alpha, beta, gamma, grads, chunk):
        """Bounds of all rows, and the gradients of their sum."""
        out, ga = [], []
        for r0 in range(0, alpha.shape[0], chunk):
            rows = torch.arange(r0, min(alpha.shape[0], r0 + chunk), device=self.dev)
            par = [x[r0:r0 + chunk].detach().requires_grad_(grads) for x in (alpha, beta, gamma)]
            with torch.set_grad_enabled(grads):
                g = self.value(rows, *par)
                if grads:
                    ga.append([torch.zeros_like(x) if d is None else d for x, d in
                               zip(par, torch.autograd.grad(g.sum(), par, allow_unused=True))])
            out.append(g.detach())
        return torch.cat(out), [torch.cat(x) for x in zip(*ga)]


def _ascend(dual, par, iters, chunk):
    m = [[torch.zeros_like(p), torch.zeros_like(p)] for p in par]
    lr = (OPT["lr_alpha"], OPT["lr_mult"], OPT["lr_mult"])
    b1, b2 = OPT["b1"], OPT["b2"]
    for t in range(iters):
        _, grads = dual.evaluate(*par, True, chunk)
        for k, g in enumerate(grads):
            m[k][0] = b1 * m[k][0] + (1 - b1) * g
            m[k][1] = b2 * m[k][1] + (1 - b2) * g * g
            step = m[k][0] / (1 - b1 ** (t + 1)) / ((m[k][1] / (1 - b2 ** (t + 1))).sqrt() + OPT["adam_eps"])
            par[k] = (par[k] + lr[k] * OPT["decay"] ** t * step).clamp(0.0, 1.0 if k == 0 else math.inf)
    return [dual.evaluate(*par, False, chunk)[0], None] + par


class _Prefix:
    """The network up to node k's pre-activation, with spec rows +e_j and -e_j."""

    def __init__(self, inp, k, lu):
        self.net = gen.Net(inp.net.in_shape, inp.net.nodes[:k] + [gen.Node(inp.net.nodes[k].shape, inp.net.nodes[k].bias,
                                                                        inp.net.nodes[k].edges, relu=False)])
        self.lu, self.x0, self.eps = lu, inp.x0, inp.eps
        eye = np.eye(self.net.nodes[k].size)
        self.C = np.concatenate([eye, -eye])
        self.S, self.splits, self.cuts = self.C.shape[0], inp.splits, gen.Cuts.empty()


def _crown(inp, dev):
    """Layer-by-layer CROWN: every layer's bounds are rows over the layers before it."""
    lu, out = [], []
    for k in inp.net.relu_nodes:
        pre = _Prefix(inp, k, lu)
        alpha = _t(gen.crown_alpha_init(lu), dev).expand(pre.S, -1)
        none = torch.zeros(pre.S, 0, dtype=torch.float64, device=dev)
        g = _Dual(pre, dev).evaluate(alpha, none, none, False, 2048)[0].cpu().numpy()
        l, u = g[:pre.S // 2], -g[pre.S // 2:]
        lu.append((l, u))
        out += [l, u]
    return out


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["call"] == "crown":
        return _crown(_inputs(case, seed)[0], dev)
    conv = case["net"] in ("cnn", "resnet")
    cost = work(case)["flops"]
    if cost > (1e14 if not conv else 2.5e13):
        return None
    res = []
    for inp in _inputs(case, seed):
        dual = _Dual(inp, dev)
        par = [t.double() for t in inp.on(dev)]
        chunk = {"resnet": 512, "cnn": 2048}.get(case["net"], 16384)
        if case["call"] in ("optimize", "batch"):
            res.append(tuple(_ascend(dual, par, case["iters"], chunk)))
            continue
        # with outward rounding the value returned lies below this one, by its rounding slack
        g, grads = dual.evaluate(*par, case["call"] == "grad", chunk)
        res.append((g, None) + tuple(grads))
    return res if case["net"] == "batch" else res[0]
