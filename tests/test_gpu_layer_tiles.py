"""The launch shapes of the layer kernels at the sizes where they can go wrong,
through the C ABI: every dense tile (staged and direct K loops) forced by a
tile file, and conv plans outside the ordinary one (one batch row per slab,
results beside the slab, bands with a remainder), against the FP64 oracle.

Every dense tile accumulates over K in the same order with the same MFMA
instructions and runs the same epilogue, so the gradients must have the same
bits.  A bound's row constant is an fp64 sum of one term per neuron, grouped by
the tile's columns, so bounds may differ by the rounding of its additions: as
many as there are neurons, 2^-53 of T each, in either of the two.  Against the oracle the tolerances are those of the other
parity tests: FP32 bounds within 1e-5 of max(|g|, T) (T the sum of the
magnitudes of the terms added), gradients within 1e-4 of the row's largest,
bf16 bounds within 2e-2 of T.

The networks have a node without any unstable neuron (no alpha, no a_hat) and
a cut on a stable neuron; rows and columns leave remainders of 16, 32 and 64.
"""
import contextlib
import os

import numpy as np
import pytest

from oracle import gcp_oracle as O
from workloads import gen

pytestmark = pytest.mark.gpu

TILES = {0: "64x64", 1: "32x32d", 2: "16x64d", 4: "32x64", 5: "32x32", 6: "16x64", 7: "16x32d"}


def _dev():
    import torch
    return torch.device("cuda:0")


@contextlib.contextmanager
def _tiles(path, lines):
    """Tile choices from a file of their own, no trials."""
    saved = {k: os.environ.get(k) for k in ("GCP_TILE_CACHE", "GCP_AUTOTUNE")}
    path.write_text("".join(lines))
    os.environ["GCP_TILE_CACHE"] = str(path)
    os.environ["GCP_AUTOTUNE"] = "0"
    try:
        yield
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


def _stable_cut(cuts, lu, relu_nodes):
    """Point one cut entry at a stable neuron of its node."""
    for e in range(cuts.node.size):
        if cuts.node[e] < 0:
            continue
        l, u = lu[relu_nodes.index(int(cuts.node[e]))]
        stable = np.flatnonzero((l >= 0) | (u <= 0))
        if stable.size:
            cuts.neuron[e] = stable[0]
            return True
    return False


def _problem(net_of, seed, B, S, eps=0.1, shift=None):
    """net_of(rng) with splits and cuts; node `shift` is made all active by its bias."""
    r_w, r_x, r_cut, r_split, r_par = gen._streams([seed, 97])
    net = net_of(r_w)
    if shift is not None:
        net.nodes[shift].bias[:] = net.nodes[shift].bias + 50.0
    x0 = r_x.random(net.in_size)
    prob = gen.make_problem("tiles", net, x0, eps, S, B, 0, 3, 6, 2, 4, (r_cut, r_split, r_par), alpha_init="given",
                            gamma_dist="uniform", input_terms=1)
    assert _stable_cut(prob.cuts, prob.lu, list(net.relu_nodes))
    return prob


def _bound(prob, mode, path, lines=()):
    import torch
    from paper_2208_05740_amd import binding as B
    with _tiles(path, lines):
        P = B.Problem(prob, device=_dev())
        t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device=_dev())  # noqa: E731
        a, b, c = t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)
        B.profile_enable(True)
        out, ver, g = B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c, mode=mode, grads=True, verified=True)
        torch.cuda.synchronize()
        B.profile_enable(False)
        ran = {k for k, v in B.profile_read().items() if v["launches"]}
    n = lambda x: x.cpu().numpy()  # noqa: E731
    return dict(bound=n(out), ver=n(ver), ga=n(g[0]), gb=n(g[1]), gc=n(g[2])), (n(a), n(b), n(c)), ran


def _check_oracle(prob, got, params, mode):
    f = lambda x: x.astype(np.float64).reshape(prob.B, prob.S, -1)  # noqa: E731
    a, b, c = (f(x) for x in params)
    ref, *grads = O.bound_and_grad(prob, a, b, c)
    ref = ref.reshape(-1)
    T = O.error_scale(prob, a, b, c).reshape(-1)
    err = np.abs(got["bound"] - ref) / np.maximum(np.abs(ref), T)
    assert err.max() <= (2e-2 if mode else 1e-5), err.max()
    if mode:
        return
    for k, want in zip(("ga", "gb", "gc"), grads):
        want = want.reshape(prob.B * prob.S, -1)
        if want.size:
            d = np.abs(got[k].reshape(want.shape) - want) / (np.abs(want).max(1, keepdims=True) + 1.0)
            assert d.max() <= 1e-4, (k, d.max())


DIMS = [19, 33, 47, 65, 17, 5]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,S", [(1, 1), (7, 3), (43, 3)])
def test_dense_tiles_agree_and_match_oracle(B, S, mode, tmp_path):
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 5, B, S, shift=1)
    M = B * S
    res = {}
    for cfg, name in TILES.items():
        print(f"dense tile {name}: M={M} mode={mode}", flush=True)
        lines = [f"gemm.k{k}.b{mode}.s{s}.M{M}.N{n}.K{d} {cfg}\n" for k in range(5) for s in (0, 1) for n in DIMS for d in DIMS]
        res[cfg], params, ran = _bound(prob, mode, tmp_path / f"t{cfg}.txt", lines)
        gemms = [k for k in ran if ".t" in k]
        assert gemms and all(k.split(".t")[-1] == name for k in gemms), sorted(ran)
    _check_oracle(prob, res[5], params, mode)
    f = lambda x: x.astype(np.float64).reshape(prob.B, prob.S, -1)  # noqa: E731
    T = O.error_scale(prob, *(f(x) for x in params)).reshape(-1)
    for cfg in TILES:
        assert (np.abs(res[cfg]["bound"] - res[5]["bound"]) <= sum(DIMS) * 2.0**-52 * T).all(), TILES[cfg]
        for k in ("ga", "gb", "gc"):
            assert np.array_equal(res[cfg][k], res[5][k]), (TILES[cfg], k)


def _conv_net(r, shape, convs, fcs):
    """convs (out channels, kernel, stride, pad) on a c x h x w input, then dense layers."""
    nodes, (c, h, w) = [], shape
    for co, k, s, p in convs:
        h, w = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
        W = gen._conv_w(r, co, c, k)
        nodes.append(gen.Node((co, h, w), gen._bias(r, co * h * w), [gen.Edge(len(nodes) - 1, "conv", W, s, p)]))
        c = co
    d = c * h * w
    for i, n in enumerate(fcs):
        W = gen._f32(r.normal(0.0, np.sqrt(2.0 / d), (n, d)))
        nodes.append(gen.Node((n,), gen._bias(r, n), [gen.Edge(len(nodes) - 1, "dense", W)], relu=i + 1 < len(fcs)))
        d = n
    return gen.Net(shape, nodes)


CONVS = [
    ("row", (3, 4, 800), (2, 4, 2, 1)),       # four rows do not fit one slab: one batch row at a time
    ("beside", (1, 2, 17), (144, 3, 1, 1)),   # more 16x16 items than the waves hold: results beside the slab
    ("band", (2, 13, 11), (5, 3, 2, 1)),      # odd sizes: partial tiles, a last band of fewer rows
]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", range(len(CONVS)))
def test_conv_plans_match_oracle(case, mode, tmp_path):
    name, shape, stem = CONVS[case]
    second = ((3, 3, 1, 1),) if name == "band" else ()
    print(f"conv plan {name}: input {shape}, conv {stem}, mode={mode}", flush=True)
    prob = _problem(lambda r: _conv_net(r, shape, (stem,) + second, (5, 3)), 11 + case, 2, 3, eps=0.02)
    got, params, _ = _bound(prob, mode, tmp_path / "c.txt")
    _check_oracle(prob, got, params, mode)


def test_beta_gradient_into_betas_own_memory():
    """The clearing of d_beta at a call's start leaves beta readable when they share memory."""
    import torch
    from paper_2208_05740_amd import binding as B
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 6, 7, 3)
    P = B.Problem(prob, device=_dev())
    t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device=_dev())  # noqa: E731
    a, b, c = t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)
    ref, _, (ga, gb, gc) = B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c, grads=True)
    out = torch.empty_like(ref)
    ha, hc = torch.empty_like(ga), torch.empty_like(gc)
    B._check(B.lib().gcp_bound(P.net.h, B._ptr(P.x0), P.eps, B._ptr(P.C), P.S, P.splits.h, P.cuts.h, B._ptr(a), B._ptr(b),
                               B._ptr(c), 0, B._ptr(out), None, B._ptr(ha), B._ptr(b), B._ptr(hc), B._stream()))
    torch.cuda.synchronize()
    for x, y in ((out, ref), (ha, ga), (b, gb), (hc, gc)):
        assert torch.equal(x, y)
