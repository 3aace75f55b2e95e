"""The tiles with 64-bit addresses, which launches with rows of many million
neurons run, at small sizes: chosen by a tile file (dense 8 to 10, conv 7),
against the FP64 oracle and the layer tiles, with the tolerances of the layer
tiles' own test.  The MFMA sums and the epilogue's arithmetic are the same in
the same order, so gradients and, over conv plans with the same bands, bounds
have the same bits.  (The elementwise relaxation's 64-bit form is the one that
the persistent kernel runs.)
"""
import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import DIMS, _bound, _check_oracle, _conv_net, _problem
from workloads import gen

pytestmark = pytest.mark.gpu

WIDE = {8: "64x64", 9: "32x32", 10: "16x32"}


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,S", [(1, 1), (7, 3), (43, 3)])
def test_dense_64_bit_tiles(B, S, mode, tmp_path):
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 5, B, S, shift=1)
    res = {}
    for cfg in (5, 8, 9, 10):
        print(f"dense tile {cfg}: M={B * S} mode={mode}", flush=True)
        lines = [f"gemm.k{k}.b{mode}.s{s}.M{B * S}.N{n}.K{d} {cfg}\n" for k in range(5) for s in (0, 1) for n in DIMS for d in DIMS]
        res[cfg], params, ran = _bound(prob, mode, tmp_path / f"t{cfg}.txt", lines)
        gemms = [k for k in ran if ".t" in k]
        assert gemms and (cfg == 5 or all(k.split(".t")[-1] == WIDE[cfg] for k in gemms)), sorted(ran)
    _check_oracle(prob, res[9], params, mode)
    f = lambda x: x.astype(np.float64).reshape(prob.B, prob.S, -1)  # noqa: E731
    T = O.error_scale(prob, *(f(x) for x in params)).reshape(-1)
    for cfg in WIDE:
        assert (np.abs(res[cfg]["bound"] - res[5]["bound"]) <= sum(DIMS) * 2.0**-52 * T).all(), cfg
        for k in ("ga", "gb", "gc"):
            assert np.array_equal(res[cfg][k], res[5][k]), (cfg, k)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("shape,stem", [((2, 13, 11), (5, 3, 2, 1)), ((3, 4, 800), (2, 4, 2, 1))])
def test_conv_64_bit_epilogues(shape, stem, mode, tmp_path):
    second = ((3, 3, 1, 1),) if shape[1] == 13 else ()
    prob = _problem(lambda r: _conv_net(r, shape, (stem,) + second, (5, 3)), 11, 2, 3, eps=0.02)
    sizes = [n.size for n in prob.net.nodes] + [prob.net.in_size]
    res = {}
    for cfg in (2, 7):
        print(f"conv choice {cfg}: {shape} mode={mode}", flush=True)
        lines = [f"{fam}.k{k}.b{mode}.s{s}.M6.N{n}.K{d} {cfg}\n" for fam, k in (("convT", 1), ("conv", 3)) for s in (0, 1)
                 for n in sizes for d in sizes]
        res[cfg], params, _ = _bound(prob, mode, tmp_path / f"c{cfg}.txt", lines)
    _check_oracle(prob, res[7], params, mode)
    for k in res[7]:
        assert np.array_equal(res[7][k], res[2][k]), k
