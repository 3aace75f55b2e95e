"""Convolutions at the edge of what fits a workgroup's LDS, as bounds and
gradients through the C ABI, against the FP64 oracle.  Tolerances are those of
the other parity tests: FP32 bounds within 1e-5 of max(|g|, T) (T the sum of
the magnitudes of the terms added), gradients within 1e-4 of the row's largest,
bf16 bounds within 2e-2 of T.
"""
import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import _bound, _check_oracle, _conv_net, _problem

pytestmark = pytest.mark.gpu

# a small input and the convs on it (out channels, kernel, stride, pad)
SHAPES = [
    (1, (2, 32, 32), ((64, 3, 1, 1), (64, 3, 1, 1))),     # bf16: one row's slab fits 64 KB at two bytes an element only
    (1, (3, 16, 16), ((128, 3, 1, 1), (128, 3, 1, 1))),
    (0, (2, 8, 8), ((320, 1, 1, 0), (64, 3, 1, 1))),      # fp32: the adjoint's slab fits, but not with its tables
    (1, (2, 8, 8), ((320, 1, 1, 0), (64, 3, 1, 1))),
    (0, (2, 4, 4), ((512, 1, 1, 0), (64, 3, 1, 1))),
    (0, (2, 32, 32), ((64, 1, 1, 0), (32, 5, 1, 2))),     # one batch row in the slab, more than 64 KB with its results
    (0, (2, 32, 32), ((64, 3, 1, 1), (64, 3, 1, 1))),
    (0, (128, 64, 64), ((32, 1, 1, 0),)),                 # the transposed direction into the input, 142 KB
    (1, (128, 64, 64), ((32, 1, 1, 0),)),
]


@pytest.mark.parametrize("mode,shape,convs", SHAPES)
def test_conv_at_the_lds_limit_matches_oracle(mode, shape, convs, tmp_path):
    print(f"convs {convs} on {shape}, mode={mode}", flush=True)
    prob = _problem(lambda r: _conv_net(r, shape, convs, (3,)), 3, 2, 3, eps=0.01)
    got, params, _ = _bound(prob, mode, tmp_path / "c.txt")
    _check_oracle(prob, got, params, mode)


def test_bf16_ascent_and_its_fp32_certificate_on_plans_of_their_own():
    """A conv whose bf16 and fp32 launches run different bands: the certifying pass gives the bound, bit for bit,
    that a call at the returned parameters gives, on the first ascent and on one over the same buffers."""
    import torch
    from paper_2208_05740_amd import binding as B
    prob = _problem(lambda r: _conv_net(r, (2, 8, 8), ((320, 1, 1, 0), (64, 3, 1, 1)), (3,)), 3, 2, 3, eps=0.01)
    P = B.Problem(prob, device=torch.device("cuda:0"))
    for it in range(2):
        t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device="cuda:0")  # noqa: E731
        a, b, c = t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)
        st = torch.zeros(B.adam_state_size(P.M, a.shape[1], b.shape[1], c.shape[1]), device="cuda:0")
        out, _ = B.optimize(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c, st, iters=4, mode=B.GCP_MODE_BF16)
        again, _, _ = B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c)
        assert torch.isfinite(out).all() and torch.equal(out, again), it
