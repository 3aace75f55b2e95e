"""The launch at a call's start over more workgroups than one row of its grid holds."""
import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import _problem
from workloads import gen

pytestmark = pytest.mark.gpu


def test_many_spec_rows_over_a_wide_layer():
    """4200 spec rows (two, repeated) through an output layer over 4100 neurons: 71400 workgroups for c-hat alone.
    Every row gives what the two give by themselves, up to the grouping of a row constant's fp64 additions."""
    import torch
    from paper_2208_05740_amd import binding as B
    prob = _problem(lambda r: gen.mlp_net(r, [3, 4100, 3], w_var_num=1.0), 8, 1, 2)
    P = B.Problem(prob, device=torch.device("cuda:0"))
    t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device="cuda:0")  # noqa: E731
    par = [t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)]
    ref, _, _ = B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, *par)
    many = [x.repeat(2100, 1).contiguous() for x in par]
    out, _, _ = B.bound(P.net, P.x0, P.eps, P.C.repeat(2100, 1).contiguous(), P.splits, P.cuts, *many)
    f = lambda x: x.cpu().numpy().astype(np.float64).reshape(prob.B, prob.S, -1)  # noqa: E731
    T = O.error_scale(prob, *(f(x) for x in par)).reshape(-1)
    err = (out.view(2100, 2) - ref).abs().amax(0).cpu().numpy()
    assert (err <= (4100 + 3) * 2.0**-52 * T).all(), (err, T)
