"""The beta gradient written over an input that the bound pass reads last: the call's start may not clear it while
another part of it still reads that input."""
import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import DIMS, _problem
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["gamma", "C", "gamma, one element in"])
@pytest.mark.parametrize("mode", [0, 1])
def test_beta_gradient_over_an_input(over, mode):
    import torch
    from paper_2208_05740_amd import binding as B
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 6, 43, 3)
    P = B.Problem(prob, device=torch.device("cuda:0"))
    t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device="cuda:0")  # noqa: E731
    a, b, c = t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)
    ref, _, grads = B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c, mode=mode, grads=True)
    for _ in range(3):
        buf = torch.zeros(b.numel() + c.numel() + 2 * P.C.numel() + 1, device="cuda:0")
        Cp, cp = P.C, c
        if over == "C":
            Cp = buf[:2 * P.C.numel()].view(torch.float64)
            Cp.copy_(P.C.reshape(-1))
            db = buf[:b.numel()]
        else:
            cp = buf[:c.numel()]
            cp.copy_(c.reshape(-1))
            first = 1 if "one" in over else 0
            db = buf[first:first + b.numel()]
        out = torch.empty_like(ref)
        ha, hc = torch.empty_like(grads[0]), torch.empty_like(grads[2])
        B._check(B.lib().gcp_bound(P.net.h, B._ptr(P.x0), P.eps, Cp.data_ptr(), P.S, P.splits.h, P.cuts.h, B._ptr(a), B._ptr(b),
                                   cp.data_ptr(), mode, B._ptr(out), None, B._ptr(ha), db.data_ptr(), B._ptr(hc), B._stream()))
        torch.cuda.synchronize()
        for x, y in ((out, ref), (ha, grads[0]), (db.view_as(b), grads[1]), (hc, grads[2])):
            assert torch.equal(x, y)
