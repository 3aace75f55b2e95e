"""The profiler's operand bytes of the dense launches: every operand read once and every result written once, as the
kernels lay them out -- a_hat of unstable neurons only, row partials only where the row constants are asked for."""
import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import DIMS, _problem
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
def test_operand_bytes_of_an_ascent(mode):
    import torch
    from paper_2208_05740_amd import binding as B
    iters, esz = 3, 2 if mode else 4
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 5, 7, 3, shift=1)
    P = B.Problem(prob, device=torch.device("cuda:0"))
    M, rel = P.M, list(prob.net.relu_nodes)
    t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(M, -1), device="cuda:0")  # noqa: E731
    a, b, c = t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma)
    st = torch.zeros(B.adam_state_size(M, a.shape[1], b.shape[1], c.shape[1]), device="cuda:0")
    B.profile_enable(True)
    B.optimize(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, a, b, c, st, iters=iters, mode=mode)
    torch.cuda.synchronize()
    B.profile_enable(False)
    got = B.profile_read()
    total = lambda kind: sum(v["bytes"] for k, v in got.items() if k.split(".")[0] == kind)  # noqa: E731
    n_u = [int(((l < 0) & (u > 0)).sum()) for l, u in prob.lu]
    nnz = {i: len({(k, j) for k, i2, j in zip(prob.cuts.cut, prob.cuts.node, prob.cuts.neuron) if i2 == i}) for i in rel + [-1]}
    assert min(n_u) == 0 < max(n_u)      # a node without an a_hat
    want = dict(bound=0.0, bound_elem=0.0, conc=0.0, adj=0.0)
    d0 = DIMS[0]
    for q, i in enumerate(rel):
        d, last = DIMS[q + 1], q + 1 == len(rel)
        up = prob.S * d * 4 if last else None
        for e, times, ascent in ((esz, iters, True), (4, 1, False)):
            relax = M * d * e + (M * n_u[q] * e if ascent else 0) + M * n_u[q] * 4 + prob.B * n_u[q] + M * nnz[i] * 4
            slots = 0 if ascent else M * 8 * (-(-d // 256) if last else -(-d // 32))
            if last:
                want["bound_elem"] += times * (up + relax + slots)
            else:
                want["bound"] += times * ((M + d) * DIMS[q + 2] * e + relax + slots)
        src = d0 if q == 0 else DIMS[q]
        want["adj"] += iters * (M * src * (1 if q == 0 else esz) + d * src * esz + M * n_u[q] * esz + 24 * M * n_u[q] +
                                prob.B * n_u[q] + 8 * M * nnz[i] + M * d * esz)
    for e, times, ascent in ((esz, iters, True), (4, 1, False)):
        want["conc"] += times * ((M + d0) * DIMS[1] * e + (M * d0 if ascent else 0) + M * nnz[-1] * 4 * (2 if ascent else 1) +
                                 (0 if ascent else M * 8 * -(-d0 // 32)))
    for kind, bytes_ in want.items():
        assert total(kind) == bytes_, (kind, total(kind), bytes_, sorted(got))
