"""Tile files across the renumbering of the dense tiles: choices of the old table that its numbers no longer name are
made again and appended behind the new table's mark; with the mark, and for other numbers, a choice stands."""
import contextlib
import os

import numpy as np
import pytest

from oracle import gcp_oracle as O
from test_gpu_layer_tiles import DIMS, _problem
from workloads import gen

pytestmark = pytest.mark.gpu

MARK = "gemm.k0.b0.s0.M0.N0.K0 2"


@contextlib.contextmanager
def _file(path):
    saved = {k: os.environ.get(k) for k in ("GCP_TILE_CACHE", "GCP_AUTOTUNE")}
    os.environ["GCP_TILE_CACHE"] = str(path)
    os.environ.pop("GCP_AUTOTUNE", None)
    try:
        yield
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


def _run(path, prob):
    import torch
    from paper_2208_05740_amd import binding as B
    with _file(path):
        P = B.Problem(prob, device=torch.device("cuda:0"))
        t = lambda x: torch.tensor(np.asarray(x, np.float32).reshape(P.M, -1), device="cuda:0")  # noqa: E731
        B.bound(P.net, P.x0, P.eps, P.C, P.splits, P.cuts, t(O.full_alpha(prob)), t(prob.beta), t(prob.gamma), grads=True)
        torch.cuda.synchronize()
    return path.read_text().splitlines()


@pytest.mark.parametrize("marked", [False, True])
def test_choices_of_the_old_table(marked, tmp_path):
    B, S = 43, 3
    prob = _problem(lambda r: gen.mlp_net(r, DIMS, w_var_num=1.0), 5, B, S, shift=1)
    key = f"gemm.k1.b0.s0.M{B * S}.N{DIMS[2]}.K{DIMS[3]}"
    keep = f"gemm.k1.b0.s0.M{B * S}.N{DIMS[3]}.K{DIMS[4]}"
    lines = ([MARK] if marked else []) + [f"{key} 2", f"{keep} 5"]
    path = tmp_path / "tiles.txt"
    path.write_text("".join(x + "\n" for x in lines))
    after = _run(path, prob)
    assert after[:len(lines)] == lines
    new = after[len(lines):]
    assert len(new) > 1 and new.count(MARK) == (0 if marked else 1) and (marked or new[0] == MARK), new
    chosen = [x.split()[0] for x in new]
    assert chosen.count(key) == (0 if marked else 1) and keep not in chosen, new
    # read again (another file in between), every choice is there
    other = tmp_path / "other.txt"
    other.write_text("")
    assert _run(other, prob)[0] == MARK
    assert _run(path, prob) == after
