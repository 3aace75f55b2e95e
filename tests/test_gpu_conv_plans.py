"""Convolutions at the edge of what fits a workgroup's LDS, as bounds and
gradients through the C ABI, against the FP64 oracle.  Tolerances are those of
the other parity tests: FP32 bounds within 1e-5 of max(|g|, T) (T the sum of
the magnitudes of the terms added), gradients within 1e-4 of the row's largest,
bf16 bounds within 2e-2 of T.
"""
import pytest

from test_gpu_layer_tiles import _bound, _check_oracle, _conv_net, _problem

pytestmark = pytest.mark.gpu

# channels and side of the stacked 3x3 convs (stride 1, pad 1) on a small input
SHAPES = [
    (1, (2, 32, 32), (64, 64)),     # bf16: one row's slab fits 64 KB at two bytes an element only
    (1, (3, 16, 16), (128, 128)),
]


@pytest.mark.parametrize("mode,shape,channels", SHAPES)
def test_conv_at_the_lds_limit_matches_oracle(mode, shape, channels, tmp_path):
    print(f"convs {shape} -> {channels}, mode={mode}", flush=True)
    convs = tuple((c, 3, 1, 1) for c in channels)
    prob = _problem(lambda r: _conv_net(r, shape, convs, (3,)), 3, 2, 3, eps=0.01)
    got, params, _ = _bound(prob, mode, tmp_path / "c.txt")
    _check_oracle(prob, got, params, mode)
