"""GPU parity of LayerNorm and the dense layer behind it in one launch (narrow bf16 models: 128 rows to a workgroup, 32
columns of a wave at a time), at the edges of rows, columns and depth, against the oracle on the first and the last image.
The tolerance is the bf16 path's."""
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,Hh,M,B,in_bf16", [
    (197, 192, 3, 768, 40, False),     # 7880 rows, a last panel of 72
    (128, 384, 6, 1536, 48, False),    # whole panels
    (197, 384, 6, 1536, 32, True),     # bf16 in: the first LayerNorm on its own, the second one inside
    (129, 64, 1, 64, 200, False),      # two slices, fewer sets of columns than waves
    (65, 128, 2, 1088, 160, False),    # a last group of columns that is not full
    (577, 256, 4, 1024, 20, False),
    (257, 320, 4, 1280, 30, False),    # rows that are not whole 256 bytes
])
def test_layernorm_inside_a_dense_layer(T, D, Hh, M, B, in_bf16):
    sh = synth.custom_shape(f"rows_{T}_{D}", 2, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.05) for l in range(2)]
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, layers, 0, 2, B, bf16=True, in_bf16=in_bf16), x)
    pick = [0, B - 1]
    ref = oracle.stage_forward(H.oracle_cfg(sh), layers, x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
