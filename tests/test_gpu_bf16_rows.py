"""GPU parity of LayerNorm and the dense layer behind it in one launch (narrow bf16 models: 64 or 128 rows to a workgroup, 32
columns of a wave at a time), at the edges of rows, columns and depth, against the oracle on the first and the last image
(the tolerance is the bf16 path's), and bit for bit against the two launches."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H
from tests.test_dispatch import EPI_BIAS, EPI_BIAS_GELU, dense_plan, ln_plan

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


# A stage that takes bf16 normalises its input in the launch that widens it and runs q|k|v behind that; the same values in fp32
# go through the one launch.  Panels of 64 and of 128 rows, the last one rarely whole, every depth.
@pytest.mark.parametrize("T,D,Hh,B", [
    (65, 64, 1, 1), (65, 64, 1, 150), (129, 128, 2, 20), (65, 128, 2, 600), (197, 192, 3, 2), (577, 192, 3, 71), (197, 256, 4, 7),
    (197, 256, 4, 70), (257, 320, 4, 6), (257, 320, 4, 60), (197, 384, 6, 24), (197, 384, 6, 64),
])
def test_bits_of_two_launches(T, D, Hh, B):
    assert dense_plan(T * B, 3 * D, D, EPI_BIAS).m_main == T * B        # no rows that add up in another order
    sh = synth.custom_shape(f"rowbits_{T}_{D}", 1, D, Hh, 64, T)
    p = [synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)]
    x = synth.activations(sh, B, bf16=True)
    two = H.run_stage(H.make_stage(sh, p, 0, 1, B, bf16=True, in_bf16=True), x)
    one = H.run_stage(H.make_stage(sh, p, 0, 1, B, bf16=True, in_bf16=False), x)
    np.testing.assert_array_equal(one, two)


# The first MLP layer, with GELU: past 256 wide few rows take two launches and more rows one (asked of the library)
@pytest.mark.parametrize("T,D,Hh", [(197, 320, 4), (197, 384, 6)])
def test_bits_of_two_launches_with_gelu(T, D, Hh):
    B, few = 40, 2
    assert ln_plan(T * few, 512, D, EPI_BIAS_GELU)[0] == 0 < ln_plan(T * B, 512, D, EPI_BIAS_GELU)[0]
    assert dense_plan(T * few, 512, D, EPI_BIAS_GELU).m_main == T * few
    sh = synth.custom_shape(f"rowgelu_{T}_{D}", 1, D, Hh, 512, T)       # 512 deep: the second MLP layer is never cut
    p = [synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)]
    x = synth.activations(sh, B, bf16=True)
    st = H.make_stage(sh, p, 0, 1, B, bf16=True)
    one = H.run_stage(st, x)
    for i in range(0, B, few):
        np.testing.assert_array_equal(H.run_stage(st, x[i:i + few]), one[i:i + few])
