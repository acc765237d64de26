"""GPU parity of LayerNorm and the dense layer behind it in one launch at widths of 512 to 1024, and of narrow models on
few rows: every height of a panel, with a last panel that is rarely whole and column groups of less than a set of columns up to
all of them.  Bit for bit against the two launches, with the height asked of the library, and against the oracle (the tolerance is the
bf16 path's)."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import binding, synth
from tests import harness as H
from tests.test_dispatch import EPI_BIAS, EPI_BIAS_GELU, TOUCH_ALL, dense_plan, ln_plan, touch_plan

pytestmark = pytest.mark.gpu


def panel_rows(rows, n, k, epi):
    return ln_plan(rows, n, k, epi)[0]


# q|k|v: a stage that takes bf16 normalises its input where it widens it, the same values in fp32 go through the one launch
@pytest.mark.parametrize("T,D,Hh,B,height", [
    (17, 64, 1, 1, 64), (197, 192, 3, 1, 64), (65, 320, 4, 8, 64), (197, 384, 6, 3, 64), (197, 384, 6, 5, 64),
    (197, 512, 8, 3, 64), (577, 512, 8, 5, 64), (192, 512, 8, 29, 96), (197, 512, 8, 97, 96),
    (200, 768, 12, 13, 64), (197, 768, 12, 24, 64), (577, 768, 12, 16, 80), (197, 768, 12, 100, 80),
    (220, 1024, 16, 25, 64), (197, 1024, 16, 41, 64),
])
def test_bits_of_two_launches(T, D, Hh, B, height):
    assert panel_rows(T * B, 3 * D, D, EPI_BIAS) == height
    assert dense_plan(T * B, 3 * D, D, EPI_BIAS).m_main == T * B        # no rows that add up in another order
    sh = synth.custom_shape(f"widebits_{T}_{D}", 1, D, Hh, 64, T)
    p = [synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)]
    x = synth.activations(sh, B, bf16=True)
    two = H.run_stage(H.make_stage(sh, p, 0, 1, B, bf16=True, in_bf16=True), x)
    one = H.run_stage(H.make_stage(sh, p, 0, 1, B, bf16=True, in_bf16=False), x)
    np.testing.assert_array_equal(one, two)


# the first MLP layer, with GELU: few rows take two launches and more rows one; 576 columns leave a last set that is not full
@pytest.mark.parametrize("T,D,Hh,M,few,B", [(197, 768, 12, 512, 4, 16), (197, 768, 12, 576, 4, 52), (197, 512, 8, 512, 2, 12), (197, 512, 8, 576, 2, 98),
                                              (197, 1024, 16, 576, 6, 30)])
def test_bits_of_two_launches_with_gelu(T, D, Hh, M, few, B):
    assert panel_rows(T * few, M, D, EPI_BIAS_GELU) == 0 < panel_rows(T * B, M, D, EPI_BIAS_GELU)
    assert dense_plan(T * few, M, D, EPI_BIAS_GELU).m_main == T * few
    sh = synth.custom_shape(f"widegelu_{T}_{D}", 1, D, Hh, M, T)        # a second MLP layer this shallow is never cut
    p = [synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)]
    x = synth.activations(sh, B, bf16=True)
    st = H.make_stage(sh, p, 0, 1, B, bf16=True)
    one = H.run_stage(st, x)
    for i in range(0, B, few):
        np.testing.assert_array_equal(H.run_stage(st, x[i:i + few]), one[i:i + few])


# at 1024 wide below 5500 rows only where attention touches the weights; at 768 from 1900 rows on
@pytest.mark.parametrize("T,D,Hh,M,few,B", [(197, 1024, 16, 4096, 4, 16), (577, 1024, 16, 4352, 1, 5), (50, 1024, 16, 3136, 16, 77), (197, 768, 12, 3072, 4, 10),
                                              (577, 768, 12, 4608, 2, 4)])
def test_bits_of_two_launches_behind_touching(T, D, Hh, M, few, B):
    touched = binding.lib().ep_query_ln_gemm_touched_mlp
    touched.argtypes, touched.restype = [C.c_int64, C.c_int32, C.c_int32], C.c_int32
    assert touch_plan(D, Hh, M, T, B).kind == TOUCH_ALL and touched(T * B, M, D) and not touched(T * few, M, D)
    assert dense_plan(T * few, M, D, EPI_BIAS_GELU).m_main == T * few
    sh = synth.custom_shape(f"touched_{T}_{D}", 1, D, Hh, M, T)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)
    # the second MLP layer passes hidden units on, one to a column: its sums are exact however K is cut
    p["w_fc2"] = np.zeros_like(p["w_fc2"])
    p["w_fc2"][np.arange(D), np.linspace(0, M - 1, D).astype(int)] = 1.0
    x = synth.activations(sh, B, bf16=True)
    st = H.make_stage(sh, [p], 0, 1, B, bf16=True)
    one = H.run_stage(st, x)
    for i in range(0, B - few + 1, few):
        np.testing.assert_array_equal(H.run_stage(st, x[i:i + few]), one[i:i + few])


@pytest.mark.parametrize("T,D,Hh,M,B", [(197, 512, 8, 2048, 20), (197, 768, 12, 3072, 16), (197, 1024, 16, 4096, 32)])
def test_against_the_oracle(T, D, Hh, M, B):
    sh = synth.custom_shape(f"wide_{T}_{D}", 2, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.02) for l in range(2)]
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, layers, 0, 2, B, bf16=True), x)
    pick = [0, B - 1]
    ref = oracle.stage_forward(H.oracle_cfg(sh), layers, x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
