"""GPU parity of LayerNorm and the first MLP layer in one launch on few rows of narrow models: panels of 32 rows, 16 columns to a wave, at the edges
of rows, columns and of where they are taken, bit for bit against the same images in a micro-batch that takes other panels, and against the oracle
(the tolerance is the bf16 path's)."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H
from tests.test_dispatch import EPI_BIAS_GELU, ln_plan

pytestmark = pytest.mark.gpu


def panel_rows(rows, n, k):
    return ln_plan(rows, n, k, EPI_BIAS_GELU)[0]


# tokens, width, heads, MLP, images that take panels of 32 rows, images that do not
@pytest.mark.parametrize("T,D,Hh,M,few,B", [
    (1, 64, 1, 256, 1, 2561),        # one row, two slices of K
    (33, 64, 1, 320, 1, 80),         # a panel and a row; columns that are not whole sets of a workgroup
    (65, 128, 2, 512, 3, 40),        # 195 rows, three in the last panel
    (160, 192, 3, 768, 16, 17),      # the most rows that take them
    (31, 256, 4, 4096, 29, 30),      # up to 3.8 million outputs
    (257, 320, 4, 1280, 1, 11),      # ten slices
    (197, 384, 6, 1536, 4, 13),      # a set and a half of columns to a wave
])
def test_the_same_bits_in_other_panels(T, D, Hh, M, few, B):
    assert panel_rows(T * few, M, D) == 32 < panel_rows(T * B, M, D)
    sh = synth.custom_shape(f"few_{T}_{D}", 1, D, Hh, M, T)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)
    # out of the first MLP layer as it is: the second one passes hidden units on, one to a column, so that its sum is exact
    p["w_fc2"] = np.zeros_like(p["w_fc2"])
    pick = np.linspace(0, M - 1, D).astype(int)
    p["w_fc2"][np.arange(D), pick] = 1.0
    x = synth.activations(sh, B, bf16=True)
    many = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=True), x)
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, few, bf16=True), x[:few])
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[:1])
    assert H.rel_err(got[0], ref[0]) <= H.TOL_BF16
    np.testing.assert_array_equal(got, many[:few])


@pytest.mark.parametrize("T,D,Hh,M,B", [(197, 384, 6, 1536, 12), (65, 192, 3, 768, 2)])
def test_against_the_oracle(T, D, Hh, M, B):
    assert panel_rows(T * B, M, D) == 32
    sh = synth.custom_shape(f"fewrows_{T}_{D}", 2, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.05) for l in range(2)]
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, layers, 0, 2, B, bf16=True), x)
    pick = [0, B - 1]
    ref = oracle.stage_forward(H.oracle_cfg(sh), layers, x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
