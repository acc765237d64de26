"""Attention that touches the weights of the launches behind it, nothing, some or all of them as the library says it will (which weights
these are is asked without a GPU, in test_dispatch.py): a stage of three layers, each with a next one to touch but for the last, gives the bits of
three stages of one layer, whose range ends with the layer.  Touching only reads, so the bits say that the launches in front and behind
are undisturbed, not that the weights came nearer."""
import numpy as np
import pytest

from paper_2110_14895_amd import synth
from tests import harness as H
from tests.test_dispatch import TOUCH_ALL, TOUCH_LONG, TOUCH_NONE, touch_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,Hh,M,B,kind", [
    (197, 128, 2, 512, 4, TOUCH_ALL),        # 8 pairs: one query wave, two loaders, the one that touches
    (15, 64, 1, 128, 1, TOUCH_ALL),          # one workgroup, which goes through all lines
    (15, 64, 1, 128, 256, TOUCH_ALL),        # more lanes in the launch than lines: most workgroups touch none
    (257, 320, 4, 640, 65, TOUCH_ALL),       # nine query waves: twelve in all
    (320, 128, 2, 256, 140, TOUCH_NONE),     # ten: no room
    (50, 768, 12, 3072, 7, TOUCH_NONE),      # 350 rows to 14.2 MB
    (50, 768, 12, 3072, 8, TOUCH_ALL),       # 400
    (101, 832, 13, 1024, 2, TOUCH_NONE),     # past 768 wide: 202 rows to 8.9 MB
    (101, 832, 13, 1024, 10, TOUCH_ALL),     # 1010
    (50, 832, 13, 3328, 20, TOUCH_LONG),     # 1000 rows to 16.6 MB: projection and second MLP layer
    (197, 1024, 16, 1024, 3, TOUCH_LONG),    # 591 rows to 12.6 MB
])
def test_the_same_bits(T, D, Hh, M, B, kind):
    assert touch_plan(D, Hh, M, T, B).kind == kind
    sh = synth.custom_shape(f"touch_{D}", 3, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.05) for l in range(3)]
    x = synth.activations(sh, B, bf16=True)
    whole = H.run_stage(H.make_stage(sh, layers, 0, 3, B, bf16=True, in_bf16=False), x)
    for l in range(3):
        x = H.run_stage(H.make_stage(sh, layers[l:l + 1], l, l + 1, B, bf16=True, in_bf16=False), x)
    assert np.isfinite(whole).all() and np.array_equal(whole.view(np.uint32), x.view(np.uint32))
