"""Attention that touches the weights of the launches behind it: a stage of three layers (each with a next one to touch, but for the last) gives
the bits of three stages of one layer (whose range ends with the layer), with and without room for the wave that does it."""
import numpy as np
import pytest

from paper_2110_14895_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,Hh,M,B", [
    (197, 128, 2, 512, 4),       # 8 pairs: one query wave, two loaders, the one that touches
    (15, 64, 1, 128, 1),         # a workgroup with more lanes than there are lines
    (257, 320, 4, 640, 65),      # nine query waves: twelve in all
    (320, 128, 2, 256, 140),     # ten: no room
    (50, 768, 12, 3072, 7),      # 350 rows to 14.2 MB: not touched
    (50, 768, 12, 3072, 8),      # 400: touched
    (101, 832, 13, 1024, 2),     # past 768 wide: 202 rows to 8.9 MB, not touched
    (101, 832, 13, 1024, 10),    # and by how the second MLP layer runs
])
def test_the_same_bits(T, D, Hh, M, B):
    sh = synth.custom_shape(f"touch_{D}", 3, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.05) for l in range(3)]
    x = synth.activations(sh, B, bf16=True)
    whole = H.run_stage(H.make_stage(sh, layers, 0, 3, B, bf16=True, in_bf16=False), x)
    for l in range(3):
        x = H.run_stage(H.make_stage(sh, layers[l:l + 1], l, l + 1, B, bf16=True, in_bf16=False), x)
    assert np.isfinite(whole).all() and np.array_equal(whole.view(np.uint32), x.view(np.uint32))
