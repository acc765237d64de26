"""GPU parity of the dense layers at the edges of their tile shapes: one layer whose four dense layers fall, on 256
compute units, on the shapes named beside it, rows and columns never whole numbers of tiles.  Against the checker on
the first, a middle and the last image (the last one sits in the partly filled tile row); the tolerance is the bf16
path's."""
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu


# tokens, width, heads, MLP width, images; tiles of q|k|v, projection, first and second MLP layer
# (P: persistent kernel, its rows past the tile walk behind the +)
@pytest.mark.parametrize("T,D,Hh,M,B", [
    (197, 128, 2, 512, 4),       # 64x64 throughout, two K steps
    (65, 256, 4, 1024, 30),      # 64x128, 64x64, 64x128, 64x64
    (197, 256, 4, 1280, 24),     # 128x128, 64x128, 192x128, 64x128
    (197, 384, 6, 1536, 26),     # 192x128, 64x128, two 128x128 to a unit, 64x128
    (197, 256, 4, 768, 64),      # 192x256, 128x128, 192x256, 128x128
    (197, 512, 8, 2048, 32),     # 256x192, 128x128, 256x256, 128x128
    (257, 320, 4, 1280, 64),     # P256 + 64, two 128x128, two 128x128, 256x128
    (197, 448, 7, 1792, 48),     # 256x256, 192x128, P256 + 240, 192x128; N = 448 and 1344 leave half and quarter tiles
])
def test_tile_shapes(T, D, Hh, M, B):
    sh = synth.custom_shape(f"tiles_{T}_{D}", 1, D, Hh, M, T)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=True), x)
    pick = sorted({0, B // 2, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
