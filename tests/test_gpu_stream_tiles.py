"""GPU parity of the dense layers whose tiles are at most 128 columns wide (loader waves, weights in fragment order) where
their pipelines are shorter than they are deep and where rows end inside a tile: K of one to nine steps of 64, one row to
one past a tile.  `shapes` is what the dispatcher runs on 256 compute units (tiles of q|k|v, projection, first and second
MLP layer as in test_gpu_dense_tiles.py, whose cases hold every shape at greater depths); up to 256 wide, and at the 2561 rows of
512, every first MLP layer here and q|k|v behind a first layer are one launch of another kernel with their LayerNorm.  Against the oracle on
the first and the last image; the tolerance is the bf16 path's."""
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H
from tests.test_gpu_dense_tiles import shapes_of

SMALL = "64x64x2 64x64x2 64x64x2 64x64x2"

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,Hh,M,B,shapes", [
    (1, 64, 1, 64, 1, SMALL),          # one row, one K step everywhere
    (17, 64, 1, 128, 1, SMALL),        # one and two steps
    (64, 128, 2, 192, 1, SMALL),       # two and three: whole tiles of 64 rows
    (65, 192, 3, 256, 1, SMALL),       # three and four, one row past
    (64, 256, 4, 320, 3, SMALL),       # four and five
    (127, 320, 4, 384, 1, SMALL),      # five and six, d_head 80
    (129, 448, 7, 512, 1, SMALL),      # seven and eight
    (193, 128, 2, 576, 7, SMALL),      # two and nine
    (197, 512, 8, 1024, 13, "128x128 64x128x2 128x128 64x128x2"),        # eight and sixteen
    (197, 448, 7, 1024, 13, "128x128 64x128x2 128x128 64x128x2"),        # seven and sixteen, with GELU too
    (193, 64, 1, 64, 100, "192x128 64x64x2 64x64x2 64x64x2"),            # 192 rows, one step, a remainder of 100
    (193, 128, 2, 64, 200, "128x128x2 192x128 64x64x2 192x128"),         # 192 rows with a residual, two steps and one
    (193, 64, 1, 1024, 1, "64x64x2 64x64x2 64x64x2 64x64x2/2"),          # two K ranges of eight steps
])
def test_short_k_and_ragged_rows(T, D, Hh, M, B, shapes):
    assert shapes_of(T * B, D, M) == shapes
    sh = synth.custom_shape(f"stream_{T}_{D}", 2, D, Hh, M, T)
    p = [synth.layer_params(sh, i, bf16=True, randomize_affine=True, w_std=0.05) for i in range(2)]
    x = synth.activations(sh, B, bf16=True)
    st = H.make_stage(sh, p, 0, 2, B, bf16=True)
    got = H.run_stage(st, x)
    pick = sorted({0, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), p, x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
