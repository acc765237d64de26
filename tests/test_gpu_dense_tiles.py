"""GPU parity of the dense layers at the edges of their tile shapes: one layer whose four dense layers fall, on 256
compute units, on the shapes named beside it (asked of the dispatcher, so that a change of its costs cannot move a case
to other kernels unnoticed), rows and columns rarely whole numbers of tiles.  Between them the cases run every shape with every
epilogue it is chosen for.  Against the checker on the first, a middle and the last image (the last one sits in the
partly filled tile row); the tolerance is the bf16 path's.  128x128 and 128x128x2 are one kernel at two prices.  Up to 256 wide, and from 500 rows on
at 320, 384 and 512, the first MLP layer, with its LayerNorm, is a kernel of its own (test_gpu_bf16_rows.py, test_gpu_wide_rows.py) and the
third shape is not run; the cases at 448 and 576 hold the shapes with GELU."""
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H
from tests.test_dispatch import EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESID, EPI_PARTIAL, dense_plan

pytestmark = pytest.mark.gpu


def shapes_of(rows, d, m):
    out = []
    for n, k, epi in ((3 * d, d, EPI_BIAS), (d, d, EPI_BIAS_RESID), (m, d, EPI_BIAS_GELU), (d, m, EPI_PARTIAL)):
        p = dense_plan(rows, n, k, epi)
        out.append(str(p) + (f"+{rows - p.m_main}" if rows > p.m_main else ""))
    return " ".join(out)


# tokens, width, heads, MLP width, images; tiles of q|k|v, projection, first and second MLP layer (x2: two to a unit,
# P: persistent kernel, its rows past the tile walk behind the +, K ranges behind the /)
@pytest.mark.parametrize("T,D,Hh,M,B,shapes", [
    (197, 128, 2, 512, 4, "64x64x2 64x64x2 64x64x2 64x64x2"),
    (65, 256, 4, 1024, 30, "64x128x2 64x64x2 64x128x2 64x64x2"),
    (197, 256, 4, 1280, 24, "128x128 64x128x2 192x128 64x128x2"),
    (197, 384, 6, 1536, 26, "192x128 64x128x2 128x128x2 64x128x2"),
    (197, 256, 4, 768, 64, "256x192 128x128x2 256x192 128x128"),
    (197, 512, 8, 2048, 32, "256x192 128x128 256x256 128x128"),
    (197, 576, 9, 2304, 32, "256x192 128x128 256x256 128x128"),
    (257, 320, 4, 1280, 64, "P256x320 128x128x2 P256x320+64 256x128"),
    (197, 448, 7, 1792, 48, "P256x256 192x128 P256x320 192x128"),
    (65, 320, 5, 1536, 1, "64x64x2 64x64x2 64x64x2 64x64x2/2"),
    (257, 128, 2, 256, 68, "128x128x2 128x128x2 192x128 128x128"),
    (197, 896, 14, 2688, 6, "128x128 64x128x2 128x128 128x128/2"),
    (577, 192, 3, 576, 71, "P256x256 192x256 256x192 256x192"),
    (577, 384, 6, 896, 57, "P256x320+121 P256x256+121 P256x256+121 256x128"),
    (197, 832, 13, 128, 73, "P256x320 P256x256 64x128x2 256x256"),
    (257, 192, 3, 384, 67, "256x192 64x64x2 128x128x2 192x128"),
    (50, 896, 14, 3840, 31, "192x128 64x128x2 256x128 192x128/4"),
    (577, 576, 9, 512, 49, "P256x256+369 P256x320 256x256 P256x320"),
    (65, 768, 12, 3200, 10, "64x128x2 64x64x2 128x128 64x128x2/2"),
    (257, 256, 4, 640, 62, "192x256 128x128x2 192x256 128x128"),
    (257, 640, 10, 320, 129, "P256x320+385 P256x320+385 P256x320 P256x320+385"),
    (50, 448, 7, 192, 90, "256x128 64x64x2 64x64x2 64x64x2"),
    (577, 128, 2, 448, 86, "128x128x2 128x128x2 P256x256 256x128"),
    (577, 256, 4, 576, 57, "P256x256 192x256 P256x320+121 192x256"),
    (257, 448, 7, 2048, 8, "128x128 64x64x2 192x128 64x64x2"),
    (257, 448, 7, 2048, 12, "192x128 64x128x2 256x128 64x128x2"),
    (197, 448, 7, 2048, 21, "192x128 64x64x2 256x192 64x64x2"),
    (257, 448, 7, 1792, 25, "256x192 128x128 192x256 128x128"),
    (257, 448, 7, 2048, 24, "256x192 128x128 256x256 128x128"),
    (197, 448, 7, 2048, 63, "P256x320 256x128 P256x256 256x128"),
    (65, 448, 7, 2048, 127, "256x192 192x128 P256x256+63 192x128"),
    (257, 448, 7, 2048, 36, "P256x256 192x128 P256x320+36 192x128"),
])
def test_tile_shapes(T, D, Hh, M, B, shapes):
    assert shapes_of(T * B, D, M) == shapes
    sh = synth.custom_shape(f"tiles_{T}_{D}", 1, D, Hh, M, T)
    # N(0, 0.05) weights in the narrow cases; with them the rounding of the operands to bf16 alone (the checker's rounded
    # mode against its exact one) is 1.9e-2 to 2.2e-2 at widths of 832 and 896, 1.1e-2 at 512, so wide ones take N(0, 0.02)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05 if D <= 512 else 0.02)
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=True), x)
    pick = sorted({0, B // 2, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
