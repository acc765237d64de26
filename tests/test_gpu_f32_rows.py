"""GPU parity of the fp32 path where many rows meet a dense layer with LayerNorm inside (64 rows to a workgroup, steps of
32 columns), where a dense layer takes tiles of 16 x 32, and of attention on few key blocks: one block, an odd
number of blocks, waves without keys.  fp32 tolerance."""
import pytest

from tests.test_dispatch import f32_ln_route
from tests.test_gpu_f32_kernels import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,Hh,M,B", [
    (197, 192, 3, 768, 8),     # 64 x 32 steps, a last panel of 40 rows; 16 x 32 tiles behind them
    (197, 192, 3, 772, 8),     # a last step of four columns
    (65, 100, 2, 396, 60),     # K = 100 of 192, columns not a multiple of 32, d_head 50 on the vector ALU
    (65, 100, 5, 390, 60),     # columns not a multiple of 4
    (31, 48, 4, 1100, 160),    # K = 48, more than 32 steps of columns
    (197, 384, 6, 1536, 2),    # K > 192 from the first tile more than there are compute units
    (128, 196, 1, 1024, 8),    # K = 196 of 384, whole panels
    (197, 384, 6, 384, 33),    # K > 192 beyond the line: LayerNorm on its own before the wider layer
    (65, 16, 1, 1028, 130),    # depths of 64, of K = 16 and of 64; a last step of four columns
    (65, 64, 1, 1024, 130),
    (65, 68, 1, 1028, 65),     # of 128
    (197, 128, 2, 512, 11),
    (65, 196, 7, 780, 21),     # of 256, d_head 28
    (64, 256, 4, 1024, 12),
    (65, 260, 5, 516, 20),     # of 320, d_head 52
    (33, 320, 5, 1280, 20),
    (16, 192, 3, 192, 3),      # one block of keys: three waves without any
    (33, 64, 1, 64, 2),        # three blocks, the last of one key
    (80, 192, 3, 64, 130),     # five blocks, queries to every wave, a wave with no queries
    (81, 256, 2, 64, 3),       # d_head 128, six blocks over four waves
])
def test_f32_rows(T, D, Hh, M, B):
    run(T, D, Hh, M, B)


def test_depths_of_the_rows_kernel():
    """The cases above that name a depth do keep their rows in registers, before one dense layer at least."""
    for t, d, m, b in ((65, 16, 1028, 130), (65, 64, 1024, 130), (65, 68, 1028, 65), (197, 128, 512, 11), (65, 196, 780, 21),
                       (64, 256, 1024, 12), (65, 260, 516, 20), (33, 320, 1280, 20)):
        assert 3 in (f32_ln_route(t * b, 3 * d, d), f32_ln_route(t * b, m, d)), d


def test_f32_rows_off_16_byte_alignment():
    run(197, 192, 3, 768, 8, offset=1)
