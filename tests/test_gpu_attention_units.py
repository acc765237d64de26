"""GPU parity of attention at the edges of how it deals the queries of an (image, head) pair: groups of 16- or
32-query tiles over several workgroups while pairs are few, one group to a pair (two from 321 tokens on) otherwise,
the workgroups balanced over the rounds of units.  One layer whose MLP branch is switched off, against the checker
on the first, the last and a middle image; the tolerance is the bf16 path's."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu


# tokens, width, heads, images; "tiles x groups" on 256 compute units
@pytest.mark.parametrize("T,D,Hh,B", [
    (197, 128, 2, 1),      # 2 pairs: 16 x 13, one tile to a workgroup
    (15, 128, 2, 3),       # a single, partly filled tile
    (197, 128, 2, 40),     # 80 pairs: 16 x 3, a last group of three tiles next to groups of five
    (197, 128, 2, 64),     # 128 pairs: 16 x 2, seven and six tiles
    (257, 320, 4, 4),      # 16 pairs of d_head 80: 16 x 9, the last group a single tile next to groups of two
    (577, 128, 2, 6),      # 12 pairs: 16 x 19, a last group of one tile next to groups of two
    (257, 320, 4, 24),     # 96 pairs of d_head 80: 16 x 2, nine and eight tiles
    (577, 128, 2, 30),     # 60 pairs: 32 x 4, a last group of four tiles next to groups of five
    (577, 128, 2, 70),     # 140 pairs: two groups each as they do not fit one, two rounds on 140 workgroups
    (50, 128, 2, 136),     # 272 pairs: two rounds on 136 workgroups
    (257, 320, 4, 65),     # 260 pairs of d_head 80: two rounds on 130 workgroups, not a multiple of 8
])
def test_query_groups(T, D, Hh, B):
    sh = synth.custom_shape(f"attn_{T}_{D}", 1, D, Hh, 128, T)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)
    for n in ("w_fc2", "b_fc2"):
        p[n] = np.zeros_like(p[n])
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=True), x)
    pick = sorted({0, B // 2, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
