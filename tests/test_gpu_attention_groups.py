"""GPU parity of attention where a group has up to nine tiles of 16 queries (one for each of its waves) and where it
has more, the first size past it: the rows of keys and values placed for d_head 64 and for 80.  One layer whose MLP
branch is switched off, against the oracle on the first and the last image; the tolerance is the bf16 path's."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu


# tokens, width, heads, images; "tiles x groups" on 256 compute units
@pytest.mark.parametrize("T,D,Hh,B", [
    (257, 320, 4, 16),     # 64 pairs of d_head 80: 16 x 4, a last group of two tiles next to groups of five
    (288, 128, 2, 64),     # 128 pairs: 16 x 2, nine tiles each, no row past the last token
    (289, 128, 2, 64),     # 128 pairs: ten tiles of 16 to a group, so 32 x 2, a last tile of one query
    (129, 64, 1, 128),     # 128 pairs: 16 x 2, a last tile of one query
])
def test_groups_of_sixteen_and_of_thirty_two(T, D, Hh, B):
    sh = synth.custom_shape(f"groups_{T}_{D}", 1, D, Hh, 128, T)
    p = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.05)
    for n in ("w_fc2", "b_fc2"):
        p[n] = np.zeros_like(p[n])
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=True), x)
    pick = [0, B - 1]
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i
