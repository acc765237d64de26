"""GPU parity of dense layers on tiles of the heights between 64, 128, 192 and 256 rows, and of K ranges that follow each other in one
workgroup: every height with every epilogue that takes it,
the last tile row rarely whole.  The height is asked of the library.  Rows add up in the same order whatever the height, so
an image gives the same bits in a micro-batch that runs on other heights; sums over K ranges are held against the oracle (the tolerance
is the bf16 path's)."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import binding, synth
from tests import harness as H
from tests.test_dispatch import EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESID, EPI_PARTIAL, dense_plan, group_limit

pytestmark = pytest.mark.gpu


# heights of q|k|v, projection and first MLP layer at B images (0: one of the table, or another kernel)
@pytest.mark.parametrize("T,D,M,B,few,heights", [
    (257, 1024, 1024, 8, 2, (208, 80, 80)),
    (197, 1024, 1024, 14, 2, (144, 96, 96)),
    (50, 1024, 768, 13, 2, (80, 0, 0)),
    (50, 1280, 768, 13, 2, (96, 0, 0)),
    (50, 1024, 768, 29, 2, (160, 0, 0)),
    (257, 1280, 768, 5, 2, (176, 0, 0)),
    (239, 1280, 768, 7, 2, (224, 80, 0)),
    (50, 1024, 768, 42, 2, (240, 80, 0)),
    (50, 1280, 768, 65, 2, (0, 144, 80)),
    (50, 768, 768, 121, 2, (0, 160, 0)),
    (65, 1280, 768, 62, 2, (0, 176, 96)),
    (65, 1280, 768, 74, 2, (0, 208, 0)),
    (257, 768, 768, 34, 2, (0, 224, 0)),
    (197, 384, 768, 32, 2, (0, 80, 0)),
    (197, 384, 768, 64, 2, (0, 80, 0)),
    (50, 1280, 768, 113, 2, (0, 240, 0)),
])
def test_bits_of_another_height(T, D, M, B, few, heights):
    layers = ((3 * D, D, EPI_BIAS), (D, D, EPI_BIAS_RESID), (M, D, EPI_BIAS_GELU), (D, M, EPI_PARTIAL))
    plans = [dense_plan(T * B, *l) for l in layers]
    assert [(p.bm, p.bn) for p in plans[:3]] == [(h, 128) if h else (plans[i].bm, plans[i].bn) for i, h in enumerate(heights)]
    for l, p in zip(layers, plans):
        other = dense_plan(T * few, *l)
        assert p.splits == other.splits == 1 and p.m_main == T * B and other.m_main == T * few
    sh = synth.custom_shape(f"heights_{T}_{D}", 1, D, D // 64, M, T)
    p = [synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.03)]
    x = synth.activations(sh, B, bf16=True)
    st = H.make_stage(sh, p, 0, 1, B, bf16=True)
    got = H.run_stage(st, x)
    for i in (0, B // 2, B - few):
        np.testing.assert_array_equal(H.run_stage(st, x[i:i + few]), got[i:i + few])


@pytest.mark.parametrize("T,D,M,B,height", [
    (50, 768, 3072, 13, 80),
    (50, 768, 3072, 27, 144),
    (50, 768, 3072, 29, 160),
    (50, 768, 3072, 34, 96),
    (50, 1024, 4096, 26, 176),
    (50, 1280, 5120, 47, 208),
    (50, 1280, 5120, 50, 240),
    (50, 1280, 5120, 53, 224),
])
def test_sums_over_k_ranges(T, D, M, B, height):
    p = dense_plan(T * B, D, M, EPI_PARTIAL)
    assert p.splits > 1 and (p.bm, p.bn) == (height, 128)
    sh = synth.custom_shape(f"ranges_{T}_{D}", 1, D, D // 64, M, T)
    w = synth.layer_params(sh, 0, bf16=True, randomize_affine=True, w_std=0.02)
    x = synth.activations(sh, B, bf16=True)
    got = H.run_stage(H.make_stage(sh, [w], 0, 1, B, bf16=True), x)
    pick = sorted({0, B // 2, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), [w], x[pick])
    for k, i in enumerate(pick):
        assert H.rel_err(got[i], ref[k]) <= H.TOL_BF16, i


# K ranges of a micro-batch one after the other in one launch over a group of them: the bits of the sums that go through memory
@pytest.mark.parametrize("T,D,M,mb,n,splits,height,out_bf16", [
    (197, 1024, 4096, 2, 10, 2, 128, False),
    (197, 1024, 4096, 2, 11, 2, 160, True),
    (65, 1024, 4096, 4, 11, 4, 128, True),
    (65, 1024, 4096, 4, 16, 4, 160, False),
    (65, 1024, 4096, 1, 35, 8, 128, False),
    (257, 1280, 5120, 4, 6, 4, 128, False),     # 80 K steps: two past the unrolled three
    (257, 1280, 5120, 4, 6, 4, 128, True),
    (197, 768, 3072, 8, 8, 2, 160, False),      # 48: none
])
def test_ranges_of_a_group_in_one_launch(T, D, M, mb, n, splits, height, out_bf16):
    import torch
    f = binding.lib().ep_query_ranges_height
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32, C.c_int32], C.c_int32
    assert dense_plan(T * mb, D, M, EPI_PARTIAL).splits == splits
    assert f(T * mb * n, D, M, splits) == height and f(T * mb, D, M, splits) == 0 and n <= group_limit(D, D // 64, M, T, mb)
    sh = synth.custom_shape(f"group_ranges_{T}_{D}", 2, D, D // 64, M, T)
    p = [synth.layer_params(sh, l, bf16=True, randomize_affine=True, w_std=0.02) for l in range(2)]
    st = H.make_stage(sh, p, 0, 2, mb, bf16=True, out_bf16=out_bf16)
    pipe = binding.Pipeline([st], mb)
    x = H.to_device(synth.activations(sh, mb * n, bf16=True), True)
    out = [torch.empty(x.shape, dtype=torch.bfloat16 if out_bf16 else torch.float32, device="cuda") for _ in range(2)]
    s = torch.cuda.current_stream()
    pipe.run(x, n, out[0], s)
    for i in range(n):
        st.forward(x[i * mb:(i + 1) * mb], mb, out[1][i * mb:(i + 1) * mb], s)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    pipe.destroy()
