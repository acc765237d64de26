"""GPU parity of the fp32 path at the edges of its kernels: the matrix-core dense layers (16- and 32-wide tiles with
and without LayerNorm inside, 64 x 32 tiles), attention with the keys split over waves and not, head widths up to 128,
and the vector-ALU kernels where rows are not whole 16-byte pieces.  fp32 tolerance throughout."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import binding, synth
from tests import harness as H

pytestmark = pytest.mark.gpu


def run(T, D, Hh, M, B, offset=0):
    import torch
    sh = synth.custom_shape(f"f32k_{T}_{D}", 2, D, Hh, M, T)
    layers = [synth.layer_params(sh, l, randomize_affine=True, w_std=0.1) for l in range(2)]
    x = synth.activations(sh, B)
    st = H.make_stage(sh, layers, 0, 2, B, bf16=False)
    n = x.size
    xin = torch.empty(n + 4, dtype=torch.float32, device="cuda")[offset:offset + n]
    xin.copy_(torch.from_numpy(x).reshape(-1))
    out = torch.full((n + 8,), float("nan"), dtype=torch.float32, device="cuda")
    st.forward(xin, B, out[offset:offset + n], torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isnan(got[:offset]).all() and np.isnan(got[offset + n:]).all()        # nothing beside the output
    got = got[offset:offset + n].reshape(x.shape)
    pick = sorted({0, B // 2, B - 1})
    ref = oracle.stage_forward(H.oracle_cfg(sh), layers, x[pick])
    assert H.rel_err(got[pick], ref) <= H.TOL_F32


@pytest.mark.parametrize("T,D,Hh,M,B", [
    (65, 320, 4, 900, 1),      # 16-wide tiles, LayerNorm inside with K > 192, d_head 80
    (50, 192, 2, 768, 9),      # 32-wide tiles, LayerNorm inside, d_head 96
    (50, 320, 5, 640, 9),      # ... with K > 192
    (33, 132, 3, 520, 180),    # 64 x 32 tiles with ragged K; attention with queries to every wave, d_head 44
    (197, 256, 2, 260, 17),    # d_head 128, keys split
    (40, 256, 2, 128, 300),    # d_head 128, queries to every wave, 12000 rows
    (1, 64, 1, 64, 1),         # one row, one key
    (17, 400, 8, 64, 2),       # K > 384: LayerNorm on its own, d_head 50 on the vector ALU
    (19, 18, 3, 30, 4),        # K and N not multiples of 4
    (19, 20, 2, 30, 4),        # only N is not
    (21, 36, 6, 40, 3),        # d_head 6
    (9, 288, 2, 64, 2),        # d_head 144
])
def test_f32_shapes(T, D, Hh, M, B):
    run(T, D, Hh, M, B)


@pytest.mark.parametrize("T,D,Hh,M,B", [(65, 192, 3, 768, 1), (33, 132, 3, 520, 60)])
def test_f32_buffers_off_16_byte_alignment(T, D, Hh, M, B):
    run(T, D, Hh, M, B, offset=1)


# tokens, images; keys split over waves (65: the first wave meets finite scores after its -inf ones, 50: never) and not
@pytest.mark.parametrize("T,B", [(65, 1), (50, 1), (65, 320)])
def test_f32_attention_scores_of_minus_infinity(T, B):
    """The first 16 keys score -1e60, -inf in fp32: weight zero, the other keys share the softmax."""
    sh = synth.custom_shape(f"neginf_{T}", 1, 64, 1, 64, T)
    p = synth.layer_params(sh, 0, w_std=0.1)
    for n in ("w_fc2", "b_fc2"):
        p[n] = np.zeros_like(p[n])
    p["w_qkv"][:128] = 0.0
    p["b_qkv"][:128] = 0.0
    p["b_qkv"][0] = p["w_qkv"][64, 0] = 1e30       # q = (1e30, 0, ...), k = (1e30 LN1(x)[0], 0, ...)
    x = np.zeros((B, T, 64), np.float32)
    x[:, :16, 0], x[:, :16, 1] = -1.0, 1.0
    x[:, 16:, 2], x[:, 16:, 3] = 1.0, -1.0
    got = H.run_stage(H.make_stage(sh, [p], 0, 1, B, bf16=False), x)
    ref = oracle.stage_forward(H.oracle_cfg(sh), [p], x[:1])
    assert H.rel_err(got[[0, B // 2, B - 1]], ref) <= H.TOL_F32


def test_f32_trace_of_a_layernorm_inside_a_dense_layer():
    sh = synth.SHAPES["tiny"]
    st = H.make_stage(sh, [synth.layer_params(sh, l) for l in range(2)], 0, 2, 1, bf16=False)
    x = synth.activations(sh, 1)
    want = H.run_stage(st, x)
    for kid in range(len(binding.KERNEL_NAMES)):
        st.trace_begin(kid, 2)
        np.testing.assert_array_equal(H.run_stage(st, x), want)
        n, sec = st.trace_end()
        assert n == 2 and sec >= 0


def test_f32_attention_on_the_largest_grid():
    """2^24 - 1 (image, head) pairs of one token, a workgroup each: 256 threads less than a grid may have.  61455 images,
    the same 61 over and over: the oracle on those, and every other one their bits."""
    import torch
    n, B = 61, 61455
    sh = synth.custom_shape("f32k_grid", 1, 1092, 273, 4, 1)
    layers = [synth.layer_params(sh, 0, randomize_affine=True, w_std=0.1)]
    x = synth.activations(sh, n)
    st = H.make_stage(sh, layers, 0, 1, B, bf16=False)
    xin = torch.from_numpy(np.resize(x, (B, 1, 1092))).cuda()
    out = torch.full_like(xin, float("nan"))
    st.forward(xin, B, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert H.rel_err(out[:n].cpu().numpy(), oracle.stage_forward(H.oracle_cfg(sh), layers, x)) <= H.TOL_F32
    k = B // n * n
    assert torch.equal(out[:k].view(-1, n, 1092), out[:n].view(1, n, 1092).expand(k // n, n, 1092))
    assert torch.equal(out[k:], out[:B - k])
    st.destroy()
