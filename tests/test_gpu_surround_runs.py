"""GPU parity of the embedding and the head where pixels, tokens or buffers are not whole 16-byte pieces: patch rows
of 2 and 7 pixels, images and tokens that start 4 bytes past such a piece, an fp32 width that is not a multiple of
four.  Against the checker; tolerances of the paths."""
import numpy as np
import pytest

import oracle
from paper_2110_14895_amd import binding, synth
from tests import harness as H

pytestmark = pytest.mark.gpu


def shifted(a, shift):
    """`a` on the device, `shift` floats past a fresh allocation."""
    import torch
    flat = torch.empty(a.size + shift, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(a).cuda().reshape(-1)
    return flat[shift:].view(a.shape)


# patch runs of 2 (K = 12 of 64), 1 (K = 49 of 64) and 4 pixels, the last from an unaligned image
@pytest.mark.parametrize("size,patch,channels,d,bf16,shift", [
    (6, 2, 3, 64, True, 0), (21, 7, 1, 64, True, 0), (16, 4, 3, 128, True, 1), (16, 4, 3, 128, False, 1), (6, 2, 3, 30, False, 0),
])
def test_embedding_runs(size, patch, channels, d, bf16, shift):
    import torch
    T, B = 1 + (size // patch) ** 2, 3
    sh = synth.custom_shape(f"run{size}_{patch}", 1, d, 1, 4 * d, T)
    prm = synth.surround_params(sh, patch, channels, 8, 5, bf16=bf16)
    dt = binding.EP_BF16 if bf16 else binding.EP_F32
    emb = binding.Embed(size, patch, channels, d, dt, binding.EP_F32, synth.as_param_dtype(prm, bf16), B)
    img = synth.images(B, channels, size, seed=2)
    out = shifted(np.full((B, T, d), np.nan, np.float32), shift)
    emb.forward(shifted(img, shift), B, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = oracle.embed_forward(img, prm["w_patch"], prm["b_patch"], prm["cls"], prm["pos"], patch)
    assert H.rel_err(out.cpu().numpy(), ref) <= (H.TOL_BF16 if bf16 else H.TOL_F32)


# widths at and past the 2^20 columns that the one-tile-per-workgroup kernel takes; K of one and of two steps (two may
# run on the persistent kernel)
@pytest.mark.parametrize("d,channels", [((1 << 20) - 64, 3), (1 << 20, 3), ((1 << 20) + 192, 5)])
def test_embedding_of_a_million_columns(d, channels):
    import torch
    B, K = 3, 16 * channels
    rng = np.random.default_rng(7)
    prm = {n: synth.round_to_bf16(rng.standard_normal(s, dtype=np.float32) * 0.05).reshape(s)
           for n, s in (("w_patch", (d, K)), ("b_patch", (d,)), ("cls", (d,)), ("pos", (2, d)))}
    emb = binding.Embed(4, 4, channels, d, binding.EP_BF16, binding.EP_F32, synth.as_param_dtype(prm, True), B)
    img = synth.images(B, channels, 4, seed=2)
    out = torch.full((B, 2, d), float("nan"), dtype=torch.float32, device="cuda")
    emb.forward(torch.from_numpy(img).cuda(), B, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    emb.destroy()
    ref = oracle.embed_forward(img, prm["w_patch"], prm["b_patch"], prm["cls"], prm["pos"], 4)
    assert H.rel_err(out.cpu().numpy(), ref) <= H.TOL_BF16


# The same with 256 rows: tiles as tall as any kernel has them, in a layer whose rows of the output are 4 MB each, the last
# columns not a whole tile.  Against the same products in 64 bits of the bf16 operands: sums of 108 products in fp32 stay
# within 111 roundings of 2^-24 of the sum of the terms' magnitudes, here 4 to 7, so within 5e-5.
def test_embedding_of_a_million_columns_and_many_rows():
    import torch
    d, patch, size = 1052736, 6, 96
    T, K = 257, 108
    rng = np.random.default_rng(11)
    bits = synth.f32_to_bf16_bits(rng.standard_normal(65521, dtype=np.float32) * 0.05)       # a prime: no two rows alike
    prm = {n: np.resize(np.roll(bits, 1000 * i), s) for i, (n, s) in
           enumerate((("w_patch", (d, K)), ("b_patch", (d,)), ("cls", (d,)), ("pos", (T, d))))}
    emb = binding.Embed(size, patch, 3, d, binding.EP_BF16, binding.EP_F32, prm, 1)
    img = synth.images(1, 3, size, seed=2)
    out = torch.full((T, d), float("nan"), dtype=torch.float32, device="cuda")
    emb.forward(torch.from_numpy(img).cuda(), 1, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    emb.destroy()

    def up(a):
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16).double()

    g = size // patch
    rows = torch.from_numpy(img).cuda().to(torch.bfloat16).double().view(3, g, patch, g, patch).permute(1, 3, 0, 2, 4).reshape(g * g, K)
    for c in range(0, d, 1 << 16):
        e = min(c + (1 << 16), d)
        pos = up(np.ascontiguousarray(prm["pos"][:, c:e]))
        ref = torch.cat([up(prm["cls"][c:e])[None] + pos[:1], rows @ up(prm["w_patch"][c:e]).T.contiguous() + up(prm["b_patch"][c:e]) + pos[1:]])
        err = (out[:, c:e].double() - ref).abs().max().item()
        assert err <= 5e-5, (c, err)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shift", [0, 1])
def test_head_takes_tokens_where_they_lie(bf16, shift):
    import torch
    d, T, nc, B = 192, 65, 16, 7
    sh = synth.custom_shape("headrow", 1, d, 3, 4 * d, T)
    prm = synth.surround_params(sh, 2, 1, nc, 5, bf16=bf16)
    head = binding.Head(d, T, nc, sh.ln_eps, binding.EP_BF16 if bf16 else binding.EP_F32, synth.as_param_dtype(prm, bf16), B)
    x = (2.0 * synth.normal("head/rows", B * T * d, 1)).reshape(B, T, d).astype(np.float32)
    logits = torch.full((B, nc), float("nan"), dtype=torch.float32, device="cuda")
    head.forward(shifted(x, shift), B, logits, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = oracle.head_forward(x, prm["ln_g"], prm["ln_b"], sh.ln_eps, prm["w_head"], prm["b_head"])
    assert H.rel_err(logits.cpu().numpy(), ref) <= (H.TOL_BF16 if bf16 else H.TOL_F32)


# class tokens 2^31 floats apart and just below, where LayerNorm itself steps from one to the next; of one image no second row is there
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("T,B", [((1 << 21) - 1, 2), (1 << 21, 2), (1 << 21, 1)])
def test_head_over_many_tokens(bf16, T, B):
    import torch
    d, nc = 1024, 16
    prm = synth.surround_params(synth.custom_shape("headfar", 1, d, 16, 4 * d, 2), 2, 1, nc, 5, bf16=bf16)
    head = binding.Head(d, T, nc, 1e-6, binding.EP_BF16 if bf16 else binding.EP_F32, synth.as_param_dtype(prm, bf16), B)
    rows = (2.0 * synth.normal("head/far", B * d, 1)).reshape(B, 1, d).astype(np.float32)
    x = torch.empty((B - 1) * T * d + d, dtype=torch.float32, device="cuda")
    for i in range(B):
        x[i * T * d:][:d] = torch.from_numpy(rows[i, 0]).cuda()
    logits = torch.full((B, nc), float("nan"), dtype=torch.float32, device="cuda")
    head.forward(x, B, logits, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = oracle.head_forward(rows, prm["ln_g"], prm["ln_b"], 1e-6, prm["w_head"], prm["b_head"])
    assert H.rel_err(logits.cpu().numpy(), ref) <= (H.TOL_BF16 if bf16 else H.TOL_F32)
