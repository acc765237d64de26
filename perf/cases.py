"""Workloads of the pipeline-stage library, for timing it and for comparing two builds of it.

A case is a dict of plain values.  `entry` says which public call it goes through:

  stage     binding.Stage.forward          one pipeline stage on one micro-batch
  static    binding.Stage.forward_static   the same for callers that cannot allocate
  pipeline  binding.Pipeline.run           a model cut evenly into stages, several micro-batches in flight
  model     binding.Embed -> Stage (all layers) -> Head, images to logits

`model` names a shape of synth.SHAPES, `image` the pixels per side its token count comes from, `layers` how many
of its layers run, `dtype` the arithmetic path ("bf16" or "f32"); `in` / `out` (and `mid`, between the stages of a
pipeline) are the types of the activations at the boundaries.  Weights are N(0, 0.02), biases and LayerNorm shifts
N(0, 0.02), gains 1 + N(0, 0.02), activations and pixels N(0, 1), as in the library's own benchmark recipe.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2110_14895_amd import binding, synth

CLASSES = 1000
# pixels per side of a patch, by model: 32 / 4, 224 / 16 and 224 / 14 give the token counts of synth.SHAPES
PATCH = {"tiny": 4, "deit_tiny": 16, "deit_small": 16, "vit_base": 16, "vit_large": 16, "vit_huge": 14}
NATIVE_IMAGE = {"tiny": 32, "deit_tiny": 224, "deit_small": 224, "vit_base": 224, "vit_large": 224, "vit_huge": 224}
STATIC_WORKSPACE = 64 << 20         # EP_STATIC_SCRATCH_BYTES of include/edgepipe.h


def case(name, entry, model, layers, batch, **more):
    c = {"name": name, "entry": entry, "model": model, "layers": layers, "batch": batch, "dtype": "bf16",
         "image": NATIVE_IMAGE[model], "in": "bf16", "out": "f32"}
    c.update(more)
    if c["dtype"] == "f32":
        c["in"] = c["out"] = "f32"
    return c


def listed():
    return [
        # the smallest call: two narrow fp32 layers on one image, the configuration for exact checks
        case("tiny_f32_b1", "stage", "tiny", 2, 1, dtype="f32"),
        # fp32 inference of a narrow whole model, images to logits, on a small batch of ordinary images
        case("deit_tiny_f32_model_b8", "model", "deit_tiny", 12, 8, dtype="f32"),
        # one image through one stage: a request served on its own, as an edge pipeline does; no allocation
        case("vit_large_6l_b1_static", "static", "vit_large", 6, 1),
        # a stage of a base model at the paper's pipeline micro-batch
        case("vit_base_3l_b8", "stage", "vit_base", 3, 8),
        # a ragged micro-batch in the middle of a pipeline: fp32 in from the stage before, bf16 out to the next
        case("vit_large_6l_b5_mid", "stage", "vit_large", 6, 5, **{"in": "f32", "out": "bf16"}),
        # larger images (384 x 384: 577 tokens), two at a time
        case("vit_base_12l_b2_384", "stage", "vit_base", 12, 2, image=384),
        # narrow whole model, images to logits
        case("deit_small_model_b32", "model", "deit_small", 12, 32),
        # four stages on one device, eight micro-batches of eight images flowing through
        case("vit_base_pipeline_4x8", "pipeline", "vit_base", 12, 8, stages=4, micros=8, mid="f32"),
        # stages of a large model at ordinary micro-batches
        case("vit_large_6l_b16", "stage", "vit_large", 6, 16),
        case("vit_large_6l_b32", "stage", "vit_large", 6, 32),
        # an uneven stage of a heterogeneous partition at the largest micro-batch
        case("vit_huge_3l_b256", "stage", "vit_huge", 3, 256, **{"in": "f32"}),
        # the whole largest model on one device, the benchmark workload
        case("vit_huge_32l_b64", "stage", "vit_huge", 32, 64),
    ]


def shape_of(c):
    sh = synth.SHAPES[c["model"]]
    return dataclasses.replace(sh, n_tokens=1 + (c["image"] // PATCH[c["model"]]) ** 2)


def images_of(c):
    return c["batch"] * c.get("micros", 1)


def flops(c):
    sh = shape_of(c)
    f = images_of(c) * c["layers"] * sh.flops_per_image_per_layer()
    if c["entry"] == "model":
        k = 3 * PATCH[c["model"]] ** 2
        f += 2.0 * images_of(c) * sh.d_model * ((sh.n_tokens - 1) * k + CLASSES)
    return f


def work(c):
    """Parameters and inputs read once, outputs written once."""
    sh = shape_of(c)
    d, m, n = sh.d_model, sh.d_mlp, images_of(c)
    size = 4 if c["dtype"] == "f32" else 2
    by = c["layers"] * size * (4 * d * d + 2 * d * m + 9 * d + m)
    tokens = n * sh.n_tokens * d
    if c["entry"] == "model":
        k = 3 * PATCH[c["model"]] ** 2
        by += size * (d * k + (sh.n_tokens + 2) * d + CLASSES * (d + 1) + 2 * d)
        by += n * (3 * c["image"] ** 2 + CLASSES) * 4 + tokens * 4
    else:
        by += tokens * (4 if c["in"] == "f32" else 2) + tokens * (4 if c["out"] == "f32" else 2)
    return {"bytes": float(by), "flops": flops(c)}


def tolerance(c):
    # Four times the differences to the same layers in 64 bits.  Measured, as a share of the output's norm and at the
    # worst element of its root mean square: bf16 operands 2.8e-3 and 1.2e-2 over six layers (output in bf16),
    # 4.1e-3 and 1.8e-2 over 12 to 32 layers; fp32 sums 1.0e-6 and 4.4e-6.
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1.8e-5}
    return {"rel": 1.1e-2, "max": 5e-2} if c["layers"] <= 6 else {"rel": 1.6e-2, "max": 7e-2}


def draw(rng):
    """One more case of the ranges above, never dearer than the largest of them."""
    entry = rng.choice(["stage"] * 5 + ["static", "model", "model", "pipeline", "pipeline"])
    dtype = rng.choice(["bf16"] * 4 + ["f32"])
    most = 22e12 if dtype == "bf16" else 0.16e12
    while True:
        models = ["tiny", "deit_tiny", "deit_small"] if dtype == "f32" else \
            ["deit_tiny", "deit_small", "vit_base", "vit_large", "vit_huge"]
        model = rng.choice(models)
        full = synth.SHAPES[model].n_layers
        layers = full if entry == "model" else min(full, int(round(math.exp(rng.uniform(0.0, math.log(full + 0.49))))))
        batch = int(round(math.exp(rng.uniform(0.0, math.log(256.0)))))
        image = NATIVE_IMAGE[model]
        if model in ("deit_small", "vit_base", "vit_large") and rng.random() < 0.15:
            image = 384
        c = case("", entry, model, layers, batch, dtype=dtype, image=image)
        del c["name"]
        if dtype == "bf16" and entry != "model":
            c["in"], c["out"] = rng.choice(["bf16", "bf16", "f32"]), rng.choice(["f32", "f32", "bf16"])
        if entry == "pipeline":
            if layers < 2:
                continue
            c["stages"] = rng.randint(2, min(4, layers))
            c["micros"] = rng.randint(2, 8)
            c["mid"] = rng.choice(["f32", "bf16"]) if dtype == "bf16" else "f32"
        # a layer of the smallest micro-batch costs about as much time as 70 GFLOP of a large one (f32: 2 GFLOP)
        if flops(c) + (7e10 if dtype == "bf16" else 2e9) * layers * c.get("micros", 1) > most:
            continue
        if entry == "static":
            sh = shape_of(c)
            e = 4 if dtype == "f32" else 2
            row = 4 * sh.d_model + e * sh.d_model + e * max(3 * sh.d_model, sh.d_mlp)
            if batch * sh.n_tokens * row + 4096 > STATIC_WORKSPACE:
                continue
        return c


# ------------------------------------------------------------------------------------------ states
class _Maker:
    """Host parameters and device activations from one seed, drawn on the GPU."""

    def __init__(self, seed, bf16):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.bf16 = bf16

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)

    def param(self, *shape, mean=0.0, std=0.02):
        a = self.normal(*shape).mul_(std).add_(mean)
        if self.bf16:
            return a.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
        return a.cpu().numpy()

    def layer(self, sh):
        return {n: self.param(*s, mean=1.0 if n.endswith("_g") else 0.0) for n, s in sh.param_shapes().items()}


def _dt(name):
    return binding.EP_F32 if name == "f32" else binding.EP_BF16


def _buffer(name, *shape):
    return torch.zeros(shape, dtype=torch.float32 if name == "f32" else torch.bfloat16, device="cuda")


def prepare(c, seed):
    sh = shape_of(c)
    bf16 = c["dtype"] == "bf16"
    p = _dt(c["dtype"])
    mk = _Maker(seed, bf16)
    n, t, d = images_of(c), sh.n_tokens, sh.d_model

    def stage(begin, end, i, o, max_batch):
        cfg = binding.VitConfig(sh.n_layers, d, sh.n_heads, sh.d_mlp, t, sh.ln_eps, p, _dt(i), _dt(o))
        return binding.Stage(cfg, begin, end, [mk.layer(sh) for _ in range(begin, end)], max_batch)

    s = {"case": c}
    if c["entry"] == "model":
        k = PATCH[c["model"]]
        prm = {"w_patch": mk.param(d, 3 * k * k), "b_patch": mk.param(d), "cls": mk.param(d), "pos": mk.param(t, d),
               "ln_g": mk.param(d, mean=1.0), "ln_b": mk.param(d), "w_head": mk.param(CLASSES, d),
               "b_head": mk.param(CLASSES)}
        s["embed"] = binding.Embed(c["image"], k, 3, d, p, _dt(c["in"]), prm, n)
        s["stage"] = stage(0, c["layers"], c["in"], "f32", n)
        s["head"] = binding.Head(d, t, CLASSES, sh.ln_eps, p, prm, n)
        s["images"] = mk.normal(n, 3, c["image"], c["image"])
        s["x"] = _buffer(c["in"], n, t, d)
        s["out"] = _buffer("f32", n, t, d)
        s["logits"] = _buffer("f32", n, CLASSES)
        return s
    x = mk.normal(n, t, d)
    s["x"] = x if c["in"] == "f32" else x.to(torch.bfloat16)
    s["out"] = _buffer(c["out"], n, t, d)
    if c["entry"] == "pipeline":
        k = c["stages"]
        cuts = [round(i * c["layers"] / k) for i in range(k + 1)]
        s["stages"] = [stage(cuts[i], cuts[i + 1], c["in"] if i == 0 else c["mid"], c["out"] if i + 1 == k else c["mid"],
                             c["batch"]) for i in range(k)]
        s["pipeline"] = binding.Pipeline(s["stages"], c["batch"])
    else:
        s["stage"] = stage(0, c["layers"], c["in"], c["out"], 1 if c["entry"] == "static" else n)
    return s


def run(s):
    c = s["case"]
    stream = torch.cuda.current_stream()
    if c["entry"] == "model":
        s["embed"].forward(s["images"], c["batch"], s["x"], stream)
        s["stage"].forward(s["x"], c["batch"], s["out"], stream)
        s["head"].forward(s["out"], c["batch"], s["logits"], stream)
        return {"logits": s["logits"], "tokens": s["out"]}
    if c["entry"] == "pipeline":
        s["pipeline"].run(s["x"], c["micros"], s["out"], stream)
    elif c["entry"] == "static":
        s["stage"].forward_static(s["x"], c["batch"], s["out"], stream)
    else:
        s["stage"].forward(s["x"], c["batch"], s["out"], stream)
    return s["out"]
