"""What a user of this package has it do, at the sizes and with the options they use, as cases that can be timed.

A case is a dict of plain values.  `kind` names the entry points it goes through:
  vit     slide_step_fwd + slide_step_bwd (`chunk` > 0: slide_step_chunked; `op` "encode": encoder_fwd_tiles)
  resnet  resnet_slide_step_fwd + resnet_slide_step_bwd
  pool    mil_pool_fwd + mil_pool_bwd (`op` "serve": mil_pool_fwd_static)
  adamw   slide_adamw_step
Everything is enqueued on torch's current stream and nothing is waited for, as in a training or serving loop.
"""
import math

import torch

from paper_2403_04865_amd import ResNetConfig, ResNetLib, SlideConfig, SlideLib

# encoder shapes: tile, patch, width, blocks, heads (MLP ratio 4).  The two-block one is the shape of the quick-start
# step, the others are ViT-S/16 and ViT-B/16 on 224-pixel tiles.
VIT = {
    "tiny": (32, 8, 64, 2, 2),
    "vit_s": (224, 16, 384, 12, 6),
    "vit_b": (224, 16, 768, 12, 12),
}
RESNET = {
    "rn18": (0, (2, 2, 2, 2)),
    "rn50": (1, (3, 4, 6, 3)),
}
TILE = 224
WIDTH = 64


def _vit(model, tiles, dtype="bf16", mil_hidden=128, classes=1, recompute=False, pixel_grad=False, chunk=0, op="step"):
    return dict(kind="vit", op=op, model=model, tiles=tiles, dtype=dtype, mil_hidden=mil_hidden, classes=classes,
                recompute=recompute, pixel_grad=pixel_grad, chunk=chunk)


def _pool(op, rows, dim=384, mil_hidden=128, classes=1):
    return dict(kind="pool", op=op, rows=rows, dim=dim, mil_hidden=mil_hidden, classes=classes)


def _resnet(model, tiles):
    return dict(kind="resnet", model=model, tiles=tiles, mil_hidden=128, classes=1)


def listed():
    return [
        # the quick-start step: a few hundred short launches, so it is their number and their gaps that count
        dict(_vit("tiny", 16, mil_hidden=32), name="tiny_step_16"),
        # a needle biopsy: a bag of a few dozen tiles
        dict(_vit("vit_s", 37), name="vit_s_step_37"),
        # a slide that is held whole: the ordinary training step
        dict(_vit("vit_s", 2048), name="vit_s_step_2048"),
        # a slide beyond the arena, chunk by chunk, with gradients to the pixels (saliency, adversarial training) and the
        # wider aggregator over four classes; neither count fits a power of two
        dict(_vit("vit_s", 1100, mil_hidden=256, classes=4, pixel_grad=True, chunk=384), name="vit_s_chunked_1100_pixels"),
        # 728 tiles through the large encoder, block inputs kept and blocks run again in the backward
        dict(_vit("vit_b", 728, mil_hidden=256, recompute=True), name="vit_b_recompute_728"),
        # float32 throughout: the gradient checks and the runs that settle whether a difference is rounding
        dict(_vit("vit_s", 61, dtype="fp32"), name="vit_s_step_fp32_61"),
        # feature extraction: forward only, nothing kept (`recompute` is what makes the stated arena a small one)
        dict(_vit("vit_s", 3001, recompute=True, op="encode"), name="vit_s_encode_3001"),
        # training the aggregator alone on the stored features of a whole slide (11 x 4,096 tiles)
        dict(_pool("train", 45056, mil_hidden=256), name="pool_train_45056"),
        # slide-level prediction from stored features in a serving loop: one short call
        dict(_pool("serve", 1037), name="pool_serve_1037"),
        # convolutional tile encoders, whole-slide batch statistics
        dict(_resnet("rn18", 1024), name="rn18_step_1024"),
        dict(_resnet("rn50", 300), name="rn50_step_300"),
        # the optimiser's update of every ViT-S parameter
        dict(kind="adamw", count=21_860_000, name="adamw_vit_s"),
    ]


def _spread(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.randrange(12)
    classes = rng.choice((1, 1, 2, 4))
    hidden = rng.choice((128, 256))
    if family == 0:
        return _vit("tiny", _spread(rng, 3, 256), dtype=rng.choice(("bf16", "fp32")), mil_hidden=rng.choice((32, 64)),
                    classes=classes)
    if family == 1:
        return _vit("vit_s", _spread(rng, 8, 256), mil_hidden=hidden, classes=classes, pixel_grad=rng.random() < 0.3)
    if family == 2:
        return _vit("vit_s", _spread(rng, 257, 2048), mil_hidden=hidden, classes=classes, recompute=rng.random() < 0.3)
    if family == 3:
        n = _spread(rng, 96, 1280)
        return _vit("vit_s", n, mil_hidden=hidden, classes=classes, pixel_grad=rng.random() < 0.5,
                    chunk=rng.randint(max(16, n // 6), n // 2))
    if family == 4:
        return _vit("vit_b", _spread(rng, 16, 728), mil_hidden=hidden, classes=classes, recompute=rng.random() < 0.5)
    if family == 5:
        return _vit("vit_s", _spread(rng, 4, 61), dtype="fp32", mil_hidden=hidden, classes=classes)
    if family == 6:
        model = rng.choice(("vit_s", "vit_s", "vit_b"))
        return _vit(model, _spread(rng, 1, 3072 if model == "vit_s" else 1024), recompute=True, op="encode")
    if family == 7:
        return _pool("train", _spread(rng, 512, 131072), dim=rng.choice((384, 384, 768)), mil_hidden=hidden, classes=classes)
    if family == 8:
        return _pool("serve", _spread(rng, 100, 65536), dim=rng.choice((384, 384, 768)), mil_hidden=hidden, classes=classes)
    if family == 9:
        return _resnet("rn18", _spread(rng, 32, 1024))
    if family == 10:
        return _resnet("rn50", _spread(rng, 16, 300))
    return dict(kind="adamw", count=_spread(rng, 150_000, 86_500_000))


# ---- inputs ------------------------------------------------------------------------------------------------------

def _pixels(n, side, dtype, g):
    """Normalised tiles: smoothed noise around mid-grey, clipped to what an 8-bit scanner can deliver."""
    out = torch.empty((n, 3, side, side), dtype=dtype, device="cuda")
    for lo in range(0, n, 512):
        k = min(512, n - lo)
        x = torch.nn.functional.avg_pool2d(torch.randn((k, 3, side + 4, side + 4), device="cuda", generator=g), 5, stride=1)
        out[lo:lo + k] = (x * 1.25).clamp_(-0.5, 0.5).mul_(4.0)
    return out


def _vit_params(layout, count, g):
    """Matrices, tables, biases and shifts of a network some way into its training: normal with deviation 0.02, cut at two
    deviations; LayerNorm gains around one."""
    p = torch.randn(count, device="cuda", generator=g).clamp_(-2.0, 2.0).mul_(0.02)
    for name, off, length in layout:
        if name.endswith(".g"):
            p[off:off + length] += 1.0
    return p


def _resnet_params(layout, count, g):
    """Convolutions with the fan-out law of rectifier networks, batch-norm gains around one, shifts around zero."""
    p = torch.randn(count, device="cuda", generator=g)
    for i, (name, off, length) in enumerate(layout):
        v = p[off:off + length]
        if name.startswith(("mil.", "head.")):
            v.clamp_(-2.0, 2.0).mul_(0.02 if name.endswith(".b") else 0.05)
        elif name.endswith(".W"):
            out = layout[i + 1][2]     # the batch-norm gain behind a convolution has one entry per output channel
            taps = 49 if name.startswith("stem") else 9 if _three_by_three(name, layout) else 1
            v.mul_(math.sqrt(2.0 / (out * taps)))
        elif name.endswith(".g"):
            v.mul_(0.1).add_(1.0)
        else:
            v.mul_(0.1)
    return p


def _three_by_three(name, layout):
    """Whether a block's convolution is 3x3: all of a basic block's, the middle one of a bottleneck block's; never a
    shortcut's."""
    if ".down." in name:
        return False
    bottleneck = any(n.endswith("conv3.W") for n, _, _ in layout)
    return name.endswith("conv2.W") if bottleneck else True


def _features(rows, dim, g):
    """Rows as a final LayerNorm leaves them: a component that all tiles share plus a smaller one of the tile's own."""
    return torch.randn(dim, device="cuda", generator=g) + 0.25 * torch.randn((rows, dim), device="cuda", generator=g)


def _arena(nbytes):
    a = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    o = (-a.data_ptr()) % 256
    return a[o:o + nbytes]


def _label(case, seed):
    return seed % (2 if case["classes"] == 1 else case["classes"])


def _vit_config(case):
    tile, patch, dim, layers, heads = VIT[case["model"]]
    return SlideConfig(tile, patch, dim, layers, heads, 4, case["mil_hidden"], case["classes"],
                       dtype=1 if case["dtype"] == "bf16" else 0, recompute=int(case["recompute"]))


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "adamw":
        n = case["count"]
        s["params"] = torch.randn(n, device="cuda", generator=g).mul_(0.02)
        s["grads"] = torch.randn(n, device="cuda", generator=g).mul_(1e-3)
        s["m"] = torch.randn(n, device="cuda", generator=g).mul_(3e-4)
        s["v"] = torch.rand(n, device="cuda", generator=g).mul_(2e-6)
        s["step"] = 100
        s["lib"] = SlideLib(SlideConfig(32, 8, 64, 2, 2, 4, 32, 1))
        return s
    s["label"] = _label(case, seed)
    s["loss"] = torch.zeros(1, device="cuda")
    s["logits"] = torch.zeros(case["classes"], device="cuda")
    if kind == "pool":
        rows, dim = case["rows"], case["dim"]
        lib = SlideLib(SlideConfig(TILE, 16, dim, 0, dim // 64, 4, case["mil_hidden"], case["classes"], dtype=1))
        s["params"] = _vit_params(lib.param_layout(), lib.slide_param_count(), g)
        s["feats"] = _features(rows, dim, g)
        s["alpha"] = torch.zeros(rows, device="cuda")
        if case["op"] == "train":
            s["grads"] = torch.zeros_like(s["params"])
            s["dfeats"] = torch.zeros_like(s["feats"])
            lib.slide_bind(s["params"], s["grads"], _arena(lib.slide_pool_arena_bytes(rows)))
        s["lib"] = lib
        return s
    n = case["tiles"]
    if kind == "resnet":
        block, depths = RESNET[case["model"]]
        lib = ResNetLib(ResNetConfig(TILE, block, depths, WIDTH, case["mil_hidden"], case["classes"]))
        s["params"] = _resnet_params(lib.param_layout(), lib.resnet_param_count(), g)
        s["grads"] = torch.zeros_like(s["params"])
        s["alpha"] = torch.zeros(n, device="cuda")
        s["pixels"] = _pixels(n, TILE, torch.bfloat16, g)
        lib.resnet_bind(s["params"], s["grads"], _arena(lib.resnet_arena_bytes(n)))
        s["lib"] = lib
        return s
    lib = SlideLib(_vit_config(case))
    s["params"] = _vit_params(lib.param_layout(), lib.slide_param_count(), g)
    s["grads"] = torch.zeros_like(s["params"])
    s["pixels"] = _pixels(n, VIT[case["model"]][0], torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, g)
    if case["op"] == "encode":
        s["feats"] = torch.zeros((n, VIT[case["model"]][2]), device="cuda")
    nbytes = lib.slide_chunked_arena_bytes(n, case["chunk"]) if case["chunk"] else lib.slide_arena_bytes(n)
    s["alpha"] = torch.zeros(n, device="cuda")
    s["dpixels"] = torch.zeros_like(s["pixels"]) if case["pixel_grad"] else None
    lib.slide_bind(s["params"], s["grads"], _arena(nbytes))
    s["lib"] = lib
    return s


def run(s):
    case, lib = s["case"], s["lib"]
    kind = case["kind"]
    if kind == "adamw":
        s["step"] += 1
        lib.slide_adamw_step(s["params"], s["grads"], s["m"], s["v"], case["count"], s["step"], 5e-5)
        return {"params": s["params"], "m": s["m"], "v": s["v"]}
    out = {"loss": s["loss"], "logits": s["logits"]}
    if kind == "pool":
        rows = case["rows"]
        out["alpha"] = s["alpha"]
        if case["op"] == "serve":
            lib.mil_pool_fwd_static(s["params"], s["feats"], rows, s["label"], s["loss"], s["logits"], s["alpha"])
            return out
        lib.mil_pool_fwd(s["feats"], rows, s["label"], s["loss"], s["logits"], s["alpha"])
        lib.mil_pool_bwd(s["feats"], rows, s["label"], s["dfeats"], 0)
        out.update(dfeats=s["dfeats"], grads=s["grads"])
        return out
    n = case["tiles"]
    out.update(alpha=s["alpha"], grads=s["grads"])
    if kind == "resnet":
        lib.resnet_slide_step_fwd(s["pixels"], n, s["label"], s["loss"], s["logits"], s["alpha"])
        lib.resnet_slide_step_bwd(0)
        return out
    if case["op"] == "encode":
        lib.encoder_fwd_tiles(s["pixels"], n, s["feats"], 0)
        return {"feats": s["feats"]}
    if case["chunk"]:
        lib.slide_step_chunked(s["pixels"], n, case["chunk"], s["label"], 0, s["loss"], s["logits"], s["alpha"], s["dpixels"])
    else:
        lib.slide_step_fwd(s["pixels"], n, s["label"], s["loss"], s["logits"], s["alpha"])
        lib.slide_step_bwd(0, s["dpixels"])
    if s["dpixels"] is not None:
        out["dpixels"] = s["dpixels"]
    return out


# ---- work and tolerance --------------------------------------------------------------------------------------------

def _pool_work(rows, dim, hidden, train):
    """Gate projections forward; backward: the gradient of the features and of the two gate matrices."""
    return {"bytes": rows * dim * 4.0 * (2 if train else 1) + rows * 4.0 + 2.0 * hidden * dim * 4 * (2 if train else 1),
            "flops": 4.0 * rows * dim * hidden * (3 if train else 1)}


def _resnet_flops(model):
    """Forward flops of one tile and those of them that have an input gradient (all convolutions but the first)."""
    block, depths = RESNET[model]
    grow = 4 if block else 1
    stem = 2.0 * (TILE // 2) ** 2 * WIDTH * 3 * 49
    rest, side, cin = 0.0, TILE // 4, WIDTH
    for stage, depth in enumerate(depths):
        mid = WIDTH << stage
        for b in range(depth):
            stride = 2 if b == 0 and stage > 0 else 1
            o = side // stride
            if block:
                rest += 2.0 * (side * side * cin * mid + o * o * mid * mid * 9 + o * o * mid * mid * grow)
            else:
                rest += 2.0 * 9 * o * o * (cin * mid + mid * mid)
            if stride != 1 or cin != mid * grow:
                rest += 2.0 * o * o * cin * mid * grow
            side, cin = o, mid * grow
    return stem, rest


def work(case):
    kind = case["kind"]
    if kind == "adamw":
        return {"bytes": 28.0 * case["count"], "flops": 12.0 * case["count"]}
    if kind == "pool":
        return _pool_work(case["rows"], case["dim"], case["mil_hidden"], case["op"] == "train")
    n = case["tiles"]
    if kind == "resnet":
        stem, rest = _resnet_flops(case["model"])
        params = 11.2e6 if case["model"] == "rn18" else 23.5e6
        return {"bytes": n * 3.0 * TILE * TILE * 2 + params * 8, "flops": n * (2 * stem + 3 * rest)}
    side, patch, D, L, H = VIT[case["model"]]
    T, F, Kp, dh = (side // patch) ** 2 + 1, 4 * D, 3 * patch * patch, D // H
    e = 2 if case["dtype"] == "bf16" else 4
    block = 2.0 * T * D * 3 * D + 2.0 * T * D * D + 4.0 * T * D * F + 4.0 * H * T * T * dh
    # of the last block's output only the class token is read: projection, MLP and attention queries of the other tokens
    # are not needed
    unread = (T - 1) * (2.0 * D * D + 4.0 * D * F) + 4.0 * H * (T - 1) * T * dh
    blocks = L * block - unread
    embed = 2.0 * (T - 1) * Kp * D
    params = D * Kp + T * D + 2 * D + L * (12 * D * D + 13 * D) + 2 * case["mil_hidden"] * D
    pixels = n * 3.0 * side * side * e
    if case["op"] == "encode":
        return {"bytes": pixels + params * 4.0 + n * D * 4.0, "flops": n * (embed + blocks)}
    flops = 2 * embed + 3 * blocks
    if case["chunk"]:
        flops += embed + blocks                # the activations do not fit: the forward runs a second time
    elif case["recompute"]:
        flops += blocks - block                # all blocks but the last run again
    if case["pixel_grad"]:
        flops += embed
    return {"bytes": pixels * (2 if case["pixel_grad"] else 1) + params * 8.0, "flops": n * flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "adamw":
        return {"rel": 1e-5}
    if kind == "resnet":
        # bf16 activations; where two correct forwards leave a pre-activation on different sides of zero their gradients
        # differ by the whole element, so the gradients agree less well than the storage type alone would give
        return {"rel": 3e-2, "max": 0.9}
    if kind == "pool":
        # the gate projections multiply bf16 numbers; what they feed averages over the rows, features and sums are float32
        return {"rel": 2e-3, "max": 2e-2}
    if case["dtype"] == "fp32":
        return {"rel": 5e-5, "max": 1e-2}
    # a dozen blocks of bf16 activations; one gradient vector holds tensors of very different size, so single elements of
    # the larger ones are off by more than the root mean square of the whole
    return {"rel": 2e-2, "max": 0.99}
