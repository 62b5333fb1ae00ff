"""The work that users have this framework do, as timed cases.

A case is one merged forward pass: M fine-tuned instances of one network, each on its own input, through
the public classes of ``paper_2009_13062_amd.workloads`` or through the operators of the package itself.
The listed cases are this repository's benchmark workloads and what surrounds them in use: fewer models,
several sequences or images per model, sequences and images of any length or size, key masks and per-task
output layers, and float32 storage (the precision of the paper's own runs) beside bfloat16.  ``draw``
gives further cases of the same ranges.
"""
from __future__ import annotations

import torch

import paper_2009_13062_amd as nf
import netfuse_inputs as NI
from netfuse_inputs.device import encoder_stack_device, resnet_params_device
from paper_2009_13062_amd.workloads import EncoderStack, ResNetForward, TinyLayer

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _encoder(name, M, seq, layers=12, batch=1, hidden=768, ffn=None, dtype="bf16", rel=False, packed=True):
    c = dict(kind="encoder", M=M, layers=layers, batch=batch, seq=seq, hidden=hidden, heads=hidden // 64,
             ffn=ffn or 4 * hidden, dtype=dtype, rel=rel, packed=packed)
    return dict(name=name, **c) if name else c


def _classifier(name, M, seq, layers, batch, hidden=768, dtype="bf16"):
    c = dict(kind="classifier", M=M, layers=layers, batch=batch, seq=seq, hidden=hidden, heads=hidden // 64,
             ffn=4 * hidden, dtype=dtype)
    return dict(name=name, **c) if name else c


def _resnet(name, M, batch=1, image=224, cardinality=1, base_width=64, dtype="bf16"):
    c = dict(kind="resnet", M=M, batch=batch, image=image, cardinality=cardinality, base_width=base_width, dtype=dtype)
    return dict(name=name, **c) if name else c


def _layer(name, M, rows, features, outputs, channels, image, dtype):
    c = dict(kind="layer", M=M, rows=rows, features=features, outputs=outputs, channels=channels, image=image, dtype=dtype)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # two models of the two-layer example network and one small convolution, float32: the smallest calls, where
        # launches are everything
        _layer("layer_m2_f32", M=2, rows=8, features=64, outputs=64, channels=16, image=8, dtype="f32"),
        # one encoder layer over 8 models: an ordinary small call
        _encoder("encoder1_m8_s128", M=8, seq=128, layers=1),
        # a whole encoder over two models: the low end of the number of models worth merging
        _encoder("encoder12_m2_s128", M=2, seq=128),
        # the headline workload: 32 models, one sequence of 128 tokens each
        _encoder("encoder12_m32_s128", M=32, seq=128),
        # the longest sequences: the largest matrix products
        _encoder("encoder12_m32_s512", M=32, seq=512),
        # relative-position attention, 32 models
        _encoder("xlnet12_m32_s128", M=32, seq=128, rel=True),
        # a served classifier: several sequences per model padded to the longest (an odd length) and masked, row-major
        # weights, a per-task output layer of its own width for each model, outputs allocated by the call
        _classifier("classifier6_m12_b3_s93", M=12, seq=93, layers=6, batch=3),
        # the encoder in float32
        _encoder("encoder12_m8_s128_f32", M=8, seq=128, dtype="f32", packed=False),
        # the image networks of the benchmark
        _resnet("resnet50_m32", M=32),
        _resnet("resnext50_m16", M=16, cardinality=32, base_width=4),
        # few models, several images each, of a size whose planes have odd widths
        _resnet("resnet50_m3_b4_i200", M=3, batch=4, image=200),
        # the image network in float32
        _resnet("resnet50_m8_f32", M=8, dtype="f32"),
    ]


# Ranges of draw(): the models merged are 1 ... 32, sequences per model 1 ... 8, tokens 16 ... 512, layers 1 ... 12,
# images per model 1 ... 8, image sides 64 ... 288.  A draw over the cost of the largest listed case of its data
# type is drawn again.
def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _cost(case):
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / (5e14 if case["dtype"] == "bf16" else 5e13)


def draw(rng):
    most = {d: max(_cost(c) for c in listed() if c["dtype"] == d) for d in DTYPES}
    while True:
        kind = rng.choice(["encoder", "encoder", "encoder", "rel", "classifier", "classifier", "resnet", "resnet",
                           "resnext", "layer", "encoder_f32", "resnet_f32"])
        M = _log(rng, 1, 32)
        seq = rng.choice([_log(rng, 16, 512), 16 * _log(rng, 1, 32), 128])
        batch = _log(rng, 1, 8)
        layers = _log(rng, 1, 12)
        hidden = rng.choice([256, 768, 768, 1024])
        image = rng.choice([32 * rng.randint(2, 9), rng.randint(64, 288), 224])
        if kind == "encoder":
            c = _encoder(None, M, seq, layers, batch, hidden, packed=rng.random() < 0.75)
        elif kind == "rel":
            c = _encoder(None, M, min(seq, 320), layers, min(batch, 2), hidden, rel=True)
        elif kind == "classifier":
            c = _classifier(None, M, seq, layers, batch, hidden)
        elif kind == "resnet":
            c = _resnet(None, M, batch, image)
        elif kind == "resnext":
            c = _resnet(None, M, batch, image, 32, 4)
        elif kind == "encoder_f32":
            c = _encoder(None, min(M, 12), seq, layers, batch, hidden, dtype="f32", packed=False)
        elif kind == "resnet_f32":
            c = _resnet(None, min(M, 12), min(batch, 4), image, *rng.choice([(1, 64), (32, 4)]), dtype="f32")
        else:
            c = _layer(None, M, _log(rng, 1, 128), _log(rng, 9, 768), _log(rng, 7, 1024), 8 * rng.randint(1, 12),
                       rng.randint(5, 56), rng.choice(["f32", "bf16"]))
        if _cost(c) <= most[c["dtype"]]:
            return c


def _classes(case):
    """Output widths of the per-task layers: 2 ... 20 classes, another number for each model."""
    return [2 + (7 * m + 3) % 19 for m in range(case["M"])]


def prepare(case, seed):
    dt, M = DTYPES[case["dtype"]], case["M"]
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1))
    normal = lambda *s, mean=0.0, std=1.0, dtype=torch.float32: torch.empty(s, device="cuda").normal_(mean, std, generator=g).to(dtype)
    if case["kind"] == "layer":
        k, n, c, hw = case["features"], case["outputs"], case["channels"], case["image"]
        inp = dict(X=normal(M, case["rows"], k, dtype=dt), W=normal(M, k, n, std=0.02, dtype=dt), b=normal(M, n, std=0.02),
                   gamma=normal(M * n, mean=1.0, std=0.02), beta=normal(M * n, std=0.02),
                   conv_x=normal(1, M * c, hw, hw, dtype=dt), conv_w=normal(M * c, c, 3, 3, std=0.05, dtype=dt))
        return dict(kind="layer", net=TinyLayer(inp, M, dt))
    if case["kind"] == "resnet":
        spec = NI.resnet_spec(case["cardinality"], case["base_width"], case["image"])
        inp = resnet_params_device(spec, M, cfg=seed, dtype=dt, batch=case["batch"])
        return dict(kind="resnet", x=inp["x"], net=ResNetForward(spec, inp["params"], M, dtype=dt, batch=case["batch"]))
    B, S = case["batch"], case["seq"]
    shape = NI.EncoderShape(case["hidden"], case["heads"], case["ffn"], case["layers"], S, B)
    inp = encoder_stack_device(M, shape, cfg=seed, dtype=dt, rel=case.get("rel", False))
    if case["kind"] == "encoder":
        return dict(kind="encoder", x=inp["X"],
                    net=EncoderStack(inp["layers"], M, B, S, case["heads"], R=inp.get("R"), packed=case["packed"]))
    lengths = torch.randint(max(1, S // 2), S + 1, (M, B, 1), device="cuda", generator=g)
    mask = (torch.arange(S, device="cuda") >= lengths).float() * -10000.0
    nout = _classes(case)
    return dict(kind="classifier", x=inp["X"], layers=inp["layers"], M=M, B=B, S=S, heads=case["heads"], mask=mask, nout=nout,
                head_w=normal(case["hidden"] * sum(nout), std=0.02, dtype=dt), head_b=normal(sum(nout), std=0.02))


def _classify(s):
    x, M, B, S = s["x"], s["M"], s["B"], s["S"]
    for L in s["layers"]:
        qkv = nf.linear(x, L["Wqkv"], bias=L["bqkv"])
        att = nf.attention_packed(qkv, B, S, s["heads"], mask=s["mask"])
        h = nf.linear(att, L["Wo"], bias=L["bo"], residual=x)
        x1 = nf.layernorm(h, L["ln1_g"], L["ln1_b"], M)
        f1 = nf.linear(x1, L["W1"], bias=L["b1"], act=nf.ACT_GELU)
        f2 = nf.linear(f1, L["W2"], bias=L["b2"], residual=x1)
        x = nf.layernorm(f2, L["ln2_g"], L["ln2_b"], M)
    first = x.view(M, B, S, -1)[:, :, 0].contiguous()          # each sequence's first token goes to its model's output layer
    return dict(hidden=x, logits=nf.linear_ragged(first, s["head_w"], s["nout"], bias=s["head_b"]))


def run(state):
    if state["kind"] == "classifier":
        return _classify(state)
    if state["kind"] == "layer":
        return state["net"].forward()
    return state["net"].forward(state["x"])


def work(case):
    """Weights, inputs and final outputs once each (activations between the operators could stay on the chip);
    the multiplications and additions of the matrix products, convolutions and attention scores."""
    e, M = 2 if case["dtype"] == "bf16" else 4, case["M"]
    if case["kind"] == "layer":
        r, k, n, c, px = case["rows"], case["features"], case["outputs"], case["channels"], case["image"] ** 2
        # the matmul's output is returned beside the normalised one
        return dict(bytes=M * (e * (r * k + k * n + 2 * r * n + 9 * c * c + 2 * c * px) + 12 * n),
                    flops=2 * M * (r * k * n + 9 * c * c * px))
    if case["kind"] == "resnet":
        spec = NI.resnet_spec(case["cardinality"], case["base_width"], case["image"])
        B, wts, fl, vec = case["batch"], 0, 0, 0

        def conv(c, hw):
            nonlocal wts, fl, vec
            out = nf.conv_out_size(hw, c.k, c.stride, c.pad)
            n = c.cout * (c.cin // c.groups) * c.k * c.k
            wts, fl, vec = wts + n, fl + 2 * B * n * out * out, vec + 8 * c.cout
            return out
        hw = (conv(spec.stem, spec.image) - 1) // 2 + 1
        for b in spec.blocks:
            conv(b.conv1, hw)
            out = conv(b.conv2, hw)
            conv(b.conv3, out)
            if b.down is not None:
                conv(b.down, hw)
            hw = out
        return dict(bytes=M * (e * (wts + B * (3 * spec.image ** 2 + spec.out_channels)) + vec), flops=M * fl)
    H, F, L, S, N = case["hidden"], case["ffn"], case["layers"], case["seq"], case["batch"] * case["seq"]
    mats = 4 * H * H + 2 * H * F
    rel = case.get("rel", False)
    by = e * (L * (mats + rel * H * H) + 2 * N * H + rel * 2 * S * H) + 4 * L * (9 * H + F + rel * 2 * H)
    fl = L * (2 * N * mats + 4 * N * S * H + rel * (4 * S * H * H + 2 * N * S * H))
    if case["kind"] == "classifier":
        c = sum(_classes(case)) / M
        by, fl = by + e * (H * c + case["batch"] * c) + 4 * N + 4 * c, fl + 2 * case["batch"] * H * c
    return dict(bytes=M * by, flops=M * fl)


def tolerance(case):
    """Measured.  bfloat16 encoders: one run against the same weights in float32 storage is off by 3.4e-3 after one
    layer, 8e-3 after 6, 1.15e-2 after 12 (largest element 1.6e-2 and 7e-2), another order of the sums by 9e-3 after 12 (a last-bit
    difference flips roundings of activations, and those spread); 2.5 times that.  Image networks average over
    positions at the end: 2e-3, largest element 6e-3; four times that.  float32 against float64: 1.4e-6 and 7e-6."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 4e-5}
    if case["kind"] == "resnet":
        return {"rel": 8e-3, "max": 2.5e-2}
    deep = case.get("layers", 1) ** 0.5
    return {"rel": round(8.5e-3 * deep, 5), "max": round(8e-2 * deep, 4)}
