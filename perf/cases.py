"""The work a user of this library has it do, as cases to be measured.

Whole calls: an elastic ViT answering one image or a full batch in a chosen
mode, an elastic ResNet, and a run of growth steps up to its checkpoint.  The
rest are the single layers behind the library's public entry points (linear,
attention, LayerNorm, convolution), with the shapes those models give them.

``listed()`` names the cases; ``draw(rng)`` gives one more of the same ranges.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2609_10018_amd import ffi, inputs, inputs_cnn

DEV = "cuda"
BF, F32 = torch.bfloat16, torch.float32
EPI = {"bias": ffi.EPI_BIAS, "gelu": ffi.EPI_BIAS_GELU, "resid": ffi.EPI_BIAS_RESID,
       "f32out": ffi.EPI_BIAS_F32OUT}
T224 = 197                       # tokens of a 224x224 image in 16x16 patches, with the class token


def listed():
    return [
        # One image through ViT-B in a half-width mode, the mode set before the call: the
        # serving latency that a mode switch is there for.
        {"name": "vit_b_serve_one", "op": "vit", "model": "vit_b", "dtype": "bf16", "mode": 2,
         "batch": 1},
        # A full batch through the full-width ViT-B: throughput.
        {"name": "vit_b_batch", "op": "vit", "model": "vit_b", "dtype": "bf16", "mode": 0,
         "batch": 256},
        # A full batch through the elastic ResNet-50 in its middle mode.
        {"name": "resnet50_batch", "op": "resnet", "model": "resnet50", "mode": 2, "batch": 256},
        # A stretch of training (mode 0 grown from mode 1) up to the checkpoint that is read
        # back: forward, backward, clipping and update.
        {"name": "growth_vit_b", "op": "growth", "model": "vit_b", "mode": 0, "batch": 64,
         "steps": 24},
        # The classifier on a small batch.
        {"name": "head_small", "op": "linear", "dtype": "bf16", "epi": "f32out", "M": 8, "N": 1000,
         "K": 768, "lda": 768},
        # The first MLP layer of ViT-B on a full batch.
        {"name": "fc1_batch", "op": "linear", "dtype": "bf16", "epi": "gelu", "M": 256 * T224,
         "N": 3072, "K": 768, "lda": 768},
        # The second MLP layer of a ViT-S mode with an odd number of active units, read as a
        # prefix of the full-width rows, added to the residual stream.
        {"name": "fc2_ragged", "op": "linear", "dtype": "bf16", "epi": "resid", "M": 37 * T224,
         "N": 384, "K": 691, "lda": 1536},
        # The q/k/v projection of ViT-S in fp32.
        {"name": "qkv_fp32", "op": "linear", "dtype": "fp32", "epi": "bias", "M": 32 * T224,
         "N": 1152, "K": 384, "lda": 384},
        # Attention of the full-width ViT-B, and of an fp32 ViT-S.
        {"name": "attn_batch", "op": "attention", "dtype": "bf16", "batch": 256, "tokens": T224,
         "heads": 12, "dim": 64},
        {"name": "attn_fp32", "op": "attention", "dtype": "fp32", "batch": 16, "tokens": T224,
         "heads": 6, "dim": 64},
        # LayerNorm of a full batch's residual stream with its fp32 class-token rows.
        {"name": "norm_batch", "op": "norm", "dtype": "bf16", "rows": 256 * T224, "d": 768,
         "cls": True},
        # A 3x3 convolution of a ResNet-50 bottleneck with pruned filters.
        {"name": "conv3x3", "op": "conv", "batch": 64, "hw": 28, "cs": 128, "ca": 88, "n": 88,
         "k": 3, "stride": 1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["vit", "vit", "resnet", "growth", "linear", "linear", "linear", "attention",
                     "attention", "norm", "conv"])
    if op == "vit":
        model = rng.choice(["tiny", "tiny_emb", "vit_ti", "vit_s", "vit_b", "vit_ti_emb",
                            "vit_b_emb"])
        tiny = model.startswith("tiny")
        dtype = "fp32" if tiny or (model == "vit_ti" and rng.random() < 0.5) else "bf16"
        return {"op": op, "model": model, "dtype": dtype,
                "mode": rng.randrange(len(inputs.MODE_CAPS[model])),
                "batch": _log(rng, 1, 32 if dtype == "fp32" else 200)}
    if op == "resnet":
        model = rng.choice(["resnet50", "resnet50", "resnet_small"])
        return {"op": op, "model": model,
                "mode": rng.randrange(len(inputs_cnn.CNN_MODE_RATIOS[model])),
                "batch": _log(rng, 1, 200)}
    if op == "growth":
        model = rng.choice(["vit_ti", "vit_s", "vit_b"])
        return {"op": op, "model": model, "mode": rng.randrange(len(inputs.MODE_CAPS[model]) - 1),
                "batch": _log(rng, 2, 48), "steps": rng.randint(4, 16)}
    if op == "linear":
        dtype = rng.choice(["bf16", "bf16", "fp32"])
        epi = rng.choice(list(EPI))
        n, k = _log(rng, 24, 3072), _log(rng, 24, 3072)
        if rng.random() < 0.6:                       # the widths of whole models
            n, k = max(64, n // 64 * 64), max(64, k // 64 * 64)
        lda = (k + 7) // 8 * 8 + rng.choice([0, 0, 64, 8 * rng.randint(1, 40)])
        return {"op": op, "dtype": dtype, "epi": epi,
                "M": _log(rng, 1, 50000 if dtype == "bf16" else 8000), "N": n, "K": k, "lda": lda}
    if op == "attention":
        dtype = rng.choice(["bf16", "bf16", "fp32"])
        bf = dtype == "bf16"
        return {"op": op, "dtype": dtype, "batch": _log(rng, 1, 250 if bf else 16),
                "tokens": rng.choice([T224, rng.randint(2, 240)]),
                "heads": rng.randint(1, 12 if bf else 6),
                "dim": 64 if bf else rng.choice([32, 64, 64, rng.randint(8, 128)])}
    if op == "norm":
        dtype = rng.choice(["bf16", "fp32"])
        bf = dtype == "bf16"
        return {"op": op, "dtype": dtype, "rows": _log(rng, 1, 50000),
                "d": 8 * _log(rng, 8, 256) if bf else _log(rng, 24, 2048),
                "cls": bf and rng.random() < 0.5}
    ca = 8 * _log(rng, 1, 32)
    cs, n = ca + 8 * rng.choice([0, rng.randint(0, 8)]), 8 * _log(rng, 1, 64)
    return {"op": op, "batch": _log(rng, 1, 64), "hw": rng.choice([7, 14, 28, 56]), "cs": cs,
            "ca": ca, "n": n, "k": rng.choice([1, 3, 3]), "stride": rng.choice([1, 1, 2])}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, *shape, dtype=F32, std=1.0):
    return (torch.randn(*shape, generator=g, device=DEV) * std).to(dtype)


def _vit_cfg(case):
    return dataclasses.replace(inputs.CONFIGS[case["model"]],
                               dtype=inputs.FP32 if case.get("dtype") == "fp32" else inputs.BF16)


def _vit_parts(cfg, seed):
    """Random weights (as inputs.make_weights describes them) and a DN table of the
    config's widths with random channel orders."""
    g, w = _gen(seed), {}
    for key, shape in inputs.param_shapes(cfg).items():
        w[key] = _randn(g, *shape, std=inputs.INIT_STD) + (1.0 if key.endswith("_g") else 0.0)
    r = np.random.default_rng(seed)
    caps, L = inputs.MODE_CAPS[cfg.name], cfg.depth
    ratio = inputs.layer_ratios(cfg) if cfg.name in inputs.LAYER_RATIO_CONFIGS else np.ones(L)
    wide = lambda c, k: [c if k == 0 else max(1, int(np.floor(c * x + 0.5))) for x in ratio]  # noqa: E731
    table = inputs.DNTable(
        np.array([wide(c[0], k) for k, c in enumerate(caps)], dtype=np.int32),
        np.array([wide(c[1], k) for k, c in enumerate(caps)], dtype=np.int32),
        np.stack([r.permutation(cfg.heads) for _ in range(L)]).astype(np.int32),
        np.stack([r.permutation(cfg.mlp_hidden) for _ in range(L)]).astype(np.int32),
        np.array([c[2] if len(c) > 2 else cfg.dim for c in caps], dtype=np.int32),
        r.permutation(cfg.dim).astype(np.int32) if len(caps[0]) > 2
        else np.arange(cfg.dim, dtype=np.int32))
    return w, table


def _vit_images(cfg, batch, seed):
    return _randn(_gen(seed + 1), batch, cfg.in_chans, cfg.img, cfg.img,
                  dtype=F32 if cfg.dtype == inputs.FP32 else BF)


def _host(w):
    return {k: v.cpu().numpy() for k, v in w.items()}


def _cnn_parts(cfg, seed):
    """Random filters (as inputs_cnn.make_cnn_weights describes them) and a DN table of the
    config's widths with random filter orders."""
    g, w = _gen(seed), {}
    for key, shape in inputs_cnn.conv_shapes(cfg).items():
        std = 0.02 if key.endswith("_b") or key == "fc_w" else math.sqrt(2.0 / math.prod(shape[1:]))
        if key.endswith("_c3_w"):
            std *= inputs_cnn.RESIDUAL_BRANCH_GAIN
        w[key] = _randn(g, *shape, std=std)
    specs, r = cfg.block_specs(), np.random.default_rng(seed)
    keep = lambda width, x: min(width, max(8, int(np.floor(width * x / 8.0 + 0.5)) * 8))  # noqa: E731
    ratios = inputs_cnn.CNN_MODE_RATIOS[cfg.name]
    n = np.array([[keep(b["width"], x) for b in specs] for x in ratios], dtype=np.int32)
    order = lambda: [r.permutation(b["width"]).astype(np.int32) for b in specs]  # noqa: E731
    return w, inputs_cnn.CNNTable(n, order(), order())


def _cnn_images(cfg, batch, seed):
    """Like normalised photographs, images differ in channel means and contrast."""
    g = _gen(seed + 1)
    x = torch.randn(batch, cfg.in_chans, cfg.img, cfg.img, generator=g, device=DEV)
    contrast = 0.25 + 1.75 * torch.rand(batch, 1, 1, 1, generator=g, device=DEV)
    return (torch.randn(batch, cfg.in_chans, 1, 1, generator=g, device=DEV) + contrast * x).to(BF)


def _growth_data(case, cfg, seed):
    g, b, n = _gen(seed + 1), case["batch"], case["steps"]
    images = torch.randn(n, b, cfg.in_chans, cfg.img, cfg.img, generator=g, device=DEV).to(BF)
    labels = torch.randint(0, cfg.num_classes, (n, b), generator=g, device=DEV, dtype=torch.int32)
    return images, labels


GROWTH_LR, GROWTH_CLIP = 0.02, 1.0


def _linear_data(case, seed):
    g, dt = _gen(seed), F32 if case["dtype"] == "fp32" else BF
    M, N, K, lda = case["M"], case["N"], case["K"], case["lda"]
    ldc = (N + 7) // 8 * 8
    A, W = _randn(g, M, lda, dtype=dt), _randn(g, N, lda, dtype=dt, std=0.02)
    bias = _randn(g, N, std=0.02)
    out = F32 if case["epi"] == "f32out" else dt
    C = _randn(g, M, ldc, dtype=out) if case["epi"] == "resid" else torch.empty(M, ldc, device=DEV,
                                                                              dtype=out)
    return A, W, bias, C


def _attention_data(case, seed):
    dt = F32 if case["dtype"] == "fp32" else BF
    rows, width = case["batch"] * case["tokens"], case["heads"] * case["dim"]
    return _randn(_gen(seed), rows, 3 * width, dtype=dt), torch.empty(rows, width, device=DEV,
                                                                      dtype=dt)


def _norm_data(case, seed):
    g, dt = _gen(seed), F32 if case["dtype"] == "fp32" else BF
    rows, d = case["rows"], case["d"]
    x = _randn(g, rows, d) * (0.5 + torch.rand(rows, 1, generator=g, device=DEV))
    cls = _randn(g, (rows + T224 - 1) // T224, d) if case["cls"] else None
    return {"x": x.to(dt), "cls": cls, "g": 1.0 + _randn(g, d, std=0.02), "b": _randn(g, d, std=0.02),
            "out": torch.empty(rows, d, device=DEV, dtype=dt)}


def _conv_data(case, seed):
    g, k, hw = _gen(seed), case["k"], case["hw"]
    x = torch.relu(_randn(g, case["batch"], hw, hw, case["cs"])).to(BF)
    w = _randn(g, case["n"], k * k, case["cs"], dtype=BF, std=math.sqrt(2.0 / (k * k * case["ca"])))
    ho = (hw + 2 * (k // 2) - k) // case["stride"] + 1
    return x, w, _randn(g, case["n"], std=0.02), torch.empty(case["batch"], ho, ho, case["n"],
                                                             device=DEV, dtype=BF)


def prepare(case, seed):
    op = case["op"]
    s = {"case": case}
    if op in ("vit", "growth"):
        cfg = _vit_cfg(case)
        w, table = _vit_parts(cfg, seed)
        s["net"] = ffi.ElasticViT(cfg, _host(w), table, case["batch"])
        if op == "vit":
            s["images"] = _vit_images(cfg, case["batch"], seed)
            s["logits"] = torch.empty(case["batch"], cfg.num_classes, device=DEV)
        else:
            s["net"].set_mode(case["mode"])
            s["grow"] = ffi.GrowthContext(s["net"], case["batch"])
            s["images"], s["labels"] = _growth_data(case, cfg, seed)
            s["stats"] = torch.empty(case["steps"], 3, device=DEV)
            s["layout"] = [{t: ffi.packed_layout(cfg, t, l)[:3]
                            for t in (ffi.T_WQKV, ffi.T_WO, ffi.T_W1, ffi.T_W2, ffi.T_BQKV, ffi.T_B1)}
                           for l in range(cfg.depth)]
    elif op == "resnet":
        cfg = inputs_cnn.CNN_CONFIGS[case["model"]]
        w, table = _cnn_parts(cfg, seed)
        s["net"] = ffi.ElasticResNet(cfg, _host(w), table, case["batch"])
        s["images"] = _cnn_images(cfg, case["batch"], seed)
        s["logits"] = torch.empty(case["batch"], cfg.num_classes, device=DEV)
    elif op == "linear":
        s["A"], s["W"], s["bias"], s["C"] = _linear_data(case, seed)
    elif op == "attention":
        s["qkv"], s["o"] = _attention_data(case, seed)
    elif op == "norm":
        s.update(_norm_data(case, seed))
    else:
        s["x"], s["w"], s["b"], s["y"] = _conv_data(case, seed)
    return s


# --------------------------------------------------------------------- run
def _dtype(case):
    return ffi.FP32 if case["dtype"] == "fp32" else ffi.BF16


def run(s):
    case = s["case"]
    op = case["op"]
    if op in ("vit", "resnet"):
        s["net"].set_mode(case["mode"])
        s["net"].forward(s["images"], s["logits"])
        return s["logits"]
    if op == "growth":
        for i in range(case["steps"]):
            s["grow"].step(case["mode"], s["images"][i], s["labels"][i], GROWTH_LR, GROWTH_CLIP,
                           s["stats"][i])
        # The checkpoint: fp32 master matrices and the fp32 bias vectors of the packed image.
        master, packed = s["grow"].read(1), s["grow"].read(0)
        out = {"stats": s["stats"]}
        for t, name in ((ffi.T_WQKV, "wqkv"), (ffi.T_WO, "wo"), (ffi.T_W1, "w1"), (ffi.T_W2, "w2")):
            out[name] = [master[l[t][0] // 2:l[t][0] // 2 + l[t][1] * l[t][2]].reshape(l[t][1], l[t][2])
                         for l in s["layout"]]
        for t, name in ((ffi.T_BQKV, "bqkv"), (ffi.T_B1, "b1")):
            out[name] = np.stack([packed[l[t][0]:l[t][0] + 4 * l[t][1] * l[t][2]].view(np.float32)
                                  for l in s["layout"]])
        return out
    if op == "linear":
        ffi.op_linear(_dtype(case), EPI[case["epi"]], s["A"], case["lda"], s["W"], case["lda"],
                      s["C"], s["C"].shape[1], s["bias"], case["M"], case["N"], case["K"])
        return s["C"][:, :case["N"]]
    if op == "attention":
        width = case["heads"] * case["dim"]
        ffi.op_attention(_dtype(case), s["qkv"], 3 * width, s["o"], width, case["batch"],
                         case["tokens"], case["heads"], case["dim"], 1.0 / math.sqrt(case["dim"]))
        return s["o"]
    if op == "norm":
        ffi.op_layernorm(_dtype(case), s["x"], case["d"], s["out"], case["rows"], case["d"], s["g"],
                         s["b"], 1e-6, x_cls=s["cls"], tokens=T224)
        return s["out"]
    k, hw = case["k"], case["hw"]
    ffi.op_conv2d(s["x"], case["batch"], hw, hw, case["cs"], case["ca"], k, k, case["stride"], k // 2,
                  s["w"], k * k * case["cs"], case["cs"], s["b"], s["y"], case["n"], case["n"],
                  relu=True)
    return s["y"]


# -------------------------------------------------------------------- work
def _vit_work(case, train=False):
    cfg = _vit_cfg(case)
    caps, k, L = inputs.MODE_CAPS[cfg.name], case["mode"], cfg.depth
    eb = 4 if cfg.dtype == inputs.FP32 else 2
    ratio = inputs.layer_ratios(cfg) if cfg.name in inputs.LAYER_RATIO_CONFIGS and k else np.ones(L)
    e = caps[k][2] if len(caps[k]) > 2 else cfg.dim
    h = np.maximum(1, np.floor(caps[k][0] * ratio + 0.5)) * cfg.head_dim
    m = np.maximum(1, np.floor(caps[k][1] * ratio + 0.5))
    params = float((4 * h * e + 2 * m * e).sum()) + e * cfg.patch_k + e * cfg.num_classes
    T = cfg.tokens
    flops = 2.0 * T * float((4 * h * e + 2 * m * e).sum()) + 4.0 * T * T * float(h.sum())
    flops += 2.0 * cfg.num_patches * e * cfg.patch_k + 2.0 * e * cfg.num_classes
    B = case["batch"]
    image = cfg.in_chans * cfg.img * cfg.img * eb
    if not train:
        return {"bytes": params * eb + B * (image + 4.0 * cfg.num_classes), "flops": B * flops}
    # A step: the forward, the activation gradients, and the gradients of the slices grown.
    ratio2 = inputs.layer_ratios(cfg) if cfg.name in inputs.LAYER_RATIO_CONFIGS else np.ones(L)
    h2 = np.maximum(1, np.floor(caps[k + 1][0] * ratio2 + 0.5)) * cfg.head_dim
    m2 = np.maximum(1, np.floor(caps[k + 1][1] * ratio2 + 0.5))
    grown = float((4 * (h - h2) * e + 2 * (m - m2) * e).sum())
    step = B * (2.0 * flops + 4.0 * T * T * float(h.sum()) + 2.0 * T * grown)
    whole = 6.0 * sum(math.prod(s) for s in inputs.param_shapes(cfg).values())
    return {"bytes": case["steps"] * (params * eb + 10.0 * grown + B * image) + whole,
            "flops": case["steps"] * step}


def _cnn_work(case):
    cfg = inputs_cnn.CNN_CONFIGS[case["model"]]
    x = inputs_cnn.CNN_MODE_RATIOS[cfg.name][case["mode"]]
    hs = cfg.img // 2
    macs, params = hs * hs * cfg.stem * cfg.in_chans * 49.0, cfg.stem * cfg.in_chans * 49.0
    for b in cfg.block_specs():
        n = min(b["width"], max(8, int(np.floor(b["width"] * x / 8.0 + 0.5)) * 8))
        hi, ho = b["hw_in"] ** 2, (b["hw_in"] // b["stride"]) ** 2
        dn = b["c_in"] * b["c_out"] if b["down"] else 0
        macs += hi * n * b["c_in"] + ho * (9 * n * n + n * b["c_out"] + dn)
        params += n * b["c_in"] + 9 * n * n + n * b["c_out"] + dn
    params += cfg.features * cfg.num_classes
    macs += cfg.features * cfg.num_classes
    B = case["batch"]
    return {"bytes": 2.0 * params + B * (2.0 * cfg.in_chans * cfg.img ** 2 + 4.0 * cfg.num_classes),
            "flops": 2.0 * B * macs}


def work(case):
    op = case["op"]
    if op == "vit":
        return _vit_work(case)
    if op == "growth":
        return _vit_work(case, train=True)
    if op == "resnet":
        return _cnn_work(case)
    eb = 4.0 if case.get("dtype") == "fp32" else 2.0
    if op == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        out = 4.0 if case["epi"] == "f32out" else eb * (2 if case["epi"] == "resid" else 1)
        return {"bytes": eb * (M * K + N * K) + out * M * N + 4.0 * N, "flops": 2.0 * M * N * K}
    if op == "attention":
        B, T, w = case["batch"], case["tokens"], case["heads"] * case["dim"]
        return {"bytes": 4.0 * B * T * w * eb, "flops": 4.0 * B * T * T * w}
    if op == "norm":
        return {"bytes": 2.0 * case["rows"] * case["d"] * eb, "flops": 8.0 * case["rows"] * case["d"]}
    k, hw, B = case["k"], case["hw"], case["batch"]
    ho = (hw + 2 * (k // 2) - k) // case["stride"] + 1
    return {"bytes": 2.0 * (B * hw * hw * case["ca"] + case["n"] * k * k * case["ca"]
                            + B * ho * ho * case["n"]),
            "flops": 2.0 * B * ho * ho * case["n"] * k * k * case["ca"]}


def tolerance(case):
    """About four times the difference from exact() that was seen, by data type and depth."""
    op = case["op"]
    if op == "growth":       # seen: 5e-4 in the loss and the gradient's norm, 2e-5 in the weights
        return {"rel": 4e-3, "max": 2e-2}
    if op == "resnet":       # 2e-3
        return {"rel": 1e-2, "max": 8e-2}
    if op == "vit":          # 6e-3 in bf16
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "fp32" else {"rel": 2.4e-2, "max": 0.2}
    if case.get("dtype") == "fp32" or case.get("epi") == "f32out":   # 4e-7
        return {"rel": 2e-6, "max": 4e-5}
    return {"rel": 8e-3, "max": 4e-2}                                # 2e-3: the rounding to bf16


# ------------------------------------------------------------------- exact
def _ln64(x, g, b, eps=1e-6):
    m = x.mean(-1, keepdim=True)
    v = ((x - m) ** 2).mean(-1, keepdim=True)
    return (x - m) / torch.sqrt(v + eps) * g + b


def _gelu64(z):
    return 0.5 * z * (1.0 + torch.erf(z * math.sqrt(0.5)))


def _attend64(qkv, h, hd):
    """qkv [B, T, h * 3 * hd], each head's q, k and v side by side."""
    B, T = qkv.shape[:2]
    q, k, v = qkv.reshape(B, T, h, 3, hd).permute(3, 0, 2, 1, 4).contiguous().unbind(0)
    p = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(hd), dim=-1)
    return torch.matmul(p, v).permute(0, 2, 1, 3).reshape(B, T, h * hd)


def _packed64(cfg, w, table, rounded):
    """The weights in 64 bits, every channel in the order in which the modes take it in."""
    d, hd = cfg.dim, cfg.head_dim
    emb = torch.as_tensor(table.embed_order, device=DEV, dtype=torch.long)
    r = {k: (v.to(BF) if rounded and k in inputs.MATRIX_KEYS else v).double() for k, v in w.items()}
    p = {k: r[k][emb] for k in ("patch_b", "cls", "norm_g", "norm_b")}
    p.update(patch_w=r["patch_w"].reshape(d, -1)[emb], pos=r["pos"][:, emb],
             head_w=r["head_w"][:, emb], head_b=r["head_b"], layers=[])
    for l in range(cfg.depth):
        ho = torch.as_tensor(table.head_order[l], device=DEV, dtype=torch.long)
        mo = torch.as_tensor(table.mlp_order[l], device=DEV, dtype=torch.long)
        c = torch.arange(hd, device=DEV)
        rows = (torch.arange(3, device=DEV)[None, :, None] * d + ho[:, None, None] * hd + c).reshape(-1)
        cols = (ho[:, None] * hd + c).reshape(-1)
        q = {k: r[k][l][emb] for k in ("ln1_g", "ln1_b", "ln2_g", "ln2_b", "proj_b", "fc2_b")}
        q.update(wqkv=r["qkv_w"][l][rows][:, emb], bqkv=r["qkv_b"][l][rows],
                 wo=r["proj_w"][l][emb][:, cols], w1=r["fc1_w"][l][mo][:, emb], b1=r["fc1_b"][l][mo],
                 w2=r["fc2_w"][l][emb][:, mo])
        p["layers"].append(q)
    return p


def _vit64(cfg, p, table, k, x):
    """Logits of mode k: every matrix of p cut to the prefix that the mode keeps."""
    e, hd, P, G = int(table.n_embed[k]), cfg.head_dim, cfg.patch, cfg.grid
    B = x.shape[0]
    x = x.double().reshape(B, cfg.in_chans, G, P, G, P).permute(0, 2, 4, 1, 3, 5).reshape(B, G * G, -1)
    x = torch.matmul(x, p["patch_w"][:e].t()) + p["patch_b"][:e]
    x = torch.cat([p["cls"][:e].expand(B, 1, e), x], 1) + p["pos"][:, :e]
    for l, q in enumerate(p["layers"]):
        h, m = int(table.n_heads[k][l]), int(table.n_mlp[k][l])
        u = _ln64(x, q["ln1_g"][:e], q["ln1_b"][:e])
        qkv = torch.matmul(u, q["wqkv"][:3 * hd * h, :e].t()) + q["bqkv"][:3 * hd * h]
        o = _attend64(qkv, h, hd)
        x = x + torch.matmul(o, q["wo"][:e, :hd * h].t()) + q["proj_b"][:e]
        u = _ln64(x, q["ln2_g"][:e], q["ln2_b"][:e])
        u = _gelu64(torch.matmul(u, q["w1"][:m, :e].t()) + q["b1"][:m])
        x = x + torch.matmul(u, q["w2"][:e, :m].t()) + q["fc2_b"][:e]
    return torch.matmul(_ln64(x[:, 0], p["norm_g"][:e], p["norm_b"][:e]), p["head_w"][:, :e].t()) + p["head_b"]


def _growth64(case, seed):
    cfg = _vit_cfg(case)
    w, table = _vit_parts(cfg, seed)
    images, labels = _growth_data(case, cfg, seed)
    k, hd = case["mode"], cfg.head_dim
    p = _packed64(cfg, w, table, True)
    stats = []
    names = ("wqkv", "bqkv", "wo", "w1", "b1", "w2")
    master = [{n: q[n] for n in names} for q in p["layers"]]
    for i in range(case["steps"]):
        for q, a in zip(p["layers"], master):
            for n in names:                          # matrices are used in bf16
                t = a[n].to(F32).to(BF).double() if n[0] == "w" else a[n].clone()
                q[n] = t.requires_grad_()
        logits = _vit64(cfg, p, table, k, images[i])
        loss = F.cross_entropy(logits, labels[i].long())
        loss.backward()
        grads = []
        for l, q in enumerate(p["layers"]):
            h, m = int(table.n_heads[k + 1][l]), int(table.n_mlp[k + 1][l])
            g = {n: q[n].grad for n in names}
            for n, cut in (("wqkv", 3 * hd * h), ("bqkv", 3 * hd * h), ("w1", m), ("b1", m)):
                g[n][:cut] = 0                       # shared with the smaller mode: frozen
            g["wo"][:, :hd * h] = 0
            g["w2"][:, :m] = 0
            grads.append(g)
        norm = math.sqrt(sum(float((t * t).sum()) for g in grads for t in g.values()))
        f = GROWTH_CLIP / norm if norm > GROWTH_CLIP else 1.0
        stats.append([float(loss), norm, f])
        master = [{n: a[n] - GROWTH_LR * f * g[n] for n in names} for a, g in zip(master, grads)]
    out = {n: [a[n] for a in master] for n in ("wqkv", "wo", "w1", "w2")}
    out.update({n: torch.stack([a[n] for a in master]) for n in ("bqkv", "b1")})
    out["stats"] = torch.tensor(stats, dtype=torch.float64)
    return out


def _conv64(x, w, b, stride, pad):
    n, k = w.shape[0], w.shape[2]
    ho = (x.shape[2] + 2 * pad - k) // stride + 1
    y = torch.matmul(w.reshape(n, -1), F.unfold(x, k, padding=pad, stride=stride))
    return y.reshape(x.shape[0], n, ho, ho) + b[:, None, None]


def _cnn64(case, seed):
    cfg = inputs_cnn.CNN_CONFIGS[case["model"]]
    w, table = _cnn_parts(cfg, seed)
    images = _cnn_images(cfg, case["batch"], seed)
    r = {k: (v.to(BF) if k.endswith("_w") else v).double() for k, v in w.items()}
    out = []
    for x in images.split(16):
        x = torch.relu(_conv64(x.double(), r["stem_w"], r["stem_b"], 2, 3))
        x = F.max_pool2d(x, 3, 2, 1)
        for i, spec in enumerate(cfg.block_specs()):
            n = int(table.n_width[case["mode"]][i])
            a = torch.as_tensor(table.order1[i][:n], device=DEV, dtype=torch.long)
            c = torch.as_tensor(table.order2[i][:n], device=DEV, dtype=torch.long)
            get = lambda s: (r[f"b{i}_{s}_w"], r[f"b{i}_{s}_b"])  # noqa: E731
            (w1, b1), (w2, b2), (w3, b3) = get("c1"), get("c2"), get("c3")
            y = torch.relu(_conv64(x, w1[a], b1[a], 1, 0))
            y = torch.relu(_conv64(y, w2[c][:, a], b2[c], spec["stride"], 1))
            y = _conv64(y, w3[:, c], b3, 1, 0)
            x = torch.relu(y + (_conv64(x, *get("dn"), spec["stride"], 0) if spec["down"] else x))
        out.append(torch.matmul(x.mean((2, 3)), r["fc_w"].t()) + r["fc_b"])
    return torch.cat(out)


def exact(case, seed):
    op = case["op"]
    if op == "vit":
        cfg = _vit_cfg(case)
        w, table = _vit_parts(cfg, seed)
        p = _packed64(cfg, w, table, cfg.dtype == inputs.BF16)
        return torch.cat([_vit64(cfg, p, table, case["mode"], x)
                          for x in _vit_images(cfg, case["batch"], seed).split(64)])
    if op == "growth":
        return _growth64(case, seed)
    if op == "resnet":
        return _cnn64(case, seed)
    if op == "linear":
        A, W, bias, C = _linear_data(case, seed)
        K, N = case["K"], case["N"]
        y = torch.matmul(A[:, :K].double(), W[:, :K].double().t()) + bias.double()
        if case["epi"] == "gelu":
            y = _gelu64(y)
        return y + C[:, :N].double() if case["epi"] == "resid" else y
    if op == "attention":
        qkv, _ = _attention_data(case, seed)
        B, T, w = case["batch"], case["tokens"], case["heads"] * case["dim"]
        return torch.cat([_attend64(x.double(), case["heads"], case["dim"]).reshape(-1, w)
                          for x in qkv.reshape(B, T, 3 * w).split(64)])
    if op == "norm":
        s = _norm_data(case, seed)
        x = s["x"].double()
        if s["cls"] is not None:
            x[::T224] = s["cls"].double()
        return _ln64(x, s["g"].double(), s["b"].double())
    x, w, b, _ = _conv_data(case, seed)
    k, ca = case["k"], case["ca"]
    w = w[..., :ca].double().transpose(1, 2).reshape(case["n"], ca, k, k)
    out = [torch.relu(_conv64(t[..., :ca].double().permute(0, 3, 1, 2), w, b.double(), case["stride"],
                              k // 2)).permute(0, 2, 3, 1) for t in x.split(16)]
    return torch.cat(out).contiguous()
