"""The calls whose time this library is judged by: what a program that uses it has it do, from the smallest call to the largest.

A case names an entry point ("call"), the element type and the shape.  "groups" holds the nominal group size of every
aggregation level, first level first; "linear" makes the first level a linear one (D-CHAG-L).

  call            entry points                                 who makes it
  forward         dchag_forward                                inference on the layer as the paper defines it
  forward_pos     dchag_forward_pos                            the same with the positional embedding added
  folded          dchag_forward_folded                         inference while weights still change between calls
  prefolded       dchag_forward_prefolded                      serving: weights fixed, prepared once by dchag_fold_value
  train           dchag_forward_keep + dchag_backward_kept     a training step: output and every gradient
  level           dchag_aggregate_level                        one rank's share of the channels, tokens already there
"""
from __future__ import annotations

import math

import torch

import paper_2506_21411_amd as dchag


def _case(name, call, dtype, B, C, H, W, p, D, heads, groups, x="iid", linear=False):
    c = {"call": call, "dtype": dtype, "B": B, "C": C, "H": H, "W": W, "p": p, "D": D, "heads": heads, "groups": groups,
         "x": x, "linear": linear}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a unit test's or a notebook's call: almost nothing to compute, so launches and host work decide
        _case("tiny_f32_forward", "forward", "f32", 1, 8, 32, 64, 4, 128, 4, "4,2"),
        # one regional crop of weather fields answered by a small model: the smallest call of a serving process
        _case("crop_bf16_prefolded", "prefolded", "bf16", 1, 80, 32, 64, 4, 256, 8, "8,10", "fields"),
        # one of eight ranks' share of 512 bands: two groups of 32 whose tokens the rank has made already
        _case("shard_bf16_level", "level", "bf16", 4, 64, 128, 128, 8, 1024, 16, "32"),
        # training on 80 weather variables, 4 x 4 patches: many patches, small groups
        _case("weather_bf16_train", "train", "bf16", 2, 80, 128, 256, 4, 1024, 16, "8,10", "fields"),
        # 512 hyperspectral bands, the benchmark's headline shape
        _case("bands_bf16_forward", "forward", "bf16", 4, 512, 128, 128, 8, 1024, 16, "32,16", "bands"),
        # the same images answered by a serving process whose weights are fixed
        _case("bands_bf16_prefolded", "prefolded", "bf16", 4, 512, 128, 128, 8, 1024, 16, "32,16", "bands"),
        # the same shape, one training step
        _case("bands_bf16_train", "train", "bf16", 4, 512, 128, 128, 8, 1024, 16, "32,16", "bands"),
        # the same shape with linear first-level layers (D-CHAG-L), one training step
        _case("bands_linear_bf16_train", "train", "bf16", 4, 512, 128, 128, 8, 1024, 16, "32,16", "bands", True),
        # three levels over a channel count that no group size divides, weights changing between calls
        _case("deep_bf16_folded", "folded", "bf16", 2, 1000, 128, 128, 8, 2048, 16, "16,8,8", "bands"),
        # the widest embedding over a large grid: the largest call
        _case("wide_bf16_forward_pos", "forward_pos", "bf16", 1, 256, 256, 512, 8, 4096, 32, "32,8"),
        # single precision in earnest: a training step of a mid-sized weather model, as one debugs or validates it
        _case("weather_f32_train", "train", "f32", 1, 80, 64, 128, 4, 512, 8, "8,10", "fields"),
        # sizes that no tile divides: 77 channels, 135 patches of 16 x 16, an embedding of 384
        _case("ragged_bf16_train", "train", "bf16", 2, 77, 144, 240, 16, 384, 6, "10,8", "bands"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Channels 5 .. 1024, 12 .. 2048 patches of 4, 8 or 16 pixels a side, embeddings 128 .. 4096, 2 .. 32 heads (4 x 4 patches:
    at most 24) of 32, 64 or 128 columns, one to three levels; no case costs more than the largest listed one."""
    while True:
        call = rng.choice(["forward", "forward_pos", "folded", "prefolded", "train", "train", "level"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        B, C = rng.randint(1, 4), _log_int(rng, 5, 1024)
        p = rng.choice([4, 8, 8, 16])
        hp, wp = _log_int(rng, 3, 32), _log_int(rng, 4, 64)
        D = rng.choice([128, 256, 384, 512, 512, 768, 1024, 1024, 2048, 4096])
        dh = rng.choice([32, 64, 64, 128])
        heads = D // dh
        if D % dh or heads < 2 or heads > (24 if p == 4 else 32):
            continue
        g1 = min(C, _log_int(rng, 4, 32))
        groups, left = [g1], -(-C // g1)
        if call != "level":
            if left > 16 and rng.random() < 0.7:
                groups.append(8)
                left = -(-left // 8)
            if left > 1:
                groups.append(left)
            if left > 32:
                continue
        N, es = hp * wp, 2 if dtype == "bf16" else 4
        T = B * C * N
        G_all, c_in = 0, C
        for g in groups:
            c_in = -(-c_in // g)
            G_all += c_in
        tiled = dtype == "bf16" and D % 256 == 0
        fused = call in ("folded", "prefolded", "train")
        if G_all * D * D * es > 620_000_000 or T * p * p * es > 1_000_000_000:
            continue                                     # weights and images of the listed cases' order
        if T * D > (2 ** 29 if tiled else 2 ** 25) or (not fused and T * D * D > (2 ** 42 if tiled else 2 ** 35)):
            continue
        linear = call not in ("level",) and len(groups) > 1 and rng.random() < 0.2
        return _case("", call, dtype, B, C, hp * p, wp * p, p, D, heads, ",".join(map(str, groups)),
                     rng.choice(["fields", "bands", "iid"]), linear)


def _groups(case):
    return [int(g) for g in case["groups"].split(",")]


def _images(gen, case):
    """fields: fields smoothed over 5 x 5 pixels, standardised per channel, scaled by 0.5 .. 2; bands: AR(1) along the
    channels (0.95) plus noise of 0.1; iid: Gaussian."""
    B, C, H, W = case["B"], case["C"], case["H"], case["W"]
    dev = "cuda"
    x = torch.randn(B, C, H, W, generator=gen, device=dev)
    if case["x"] == "fields":
        x = torch.nn.functional.avg_pool2d(torch.nn.functional.pad(x, (2, 2, 2, 2), mode="circular"), 5, stride=1)
        x = (x - x.mean((0, 2, 3), keepdim=True)) / x.std((0, 2, 3), keepdim=True)
        x = x * (0.5 + 1.5 * torch.rand(1, C, 1, 1, generator=gen, device=dev))
    elif case["x"] == "bands":
        x[:, 1:] *= math.sqrt(1.0 - 0.95 ** 2)
        for c in range(1, C):
            x[:, c].add_(x[:, c - 1], alpha=0.95)
        x = x + 0.1 * torch.randn(B, C, H, W, generator=gen, device=dev)
    return x


def prepare(case, seed):
    """Images (or tokens), weights of a random initialisation, and the buffers a program keeps between its calls."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tdt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    B, C, H, W, p, D, heads = (case[k] for k in ("B", "C", "H", "W", "p", "D", "heads"))
    N, gs, call = (H // p) * (W // p), _groups(case), case["call"]

    def normal(*shape, std=1.0, mean=0.0):
        a = torch.empty(shape, dtype=tdt, device="cuda")
        flat, step = a.view(-1), 1 << 26
        for i in range(0, flat.numel(), step):
            part = flat[i:i + step]
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda").mul_(std).add_(mean))
        return a

    s = {"case": case}
    if call == "level":
        s["tokens"] = normal(B, C, N, D, std=math.sqrt(2.0))
    else:
        s["x"] = _images(gen, case).to(tdt).contiguous()
        s["We"], s["be"], s["ce"] = normal(C, D, p * p, std=1.0 / p), normal(C, D, std=1.0 / p), normal(C, D)
    levels, c_in, fin = [], C, 1.0 / math.sqrt(D)
    for i, g in enumerate(gs):
        G = -(-c_in // g)
        if case["linear"] and i == 0:
            levels.append(dchag.LevelWeights(g, None, None, None, normal(G, g, D, std=1.0 / g, mean=1.0 / g), None,
                                             bv=normal(G, D, std=1.0 / math.sqrt(g)), kind=1))
        else:
            levels.append(dchag.LevelWeights(g, normal(G, D), *(normal(G, D, D, std=fin) for _ in range(4)),
                                             *(normal(G, D, std=fin) for _ in range(4))))
        c_in = G
    s["levels"] = levels
    which = {"level": 0, "forward": 1, "forward_pos": 1, "folded": 2, "prefolded": 2, "train": 3}[call]
    code = dchag.DCHAG_F32 if case["dtype"] == "f32" else dchag.DCHAG_BF16
    need = dchag.dchag_workspace_bytes(code, B, C, H, W, p, D, heads, gs, which)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    s["out"] = torch.empty((B, c_in, N, D) if call == "level" else (B, N, D), dtype=tdt, device="cuda")
    if call == "forward_pos":
        s["pos"] = normal(N, D, std=0.02)
    if call == "prefolded":
        s["folded"] = dchag.dchag_fold_value(s["We"], s["be"], s["ce"], levels, p, heads)   # None: nothing to prepare
    if call == "train":
        s["dout"] = normal(B, N, D)
        s["dx"], s["dWe"], s["dtok_bias"] = (torch.empty_like(s[k]) for k in ("x", "We", "ce"))
        s["grads"] = []
        for lv in levels:
            names = ("Wv", "bv") if lv.kind else ("query", "Wq", "Wk", "Wv", "Wo", "bq", "bk", "bv", "bo")
            s["grads"].append(dchag.LevelGrads(**{"d" + n: torch.empty_like(getattr(lv, n)) for n in names}))
    return s


def run(s):
    case = s["case"]
    call, p, heads, out, ws = case["call"], case["p"], case["heads"], s["out"], s["workspace"]
    if call == "level":
        return dchag.dchag_aggregate_level(s["tokens"], s["levels"][0], heads, out=out, workspace=ws)
    args = (s["x"], s["We"], s["be"], s["ce"], s["levels"], p, heads)
    if call == "forward":
        return dchag.dchag_forward(*args, out=out, workspace=ws)
    if call == "forward_pos":
        return dchag.dchag_forward_pos(*args, s["pos"], out=out, workspace=ws)
    if call == "prefolded" and s["folded"] is not None:
        return dchag.dchag_forward_prefolded(*args, s["folded"], out=out, workspace=ws)
    if call != "train":
        return dchag.dchag_forward_folded(*args, out=out, workspace=ws)
    dchag.dchag_forward_keep(*args, ws, out=out)
    dchag.dchag_backward(*args, s["dout"], s["grads"], dx=s["dx"], dWe=s["dWe"], dtok_bias=s["dtok_bias"], workspace=ws,
                         kept=True)
    grads = [{k: v for k, v in vars(g).items() if v is not None} for g in s["grads"]]
    return {"out": out, "dx": s["dx"], "dWe": s["dWe"], "dtok_bias": s["dtok_bias"], "levels": grads}


def work(case):
    """Bytes: images or tokens, weights (of a prepared call: the prepared ones), outputs and gradients, once each.
    Flops: the layer as defined with the query folded into the keys (forward, level); for the other calls the cheaper of
    projecting every member's value and projecting the per-head weighted averages, or at the first level of an inference call
    the value projection folded into the tokenizer; a training step costs three forward passes."""
    B, C, H, W, p, D, h = (case[k] for k in ("B", "C", "H", "W", "p", "D", "heads"))
    N, pp, es, call = (H // p) * (W // p), p * p, 4 if case["dtype"] == "f32" else 2, case["call"]
    T = B * C * N
    prepared = call == "prefolded"
    values = T * D if call == "level" else T * pp
    weights = 0 if call == "level" else C * D * pp + C * D * (1 if prepared else 2)
    flops = 0.0 if call == "level" else 2.0 * T * pp * D
    c_in = C
    for i, g in enumerate(_groups(case)):
        G = -(-c_in // g)
        t_in, t_out = B * c_in * N, B * G * N
        if case["linear"] and i == 0:
            weights += G * g * D + G * D
            flops += 2.0 * t_in * D
        else:
            project = 2.0 * t_in * D * D
            if call not in ("level", "forward", "forward_pos"):
                project = min(project, 2.0 * t_in * D * h + 2.0 * t_out * D * D)
                if i == 0 and call != "train":
                    project = min(project, 0.0 if prepared else 2.0 * C * D * D * pp)
            first = prepared and i == 0
            flops += project + 2.0 * t_in * h * (pp if i == 0 and call != "level" else D) + 2.0 * t_out * D * D
            flops += 0.0 if prepared else 4.0 * G * D * D
            weights += G * D * D * (1 if first else 2 if prepared else 4) + G * D * (2 if prepared else 5)
            weights += (C * h * (pp + 1) if first else G * h * D) if prepared else 0
        c_in = G
    outputs = B * c_in * N * D
    if call == "forward_pos":
        weights += N * D
    if call == "train":
        outputs += values + weights
        weights += B * N * D
        flops *= 3.0
    return {"bytes": float(es * (values + weights + outputs)), "flops": flops}


def tolerance(case):
    """About four times what the listed cases and ten drawn ones show against the same path in 64 bits (bf16: outputs 3e-3 to
    6e-3, gradients 4e-3 to 7e-3, single values 0.02 to 0.16 where a gradient cancels; f32: 0.4e-6 to 1.7e-6, 2e-6 to 2e-5)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    if case["call"] == "train":
        return {"rel": 2.8e-2, "max": 0.65}
    return {"rel": 2.2e-2, "max": 0.15}
