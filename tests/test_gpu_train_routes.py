"""Training steps whose first level is taken from the pixels, attention or linear: what must hold bit for bit between calls that form
the same thing.  Every output starts at a sentinel and every workspace as NaN bytes, so that an element no kernel writes, or scratch
read before it is written, shows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_train import ATT, TOL, dev, dev_level, host, rel_err, say

pytestmark = pytest.mark.gpu

LINEAR = ("linear", "attention")


def problem(kw, linear=False, biases=True, seed=51):
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=seed, level_kinds=LINEAR if linear else None, **kw)
    pr = make_problem(cfg, biases=biases)
    args = (dev(pr.x, "bf16"), dev(pr.We, "bf16"), dev(pr.be, "bf16"), dev(pr.ce, "bf16"), [dev_level(lv, "bf16") for lv in pr.levels],
            cfg.p, cfg.heads)
    return cfg, pr, args


def nan_workspace(cfg, group_sizes, which):
    need = dchag.dchag_workspace_bytes(dchag.DCHAG_BF16, cfg.B, cfg.C, cfg.H, cfg.W, cfg.p, cfg.D, cfg.heads, group_sizes, which)
    return torch.full((need,), 255, dtype=torch.uint8, device="cuda")


def upstream(cfg, seed=77):
    return dev(np.random.Generator(np.random.PCG64(seed)).standard_normal((cfg.B, cfg.N, cfg.D)).astype(np.float32), "bf16")


def gradients(cfg, args, dout, ws, kept, want=None):
    """Gradients by name ("dx", "dWe", "dtok_bias", "l0.dWv", ...): all of them, or those in `want`."""
    x, We, _, ce, levels = args[:5]
    made = {}

    def out(name, like):
        if like is None or (want is not None and name not in want):
            return None
        made[name] = torch.full_like(like, 7.0)
        return made[name]

    grads = []
    for i, lv in enumerate(levels):
        names = ("Wv", "bv") if lv.kind else ATT
        grads.append(dchag.LevelGrads(**{"d" + n: out(f"l{i}.d{n}", getattr(lv, n)) for n in names}))
    dx, dWe, dtb = out("dx", x), out("dWe", We), out("dtok_bias", We[:, :, 0].contiguous() if ce is None else ce)
    dchag.dchag_backward(*args, dout, grads, dx=dx, dWe=dWe, dtok_bias=dtb, workspace=ws, kept=kept)
    torch.cuda.synchronize()
    return made


def training_step(cfg, args, dout, want=None):
    gs = [lv.group_size for lv in args[4]]
    ws = nan_workspace(cfg, gs, 3)
    out = dchag.dchag_forward_keep(*args, ws)
    return out, gradients(cfg, args, dout, ws, True, want)


def assert_same(a, b):
    assert a.keys() == b.keys()
    for n in a:
        assert torch.isfinite(a[n].float()).all(), n
        assert torch.equal(a[n], b[n]), n


NOMINAL = [
    (dict(B=1, C=11, H=32, W=64, p=8, D=256, heads=4, group_sizes=(11,)), False),
    (dict(B=1, C=11, H=32, W=64, p=4, D=256, heads=4, group_sizes=(11,)), False),
    (dict(B=2, C=11, H=32, W=64, p=8, D=256, heads=4, group_sizes=(11, 1)), True),
]


@pytest.mark.parametrize("kw,linear", NOMINAL)
def test_nominal_group_sizes_beyond_the_channel_count(kw, linear, monkeypatch):
    """A first level of one group, its size given as the channel count and as far more: the same numbers."""
    monkeypatch.setenv("DCHAG_LINEAR_ROUTE" if linear else "DCHAG_TRAIN_ROUTE", "tiles" if linear else "pixels")
    say(f"nominal group sizes {kw}")
    cfg, pr, args = problem(kw, linear)
    dout = upstream(cfg)
    out, want = training_step(cfg, args, dout)
    first, nominal = args[4][0], 500
    wide = dchag.LevelWeights(nominal, first.query, first.Wq, first.Wk, first.Wv, first.Wo, first.bq, first.bk, first.bv, first.bo,
                              kind=first.kind)
    if linear:
        wide.Wv = torch.zeros((1, nominal, cfg.D), dtype=torch.bfloat16, device="cuda")
        wide.Wv[:, :cfg.C] = first.Wv
    out2, got = training_step(cfg, (*args[:4], [wide, *args[4][1:]], *args[5:]), dout)
    assert torch.equal(out, out2)
    if linear:
        assert not got["l0.dWv"][:, cfg.C:].any()
        got["l0.dWv"] = got["l0.dWv"][:, :cfg.C]
    assert_same(want, got)
    ref = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    assert rel_err(host(out), ref) < TOL["bf16"]


SAME_FORWARD = [
    # 32 groups of 4, one image: half the tiles that fill the chip, so a tile's members are dealt to two workgroups
    dict(B=1, C=128, H=128, W=128, p=8, D=1024, heads=16, group_sizes=(4, 32)),
    # few tiles and many members: dealt to sixteen
    dict(B=1, C=40, H=32, W=40, p=8, D=256, heads=4, group_sizes=(20, 2)),
    # 4 x 4 patches, a short last group
    dict(B=2, C=21, H=48, W=52, p=4, D=512, heads=8, group_sizes=(8, 3)),
]


@pytest.mark.parametrize("kw", SAME_FORWARD)
def test_calls_that_take_the_first_level_from_the_pixels_agree_bit_for_bit(kw, monkeypatch):
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", "pixels")
    say(f"same forward {kw}")
    cfg, pr, args = problem(kw)
    gs = [lv.group_size for lv in args[4]]
    kept = dchag.dchag_forward_keep(*args, nan_workspace(cfg, gs, 3))
    folded = dchag.dchag_forward_folded(*args, workspace=nan_workspace(cfg, gs, 2))
    prepared = dchag.dchag_fold_value(*args[1:])
    prefolded = dchag.dchag_forward_prefolded(*args, prepared, workspace=nan_workspace(cfg, gs, 2))
    torch.cuda.synchronize()
    assert torch.isfinite(folded.float()).all()
    assert torch.equal(prefolded, folded)
    assert torch.equal(kept, folded)


# The same 256 channels and patches on both sides of the line the training step's route is chosen by (16 heads; measured: groups of
# 32, 639 us through the tokens against 674 from the pixels; groups of 16, 758 against 728).
@pytest.mark.parametrize("group_sizes,from_pixels", [((32, 8), False), ((16, 16), True)])
def test_route_of_a_training_step(group_sizes, from_pixels):
    B, C, H, W, p, D, heads = 1, 256, 128, 128, 8, 1024, 16

    def zeros(*shape):
        return torch.zeros(shape, dtype=torch.bfloat16, device="cuda")

    levels, c_in = [], C
    for g in group_sizes:
        c_in = -(-c_in // g)
        levels.append(dchag.LevelWeights(g, zeros(c_in, D), *(zeros(c_in, D, D) for _ in range(4))))
    need = dchag.dchag_workspace_bytes(dchag.DCHAG_BF16, B, C, H, W, p, D, heads, list(group_sizes), 3)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    args = (zeros(B, C, H, W), zeros(C, D, p * p), None, None, levels, p, heads)
    dchag.dchag_profile_begin()
    dchag.dchag_forward_keep(*args, ws)
    stages = {name for name, _, _ in dchag.dchag_profile_end()}
    assert ("fold_value" in stages) == from_pixels, stages
    assert ("tokenize" in stages) != from_pixels, stages


ROUTES = [
    # 8 x 8 patches, groups of 5 + 5 + 1, 130 patches (a tile and two more)
    (dict(B=2, C=11, H=80, W=104, p=8, D=512, heads=8, group_sizes=(5, 3)), False),
    # 4 x 4 patches, heads of 32, groups of 6 + 3
    (dict(B=1, C=9, H=48, W=52, p=4, D=256, heads=8, group_sizes=(6, 2)), False),
    # linear first levels, a short last group
    (dict(B=2, C=7, H=72, W=120, p=8, D=512, heads=8, group_sizes=(5, 2)), True),
    (dict(B=1, C=17, H=12, W=44, p=4, D=256, heads=4, group_sizes=(9, 2)), True),
]
IN_PART = [("dx",), ("dWe",), ("dtok_bias",), ("l0.dWv",), ("l0.dWk",), ("l0.dWq",), ("l0.dquery",), ("l0.dbq",), ("l0.dbk",),
           ("l0.dbv",), ("l0.dWo",), ("l0.dbo",), ("dx", "l0.dWv"), ("dWe", "l0.dbv"), ("dtok_bias", "l0.dWk"), ()]


def take_route(monkeypatch, linear):
    monkeypatch.setenv("DCHAG_LINEAR_ROUTE" if linear else "DCHAG_TRAIN_ROUTE", "tiles" if linear else "pixels")


@pytest.mark.parametrize("kw,linear", ROUTES)
def test_gradients_asked_for_in_part(kw, linear, monkeypatch):
    """Gradients of the first level and the tokenizer alone, in pairs and none: what the full call gives.  The second level's are
    always asked for: without them its token gradients come from other kernels."""
    take_route(monkeypatch, linear)
    say(f"gradients in part {kw}")
    cfg, pr, args = problem(kw, linear)
    dout = upstream(cfg)
    _, full = training_step(cfg, args, dout)
    assert all(torch.isfinite(v.float()).all() for v in full.values())
    second = tuple(n for n in full if n.startswith("l1."))
    for want in IN_PART:
        if linear and any(n.startswith("l0.") and n not in ("l0.dWv", "l0.dbv") for n in want):
            continue
        say(f"  {want}")
        _, got = training_step(cfg, args, dout, want + second)
        assert set(got) == set(want + second)
        for n in got:
            if linear and want == ("dx",) and n == "dx":    # dx alone: products per channel, which sum in another order
                assert rel_err(host(got[n]), host(full[n])) < TOL["bf16"]
            else:
                assert torch.equal(got[n], full[n]), n


@pytest.mark.parametrize("kw,linear", ROUTES)
def test_two_reverse_sweeps_after_one_forward(kw, linear, monkeypatch):
    """Two upstream gradients in a row on one kept workspace, against dchag_backward, which forms the forward again."""
    take_route(monkeypatch, linear)
    say(f"two reverse sweeps {kw}")
    cfg, pr, args = problem(kw, linear)
    gs = [lv.group_size for lv in args[4]]
    ws = nan_workspace(cfg, gs, 3)
    dchag.dchag_forward_keep(*args, ws)
    for seed in (61, 62):
        dout = upstream(cfg, seed)
        assert_same(gradients(cfg, args, dout, nan_workspace(cfg, gs, 3), False), gradients(cfg, args, dout, ws, True))


@pytest.mark.parametrize("kw,linear", ROUTES)
def test_training_step_repeats_itself(kw, linear, monkeypatch):
    take_route(monkeypatch, linear)
    say(f"repeats itself {kw}")
    cfg, pr, args = problem(kw, linear, biases=False)
    dout = upstream(cfg)
    out, want = training_step(cfg, args, dout)
    for _ in range(2):
        out2, got = training_step(cfg, args, dout)
        assert torch.equal(out, out2)
        assert_same(want, got)
