"""GPU parity of the products on 256 x 256 tiles (output projections, their input and weight gradients) where their tiles, segments
and ragged rows end, against the oracle."""
import re

import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_products import check_training_step, say
from .test_gpu_train import TOL, dev, dev_level, host, rel_err

pytestmark = pytest.mark.gpu

LINEAR, BACK, WEIGHTS, FOLD, IMAGE, OUTER = range(6)       # kinds of k_product_dl


def product_kinds(call):
    """Kinds of k_product_dl that a call launched."""
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return {int(k) for e in prof.events() for k in re.findall(r"k_product_dl(?:<|ILi)(\d)", e.name)}


TRAIN = [
    # two segments of the contraction of six slices each; rows of one and a half tiles; 33 groups, the last of one member
    dict(B=2, C=65, H=64, W=96, p=4, D=512, heads=8, group_sizes=(2, 33)),
    # one segment of four slices (the shortest), three tiles of columns; 387 tiles of weights, two to some workgroups, and 129 of inputs
    dict(B=1, C=86, H=64, W=64, p=4, D=768, heads=12, group_sizes=(2, 43)),
]


@pytest.mark.parametrize("kw,biases", [(TRAIN[0], True), (TRAIN[1], True), (TRAIN[1], False)])
def test_output_projection_gradients(kw, biases, monkeypatch):
    say(f"large products, training {kw}")
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", "tokens")
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=61, **kw)
    kinds = product_kinds(lambda: check_training_step(cfg, biases=biases))
    assert kinds >= {LINEAR, BACK, WEIGHTS}, kinds


@pytest.mark.parametrize("biases", [True, False])
def test_projection_of_ragged_rows(biases):
    """260 rows a group: one tile of 256 and one of 4, 16 groups, 128 tiles; the value product with 4 rows in its last tile."""
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=62, B=1, C=32, H=80, W=208, p=8, D=1024, heads=16,
                   group_sizes=(2, 16))
    pr = make_problem(cfg, biases=biases)
    args = (dev(pr.x, "bf16"), dev(pr.We, "bf16"), dev(pr.be, "bf16"), dev(pr.ce, "bf16"), [dev_level(lv, "bf16") for lv in pr.levels],
            cfg.p, cfg.heads)
    say(f"large products, forward {cfg}")
    got = host(dchag.dchag_forward(*args))
    folded = host(dchag.dchag_forward_folded(*args))
    assert product_kinds(lambda: dchag.dchag_forward(*args)) == {LINEAR}
    assert product_kinds(lambda: dchag.dchag_forward_folded(*args)) == {LINEAR, FOLD}
    rows = np.r_[0:8, 120:136, 252:260]                   # patches at the edges of the tiles
    xs = pr.x.reshape(1, cfg.C, 10, 8, 26, 8).transpose(0, 2, 4, 1, 3, 5).reshape(cfg.N, cfg.C, 64)[rows]
    xs = xs.reshape(1, len(rows), cfg.C, 8, 8).transpose(0, 2, 3, 1, 4).reshape(1, cfg.C, 8, 8 * len(rows))
    want = oracle.forward(xs, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(len(rows), cfg.D)
    for name, y in (("forward", got), ("folded", folded)):
        err = rel_err(y.reshape(cfg.N, cfg.D)[rows], want)
        say(f"  {name} {err:.3e}")
        assert err < TOL["bf16"], (name, err)


@pytest.mark.parametrize("biases", [True, False])
def test_linear_first_level_on_large_tiles(biases, monkeypatch):
    """Tiles of four members: groups of five (one and a quarter), the last of three; 384 patches (one and a half tiles, two segments of
    six slices), 16 patches a row of the image."""
    monkeypatch.setenv("DCHAG_LINEAR_ROUTE", "tiles")
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=68, B=2, C=163, H=192, W=128, p=8, D=512, heads=8,
                   group_sizes=(5, 33), level_kinds=("linear", "attention"))
    say(f"large products, linear first level {cfg}")
    kinds = product_kinds(lambda: check_training_step(cfg, biases=biases))
    assert kinds >= {IMAGE, OUTER}, kinds
