"""GPU parity of the training step whose attention first level is taken from the pixels (k_pixel_train.h), at the edges of
its tiles, and of the route through the tokens on the shapes that now take the other one."""
import pytest
import torch

from workloads import ShapeCfg

from .test_gpu_products import check_training_step, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # 8 x 8 patches, heads of 64: two full tiles of 128 patches and 4 more, groups 4 + 4 + 3
    dict(B=2, C=11, H=80, W=208, p=8, D=512, heads=8, group_sizes=(4, 3)),
    # one level, 33 patches (one past the pitch of the softmax weights), a group of 5, heads of 64
    dict(B=1, C=5, H=24, W=88, p=8, D=256, heads=4, group_sizes=(5,)),
    # heads of 32 (two per wavefront), 130 patches, groups 5 + 2
    dict(B=1, C=7, H=80, W=104, p=8, D=256, heads=8, group_sizes=(5, 2)),
    # heads of 128 and of 256 (two and four pieces of the d alpha sums)
    dict(B=1, C=6, H=64, W=64, p=8, D=512, heads=4, group_sizes=(3, 2)),
    dict(B=1, C=3, H=64, W=64, p=8, D=1024, heads=4, group_sizes=(3,)),
    # 4 x 4 patches: groups of 5 + 5 + 1 (slices of four members: one and a quarter), 156 patches, heads of 64
    dict(B=2, C=11, H=48, W=52, p=4, D=512, heads=8, group_sizes=(5, 3)),
    # 4 x 4 patches, heads of 32, three batch elements of 64 patches, groups of 8 + 4
    dict(B=3, C=12, H=32, W=32, p=4, D=256, heads=8, group_sizes=(8, 2)),
    # 4 x 4, heads of 128, a contraction over 4 x 512 patches dealt to several blocks, 12 heads (three quarters of a block)
    dict(B=4, C=9, H=64, W=128, p=4, D=768, heads=12, group_sizes=(9,)),
    # 34 members (two blocks of 32 member columns), 24 heads of 32
    dict(B=1, C=70, H=64, W=64, p=8, D=768, heads=24, group_sizes=(34, 3)),
]


@pytest.mark.parametrize("kw", SHAPES)
@pytest.mark.parametrize("route", ["pixels", "tokens"])
def test_training_step_from_the_pixels_and_through_the_tokens(kw, route, monkeypatch):
    say(f"training through the {route} {kw}")
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", route)
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=21, **kw))


def test_training_step_from_the_pixels_without_biases(monkeypatch):
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", "pixels")
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=22, **SHAPES[0]), biases=False)
