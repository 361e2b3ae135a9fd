"""GPU parity of the one-kernel scores, softmax and head sums of a level (k_level_sums) in every form it is built in: head blocks,
patches per block, member tiles and their remainders, and of the separate kernels it stands for on the same shapes, against the oracle."""
import pytest

from workloads import ShapeCfg

from .test_gpu_products import check_training_step, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # one patch a block, 4 heads an item: 35 patches, groups of 17 (a member tile and one more) + 3, 8 heads of 32
    dict(B=1, C=20, H=40, W=56, p=8, D=256, heads=8, group_sizes=(17, 2)),
    # D 1024, 16 heads, groups of one member and of 5
    dict(B=2, C=6, H=24, W=40, p=8, D=1024, heads=16, group_sizes=(5, 2)),
    # 32 heads (two blocks), one patch a block, group of 33 (two member tiles and one)
    dict(B=1, C=33, H=8, W=24, p=8, D=1024, heads=32, group_sizes=(33,)),
    # 64 heads (four blocks)
    dict(B=1, C=9, H=16, W=24, p=8, D=2048, heads=64, group_sizes=(4, 3)),
    # four patches a block (4 x 1027 patches a group, a last block of three), 4 heads
    dict(B=4, C=5, H=4, W=4108, p=4, D=256, heads=4, group_sizes=(3, 2)),
    # two patches a block beyond D 1024, 4113 patches (a last block of one), 5 heads
    dict(B=1, C=2, H=12, W=5484, p=4, D=1280, heads=5, group_sizes=(2,)),
    # two patches a block, 24 heads in two head blocks
    dict(B=1, C=2, H=68, W=964, p=4, D=768, heads=24, group_sizes=(2,)),
]


# beyond D 2048 with more than 16 heads: the separate kernels by themselves
WIDE = dict(B=1, C=10, H=16, W=24, p=8, D=4096, heads=32, group_sizes=(4, 3))


# the separate kernels on all but the two largest shapes, whose host side takes half a minute
@pytest.mark.parametrize("kw,separate", [(kw, False) for kw in SHAPES] + [(kw, True) for kw in SHAPES[:5]])
def test_training_step_with_one_kernel_level_sums(kw, separate, monkeypatch):
    say(f"level sums, {'separate kernels' if separate else 'one kernel'} {kw}")
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", "tokens")
    monkeypatch.setenv("DCHAG_TOKEN_SCORES", "1")          # the first level's scores from its tokens too
    if separate:
        monkeypatch.setenv("DCHAG_LEVEL_UNFUSED", "1")
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=31, **kw))


def test_training_step_with_a_wide_upper_level(monkeypatch):
    say(f"level sums {WIDE}")
    monkeypatch.setenv("DCHAG_TRAIN_ROUTE", "tokens")
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=31, **WIDE))
