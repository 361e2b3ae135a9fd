"""GPU parity of the single-precision products of whole slices and whole 16-byte pieces (k_gemm_f32_ring) at the edges of their tiles,
and of shapes next to them that keep the general kernel, against the oracle."""
import pytest

from workloads import ShapeCfg

from .test_gpu_products import check_training_step, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # columns of one and a half tiles, heads of 32 (one slice), 64 patches (two slices), last group of one member
    dict(B=2, C=7, H=32, W=32, p=4, D=96, heads=3, group_sizes=(3, 3)),
    # one slice of patches, rows of half a tile, 5 heads (a score product of 5 columns)
    dict(B=1, C=5, H=16, W=32, p=4, D=160, heads=5, group_sizes=(5,)),
    # columns of two tiles and 4, a contraction of whole slices only over the patches (D is no multiple of 32: the other products
    # keep the general kernel), 4 x 96 tokens dealt to several blocks
    dict(B=1, C=9, H=32, W=48, p=4, D=132 + 4, heads=2, group_sizes=(4, 3)),
    # long contractions: 2 x 512 patches in one sum, 4 heads of 64
    dict(B=2, C=4, H=64, W=128, p=4, D=256, heads=4, group_sizes=(2, 2)),
]


@pytest.mark.parametrize("kw", SHAPES)
def test_training_step_in_single_precision(kw):
    say(f"f32 ring {kw}")
    check_training_step(ShapeCfg(name="t", dtype="f32", x_kind="gauss_mu_sigma", seed=64, **kw))
