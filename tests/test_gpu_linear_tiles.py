"""GPU parity of the reverse step of a linear first level on tiles of (member, pixel) rows, at the edges of the tiles, and of the
per-channel products on the same shapes, against the oracle."""
import pytest

from workloads import ShapeCfg

from .test_gpu_products import check_training_step, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # 8 x 8 patches: groups of 5 + 2 (a tile of 256 rows and 64 more), 135 patches (two slices and 7)
    dict(B=2, C=7, H=72, W=120, p=8, D=512, heads=8, group_sizes=(5, 2)),
    # groups of 2 (tiles of 128 rows, 256 patches), 260 patches, a last group of one
    dict(B=1, C=5, H=80, W=208, p=8, D=256, heads=8, group_sizes=(2, 3)),
    # 4 x 4 patches, groups of 9 + 8 (a tile of 128 rows and 16 more), 33 patches
    dict(B=1, C=17, H=12, W=44, p=4, D=256, heads=4, group_sizes=(9, 2)),
    # 4 x 4 patches, 3 members of 16 rows in one tile, 64 patches, three levels
    dict(B=3, C=7, H=32, W=32, p=4, D=768, heads=12, group_sizes=(3, 2, 2)),
]


@pytest.mark.parametrize("kw", SHAPES)
@pytest.mark.parametrize("route", ["tiles", "channels"])
@pytest.mark.parametrize("biases", [True, False])
def test_training_step_with_a_linear_first_level(kw, route, biases, monkeypatch):
    say(f"linear first level, {route} {kw}")
    monkeypatch.setenv("DCHAG_LINEAR_ROUTE", route)
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=41,
                                 level_kinds=("linear",) + ("attention",) * (len(kw["group_sizes"]) - 1), **kw), biases=biases)
