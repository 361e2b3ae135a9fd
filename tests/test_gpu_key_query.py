"""GPU parity of the key and query gradients where rows of a head and columns of a row end: heads of 1, 6 and 8 columns (a wavefront
takes four rows of a head), rows shorter and longer than a wavefront's reach, against the oracle."""
import pytest

from workloads import ShapeCfg

from .test_gpu_products import check_training_step, say

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(B=1, C=5, H=8, W=12, p=4, D=8, heads=8, group_sizes=(3, 2)),
    dict(B=2, C=4, H=8, W=8, p=4, D=24, heads=4, group_sizes=(4,)),
    dict(B=1, C=7, H=8, W=16, p=4, D=520, heads=65, group_sizes=(4, 2)),
]


@pytest.mark.parametrize("kw", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_key_and_query_gradients(kw, dtype):
    say(f"key and query gradients {dtype} {kw}")
    check_training_step(ShapeCfg(name="t", dtype=dtype, x_kind="gauss_mu_sigma", seed=63, **kw))
