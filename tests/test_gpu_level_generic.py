"""GPU parity of the one-kernel scores, softmax and weighted sums of shapes that the bf16 level kernels do not take, at the edges of
its blocks, and of the separate kernels on the same shapes, against the oracle."""
import pytest

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_products import check_training_step, say
from .test_gpu_train import TOL, dev, dev_level, host, rel_err

pytestmark = pytest.mark.gpu

SHAPES = [
    # one patch, heads of one column: 8 columns (half of a step of 16), one member in the last group
    dict(B=1, C=4, H=4, W=4, p=4, D=8, heads=8, group_sizes=(3, 2)),
    # 17 members (a block and one), 9 heads (a block of sums and one), an odd number of patches
    dict(B=2, C=18, H=12, W=12, p=4, D=72, heads=9, group_sizes=(17, 2)),
    # 24 heads (two blocks of 16), 40 columns past whole steps of 64, enough patches for two a block
    dict(B=2, C=6, H=48, W=88, p=4, D=168 + 24, heads=24, group_sizes=(4, 2)),
    # 20 members and 20 heads (two blocks of each, not whole), enough patches for two a block
    dict(B=2, C=40, H=48, W=88, p=4, D=80, heads=20, group_sizes=(20, 2)),
    # the largest weights a block holds: 64 members, 64 heads
    dict(B=1, C=64, H=8, W=8, p=4, D=64, heads=64, group_sizes=(64,)),
    # one member more: the separate kernels
    dict(B=1, C=65, H=8, W=8, p=4, D=64, heads=64, group_sizes=(65,)),
]


@pytest.mark.parametrize("kw", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("unfused", [False, True])
def test_level_of_any_shape(kw, dtype, unfused, monkeypatch):
    if unfused:
        monkeypatch.setenv("DCHAG_LEVEL_UNFUSED", "1")
    say(f"generic level {dtype} unfused={unfused} {kw}")
    cfg = ShapeCfg(name="t", dtype=dtype, x_kind="gauss_mu_sigma", seed=65, **kw)
    check_training_step(cfg)
    pr = make_problem(cfg)
    args = (dev(pr.x, dtype), dev(pr.We, dtype), dev(pr.be, dtype), dev(pr.ce, dtype), [dev_level(lv, dtype) for lv in pr.levels],
            cfg.p, cfg.heads)
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    for call in (dchag.dchag_forward, dchag.dchag_forward_folded):
        err = rel_err(host(call(*args)), want)
        assert err < TOL[dtype], (call.__name__, err)


@pytest.mark.parametrize("dtype,B,N,D,heads,g,G,values_fused,sums_fused", [
    ("f32", 1, 2049, 128, 8, 3, 2, False, True),      # 4098 patches; not more than three members to a block of 16 heads
    ("f32", 1, 2049, 128, 8, 4, 2, True, True),
    ("f32", 1, 2048, 128, 8, 3, 2, True, True),       # 4096: few patches
    ("f32", 2, 683, 96, 24, 6, 3, False, True),       # two blocks of heads
    ("f32", 2, 683, 96, 24, 7, 3, True, True),
    ("f32", 3, 500, 160, 40, 17, 1, True, False),     # three blocks of heads, two of members
    ("f32", 3, 500, 160, 40, 9, 1, False, False),
    ("bf16", 1, 2049, 128, 32, 1, 2, True, True),
])
def test_route_by_heads_and_group(dtype, B, N, D, heads, g, G, values_fused, sums_fused):
    """Both sides of the rule for one kernel or separate ones, each against the oracle, and that it is the side meant: the separate kernels
    leave a timing record of their scores."""
    cfg = ShapeCfg(name="t", dtype=dtype, x_kind="gauss_mu_sigma", seed=72, B=B, C=g * G, H=4, W=4 * N, p=4, D=D, heads=heads,
                   group_sizes=(g, G) if G > 1 else (g,))
    pr = make_problem(cfg)
    args = (dev(pr.x, dtype), dev(pr.We, dtype), dev(pr.be, dtype), dev(pr.ce, dtype), [dev_level(lv, dtype) for lv in pr.levels],
            cfg.p, cfg.heads)
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    for call, fused in ((dchag.dchag_forward, values_fused), (dchag.dchag_forward_folded, sums_fused)):
        say(f"route {cfg} {call.__name__}")
        dchag.dchag_profile_begin()
        out = call(*args)
        records = dchag.dchag_profile_end()
        assert (("scores", 1) not in [(stage, level) for stage, level, _ in records]) == fused, records
        err = rel_err(host(out), want)
        say(f"  {err:.3e}")
        assert err < TOL[dtype], (call.__name__, err)
