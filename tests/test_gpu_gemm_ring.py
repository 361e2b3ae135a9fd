"""GPU parity of the batched bf16 products through direct-to-LDS loads (k_gemm_ring) at the edges of their tiles, and of the
register-staged kernel on the same shapes, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_products import check_training_step, say
from .test_gpu_train import TOL, dev, dev_level, host, rel_err

pytestmark = pytest.mark.gpu

SHAPES = [
    # columns of one and a half tiles, sums over two batch elements of one slice each, last group of one member
    dict(B=2, C=7, H=32, W=32, p=4, D=192, heads=3, group_sizes=(3, 3)),
    # 320 columns, three slices of patches, heads of 64; 10 heads: few tiles
    dict(B=1, C=5, H=48, W=64, p=4, D=640, heads=10, group_sizes=(5,)),
    # one head of 64 columns: a single tile of either side; 16 x 16 patches (256 columns of pixels)
    dict(B=3, C=3, H=128, W=128, p=16, D=64, heads=1, group_sizes=(2, 2)),
    # rows of a tile and 8, heads of 128, groups of 9 + 9 + 2: tiles beyond one to a compute unit
    dict(B=2, C=20, H=64, W=136, p=8, D=384, heads=3, group_sizes=(9, 3)),
]


@pytest.mark.parametrize("kw", SHAPES)
@pytest.mark.parametrize("regs", [False, True])
def test_training_step_of_whole_slices(kw, regs, monkeypatch):
    if regs:
        monkeypatch.setenv("DCHAG_GEMM_REGS", "1")
    say(f"gemm ring regs={regs} {kw}")
    check_training_step(ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=66, **kw))


@pytest.mark.parametrize("kw", [SHAPES[0], SHAPES[3], dict(B=1, C=6, H=40, W=104, p=8, D=512, heads=8, group_sizes=(3, 2))])
def test_projection_with_a_positional_embedding(kw):
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=67, **kw)
    say(f"gemm ring, positional embedding {kw}")
    pr = make_problem(cfg)
    pos_d = dev(np.random.Generator(np.random.PCG64(3)).standard_normal((cfg.N, cfg.D)).astype(np.float32), "bf16")
    out = dchag.dchag_forward_pos(dev(pr.x, "bf16"), dev(pr.We, "bf16"), dev(pr.be, "bf16"), dev(pr.ce, "bf16"),
                                  [dev_level(lv, "bf16") for lv in pr.levels], cfg.p, cfg.heads, pos_d)
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    err = rel_err(host(out), want + host(pos_d)[None])
    say(f"  err {err:.3e}")
    assert err < TOL["bf16"]
