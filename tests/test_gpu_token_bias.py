"""GPU parity of the folded token biases (k_fold_token_bias) at the edges of its passes over a group's members, against the oracle."""
import pytest

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_products import say
from .test_gpu_train import TOL, dev, dev_level, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["both", "be", "ce"])
@pytest.mark.parametrize("g,C,D", [(1, 3, 256), (16, 35, 512), (17, 30, 256), (33, 67, 512)])
def test_folded_token_bias(g, C, D, which):
    """One member; whole passes of 16 and a group of three; a pass of 32 of which 17 and 13 are there; 33: a second pass of one member.
    D 256 has the four slices that fill the ring.  The biases are 32 and 4 times their usual size (exact in bf16): half of the result and more."""
    cfg = ShapeCfg(name="t", dtype="bf16", x_kind="gauss_mu_sigma", seed=71, B=1, C=C, H=32, W=64, p=8, D=D, heads=4,
                   group_sizes=(g, -(-C // g)))
    pr = make_problem(cfg)
    be = pr.be * 32 if which != "ce" else None
    ce = pr.ce * 4 if which != "be" else None
    say(f"token bias {cfg} {which}")
    bf = lambda t: None if t is None else dev(t, "bf16")
    got = host(dchag.dchag_forward_folded(dev(pr.x, "bf16"), dev(pr.We, "bf16"), bf(be), bf(ce),
                                          [dev_level(lv, "bf16") for lv in pr.levels], cfg.p, cfg.heads))
    want = oracle.forward(pr.x, pr.We, be, ce, pr.levels, cfg.p, cfg.heads)
    err = rel_err(got.reshape(want.shape), want)
    say(f"  {err:.3e}")
    assert err < TOL["bf16"], err
