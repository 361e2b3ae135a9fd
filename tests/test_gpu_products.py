"""GPU parity at the sizes where the matrix products of the library can go wrong: contractions that no slice divides,
outputs that no tile divides, operands whose rows are not 16-byte aligned, contractions dealt to several blocks.
Forward (with and without the positional embedding) and every gradient against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_21411_amd as dchag
from workloads import ShapeCfg, make_problem

from .test_gpu_train import ATT, TOL, dev, dev_level, host, rel_err, say

pytestmark = pytest.mark.gpu


def check_training_step(cfg, seed=77, biases=True):
    pr = make_problem(cfg, biases=biases)
    d = cfg.dtype
    args = (dev(pr.x, d), dev(pr.We, d), dev(pr.be, d), dev(pr.ce, d), [dev_level(lv, d) for lv in pr.levels], cfg.p,
            cfg.heads)
    gs = [lv.group_size for lv in pr.levels]
    code = dchag.DCHAG_F32 if d == "f32" else dchag.DCHAG_BF16
    # outputs start at a sentinel and the workspace as NaN bytes: an element no kernel writes shows
    need = dchag.dchag_workspace_bytes(code, cfg.B, cfg.C, cfg.H, cfg.W, cfg.p, cfg.D, cfg.heads, gs, 3)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    out = dchag.dchag_forward_keep(*args, ws)
    dout = dev(np.random.Generator(np.random.PCG64(seed)).standard_normal((cfg.B, cfg.N, cfg.D)).astype(np.float32), d)
    dx, dWe, dtb = torch.full_like(args[0], 7.0), torch.full_like(args[1], 7.0), torch.full_like(args[3], 7.0)
    grads = []
    for lv in args[4]:
        names = [n for n in (("Wv", "bv") if lv.kind else ATT) if getattr(lv, n) is not None]
        grads.append(dchag.LevelGrads(**{"d" + n: torch.full_like(getattr(lv, n), 7.0) for n in names}))
    dchag.dchag_backward(*args, dout, grads, dx=dx, dWe=dWe, dtok_bias=dtb, workspace=ws, kept=True)
    torch.cuda.synchronize()
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    errs = {"out": rel_err(host(out), want)}
    ref = oracle.backward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads, host(dout).reshape(-1, cfg.D))
    for name, got in (("dx", dx), ("dWe", dWe), ("dtok_bias", dtb)):
        want_g = ref[name]
        if name == "dx":                                  # patch rows [B*N, C, p*p] -> image
            hp, wp = cfg.H // cfg.p, cfg.W // cfg.p
            want_g = want_g.reshape(cfg.B, hp, wp, cfg.C, cfg.p, cfg.p).transpose(0, 3, 1, 4, 2, 5).reshape(got.shape)
        errs[name] = rel_err(host(got), want_g)
    for i, (g, r) in enumerate(zip(grads, ref["levels"])):
        for name, got in vars(g).items():
            if got is None:
                continue
            if name == "dbk":
                assert not host(got).any()
                continue
            # a group of one has no gradient on its query path: the oracle's exact zeros leave nothing to divide by
            if np.abs(r[name]).max() < 1e-12:
                assert np.abs(host(got)).max() < 1e-6
                continue
            errs[f"l{i}.{name}"] = rel_err(host(got), r[name])
    worst = max(errs, key=errs.get)
    say(f"  worst {worst} {errs[worst]:.3e}  out {errs['out']:.3e}")
    assert errs[worst] < TOL[d], errs


PRODUCTS = [
    # bf16, embeddings no 256 divides: 135 patches (contraction of two slices and 7), 384 columns, 77 = 7 x 10 + 7 channels
    dict(dtype="bf16", B=2, C=21, H=144, W=240, p=16, D=384, heads=6, group_sizes=(10, 3)),
    # contraction shorter than one slice (9 patches, heads of 32 columns), 160 columns
    dict(dtype="bf16", B=1, C=5, H=12, W=12, p=4, D=160, heads=5, group_sizes=(3, 2)),
    # one patch
    dict(dtype="bf16", B=1, C=4, H=8, W=8, p=8, D=128, heads=2, group_sizes=(4,)),
    # f32: 136 columns (tiles of 64 and a remainder of 8), 7 patches, 17 columns a head: rows that are no multiple of 4
    dict(dtype="f32", B=2, C=9, H=2, W=14, p=2, D=136, heads=8, group_sizes=(4, 3)),
    # 5 heads (rows of 5 floats: no 16-byte loads), 33 patches, 40 columns
    dict(dtype="f32", B=1, C=11, H=6, W=22, p=2, D=40, heads=5, group_sizes=(11,)),
    # f32 by groups: 35 members (three tiles of 16, one of them past the group) + 1, 17 heads (two blocks; no dz by groups), 272 columns
    dict(dtype="f32", B=1, C=36, H=6, W=10, p=2, D=272, heads=17, group_sizes=(35, 2)),
    # 20 members + 9, 12 heads (three quarters of a block), an odd number of patches
    dict(dtype="f32", B=2, C=29, H=6, W=6, p=2, D=48, heads=12, group_sizes=(20, 2)),
    # a contraction over 16 x 200 tokens dealt to several blocks, the last group shorter (13 members)
    dict(dtype="f32", B=1, C=29, H=40, W=80, p=4, D=64, heads=2, group_sizes=(16, 2)),
]


@pytest.mark.parametrize("kw", PRODUCTS)
def test_training_step_at_the_edges_of_the_products(kw):
    say(f"products {kw}")
    check_training_step(ShapeCfg(name="t", x_kind="gauss_mu_sigma", seed=11, **kw))


@pytest.mark.parametrize("kw", [PRODUCTS[0], PRODUCTS[3]])
def test_positional_embedding_is_added_by_the_products(kw):
    cfg = ShapeCfg(name="t", x_kind="gauss_mu_sigma", seed=12, **kw)
    say(f"products, positional embedding {kw}")
    pr = make_problem(cfg)
    d = cfg.dtype
    pos = np.random.Generator(np.random.PCG64(3)).standard_normal((cfg.N, cfg.D)).astype(np.float32)
    pos_d = dev(pos, d)
    out = dchag.dchag_forward_pos(dev(pr.x, d), dev(pr.We, d), dev(pr.be, d), dev(pr.ce, d),
                                  [dev_level(lv, d) for lv in pr.levels], cfg.p, cfg.heads, pos_d)
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)
    err = rel_err(host(out), want + host(pos_d)[None])
    say(f"  err {err:.3e}")
    assert err < TOL[d]


# More rows a group than the row tiles of the products' grids hold (65535 tiles of 64 rows in fp32, of 128 in bf16): real ones, and
# rows of members that a nominal group size larger than the channel count only promises.
MANY_ROWS = [
    dict(dtype="f32", B=1, C=65, H=256, W=256, p=1, D=8, heads=2, group_sizes=(65,)),
    dict(dtype="f32", B=1, C=8, H=16, W=16, p=2, D=24, heads=3, group_sizes=(100000,)),
    dict(dtype="bf16", B=1, C=8, H=16, W=16, p=2, D=24, heads=3, group_sizes=(300000,)),
]


@pytest.mark.parametrize("kw", MANY_ROWS)
@pytest.mark.parametrize("call", ["forward", "folded"])
def test_more_rows_than_the_grid_has_row_tiles(kw, call):
    cfg = ShapeCfg(name="t", x_kind="gauss_mu_sigma", seed=13, **kw)
    say(f"many rows, {call} {kw}")
    pr = make_problem(cfg)
    d = cfg.dtype
    run = dchag.dchag_forward if call == "forward" else dchag.dchag_forward_folded
    out = run(dev(pr.x, d), dev(pr.We, d), dev(pr.be, d), dev(pr.ce, d), [dev_level(lv, d) for lv in pr.levels], cfg.p,
              cfg.heads)
    n = np.unique(np.linspace(0, cfg.N - 1, 40).astype(np.int32))
    want = oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads, sample=(np.zeros_like(n), n))
    assert rel_err(host(out[0, torch.from_numpy(n).long().cuda()]), want) < TOL[d]
    assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("kw", [PRODUCTS[0], PRODUCTS[3]])
def test_positional_embedding_is_added_without_the_matrix_instructions(kw, monkeypatch):
    monkeypatch.setenv("DCHAG_GEMM_GENERIC", "1")
    test_positional_embedding_is_added_by_the_products(kw)


@pytest.mark.parametrize("kw", [PRODUCTS[0], PRODUCTS[3], PRODUCTS[7]])
def test_training_step_without_the_matrix_instructions(kw, monkeypatch):
    """The fp32-FMA kernels behind the products, fp32 and bf16, on the shapes the products are checked at."""
    monkeypatch.setenv("DCHAG_GEMM_GENERIC", "1")
    check_training_step(ShapeCfg(name="t", x_kind="gauss_mu_sigma", seed=11, **kw))


# Contractions of 512 and 1024 steps, key-path sums dealt to several blocks.
PRECISION = [
    dict(dtype="f32", B=1, C=24, H=32, W=64, p=4, D=512, heads=8, group_sizes=(8, 3)),
    dict(dtype="f32", B=2, C=14, H=24, W=40, p=4, D=1024, heads=16, group_sizes=(14,)),
]


@pytest.mark.parametrize("kw", PRECISION)
def test_fp32_products_round_no_more_than_the_vector_kernels(kw, monkeypatch):
    """2-norm errors against the fp64 oracle of everything a training step gives, on the matrix instructions and on the fp32-FMA
    kernels: two orders of the same sums, so a tenth is left for chance."""
    cfg = ShapeCfg(name="t", x_kind="gauss_mu_sigma", seed=14, **kw)
    say(f"precision {kw}")
    pr = make_problem(cfg)
    dout = np.random.Generator(np.random.PCG64(78)).standard_normal((cfg.B, cfg.N, cfg.D)).astype(np.float32)
    want = {"out": oracle.forward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads).reshape(cfg.B, cfg.N, cfg.D)}
    ref = oracle.backward(pr.x, pr.We, pr.be, pr.ce, pr.levels, cfg.p, cfg.heads, dout.reshape(-1, cfg.D).astype(np.float64))
    hp, wp = cfg.H // cfg.p, cfg.W // cfg.p
    want["dx"] = ref["dx"].reshape(cfg.B, hp, wp, cfg.C, cfg.p, cfg.p).transpose(0, 3, 1, 4, 2, 5).reshape(pr.x.shape)
    want["dWe"], want["dtok_bias"] = ref["dWe"], ref["dtok_bias"]
    for i, r in enumerate(ref["levels"]):
        want.update({f"l{i}.{n}": v for n, v in r.items() if n != "dbk"})
    args = (dev(pr.x, "f32"), dev(pr.We, "f32"), dev(pr.be, "f32"), dev(pr.ce, "f32"), [dev_level(lv, "f32") for lv in pr.levels],
            cfg.p, cfg.heads)

    def errors():
        got = {"out": dchag.dchag_forward_folded(*args)}
        dx, dWe, dtb = torch.full_like(args[0], 7.0), torch.full_like(args[1], 7.0), torch.full_like(args[3], 7.0)
        grads = [dchag.LevelGrads(**{"d" + n: torch.full_like(getattr(lv, n), 7.0) for n in ATT}) for lv in args[4]]
        dchag.dchag_backward(*args, dev(dout, "f32"), grads, dx=dx, dWe=dWe, dtok_bias=dtb)
        got.update(dx=dx, dWe=dWe, dtok_bias=dtb)
        for i, g in enumerate(grads):
            got.update({f"l{i}.{n}": v for n, v in vars(g).items() if n != "dbk"})
        return {n: float(np.linalg.norm(host(got[n]) - want[n]) / np.linalg.norm(want[n])) for n in want}

    matrix = errors()
    monkeypatch.setenv("DCHAG_GEMM_GENERIC", "1")
    vector = errors()
    ratio = {n: matrix[n] / vector[n] for n in want if vector[n] > 0}
    worst = max(ratio, key=ratio.get)
    say(f"  out {vector['out']:.2e} -> {matrix['out']:.2e}, worst {worst} {ratio[worst]:.2f}")
    assert ratio[worst] < 1.1, ratio
