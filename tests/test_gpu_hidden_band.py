"""Which form of the predictor's hidden layer a batch takes, and that the matrix-core form is no less
accurate than the vector form.  Up to B * d = 20480 pf_predict, and single int4 layers, stay on the
vector units: fp32 activations over all of fp32's range."""
import math

import pytest
import torch

from paper_2312_12456_amd import workload as wl
from tests.util import small_cfg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pf():
    from paper_2312_12456_amd import pf
    pf.lib()
    return pf


def _predict(pf, cfg, lay, x, min_elems=None):
    B = x.shape[0]
    ctx = pf.Context(cfg.d, cfg.ffn, cfg.r, max_batch=B)
    if min_elems is not None:
        ctx.set_option(pf.OPT_HIDDEN_MFMA_MIN_ELEMS, min_elems)
    L = pf.Layer.from_workload(ctx, cfg, lay)
    scores = torch.full((B, cfg.ffn), float("nan"), device="cuda")
    words = torch.zeros(cfg.ffn // 64, dtype=torch.int64, device="cuda")
    ctx.predict(L, x, scores, words)
    torch.cuda.synchronize()
    return scores, words


@pytest.mark.parametrize("wtype", [wl.W_FP16, wl.W_INT4_G128])
@pytest.mark.parametrize("B,d", [(4, 4096), (4, 5120), (5, 4096), (8, 2560)])
def test_predict_with_an_activation_beyond_fp16(pf, B, d, wtype):
    cfg = small_cfg(d=d, ffn=512, r=128, wtype=wtype, rate=0.3)
    lay = wl.make_layer(cfg, 0, 11, device="cuda")
    lay["p1"][:, 77] *= 2.0 ** -14      # the outlier's share of the hidden vector stays ordinary
    x = wl.make_inputs(cfg, 0, 3, batch=B, device="cuda")
    x[1, 77] = 3.0e5
    scores, words = _predict(pf, cfg, lay, x)
    t = torch.relu(x.double() @ lay["p1"].double().T)
    ref = torch.sigmoid(t @ lay["p2"].double().T + lay["p_bias"].double())
    assert (scores.double() - ref).abs().max() < 1e-5
    bits = ((words[:, None] >> torch.arange(64, device="cuda")) & 1).reshape(-1).bool()
    clear = ((ref - cfg.threshold).abs() > 1e-4).all(0)
    assert torch.equal(bits[clear], (ref > cfg.threshold).any(0)[clear])
    # the vector form, not another of the same accuracy
    assert torch.equal(scores, _predict(pf, cfg, lay, x, 1 << 30)[0])
    if wtype == wl.W_INT4_G128:     # the layer step lists the same neurons, and its FC1 takes them
        ctx = pf.Context(cfg.d, cfg.ffn, cfg.r, max_batch=B)
        L = pf.Layer.from_workload(ctx, cfg, lay)
        y = torch.full((B, d), float("nan"), device="cuda")
        ctx.layer_step(L, x, y)
        torch.cuda.synchronize()
        got = torch.empty_like(words)
        pf.copy_from_device_address(got, ctx.last_active()[0])
        assert torch.equal(got, words) and bool(torch.isfinite(y).all())


def test_stack_takes_the_matrix_cores_where_the_input_allows(pf):
    """Between 15360 and 20480 the layers of an fp16 stack run the matrix-core form (a split or glue
    kernel in front of each), and those of an int4 stack behind the first, whose input may have any
    value."""
    for wtype in (wl.W_FP16, wl.W_INT4_G128):
        cfg = small_cfg(d=4096, ffn=512, r=128, wtype=wtype, rate=0.3, layers=3)
        lays = [wl.make_layer(cfg, l, 5, device="cuda") for l in range(3)]
        x = wl.make_inputs(cfg, 0, 5, batch=4, device="cuda")
        out = []
        for min_elems in (None, 1 << 30):
            ctx = pf.Context(cfg.d, cfg.ffn, cfg.r, max_batch=4)
            if min_elems is not None:
                ctx.set_option(pf.OPT_HIDDEN_MFMA_MIN_ELEMS, min_elems)
            out.append(torch.full_like(x, float("nan")))
            ctx.profile_begin()
            ctx.stack_step([pf.Layer.from_workload(ctx, cfg, t) for t in lays], x, out[-1])
            glues = ctx.profile_end()["k_glue"][0]
            torch.cuda.synchronize()
            assert glues == (1 if min_elems is not None else 4 if wtype == wl.W_FP16 else 3)
        assert (out[0] - out[1]).abs().max() < 1e-4


@pytest.mark.parametrize("B,d,r", [(4, 4096, 256), (8, 2048, 512), (3, 5152, 512)])
def test_matrix_hidden_layer_no_less_accurate_than_the_vector_form(pf, B, d, r):
    """Error of the scores against 64 bits behind the same output layer; mean over seeds."""
    cfg = small_cfg(d=d, ffn=4096, r=r, rate=0.3)
    err = [0.0, 0.0]
    for seed in range(4):
        lay = wl.make_layer(cfg, 0, seed, device="cuda")
        x = wl.make_inputs(cfg, 0, seed, batch=B, device="cuda")
        t = torch.relu(x.double() @ lay["p1"].double().T)
        ref = torch.sigmoid(t @ lay["p2"].double().T + lay["p_bias"].double())
        for form, min_elems in enumerate((0, 1 << 30)):
            err[form] += float((_predict(pf, cfg, lay, x, min_elems)[0].double() - ref).norm() / ref.norm())
    assert err[0] <= err[1], err


def test_matrix_hidden_layer_keeps_small_activations(pf):
    """Elements 2^-20 of the others, alone in the rows of the predictor that matter: two halves without
    a scale would leave 5 bits of them."""
    B, d = 8, 4096
    cfg = small_cfg(d=d, ffn=512, r=128, rate=0.3)
    lay = wl.make_layer(cfg, 0, 9, device="cuda")
    x = wl.make_inputs(cfg, 0, 9, batch=B, device="cuda")
    x[:, ::2] *= 2.0 ** -20
    lay["p1"][:, 1::2] = 0.0
    lay["p2"] *= 2.0 ** 14
    scores, _ = _predict(pf, cfg, lay, x)
    t = torch.relu(x.double() @ lay["p1"].double().T)
    ref = torch.sigmoid(t @ lay["p2"].double().T + lay["p_bias"].double())
    # the d / 2 elements' errors of 2^-36 (2^-16 of an element) add up like a random walk, and are then
    # multiplied by weights of 2^14 / sqrt(r) each in r terms: 8 sigma, 1/4 = the sigmoid's slope
    tol = 8 * 0.25 * 2.0 ** 14 * 2.0 ** -36 * math.sqrt(d / 2) / math.sqrt(d) + 1e-6
    assert (scores.double() - ref).abs().max() < tol
