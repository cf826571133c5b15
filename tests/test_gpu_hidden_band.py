"""The predictor's hidden layer for batches up to B * d = 20480 stays on the vector units: fp32
activations over all of fp32's range, whatever the weight type of the layer."""
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
