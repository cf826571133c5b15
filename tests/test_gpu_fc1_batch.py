"""FC1, and the predictor's hidden layer, of a batch behind the first layer of a stack."""
import numpy as np
import pytest
import torch

from paper_2312_12456_amd import workload as wl
from tests.util import MaskTrace, small_cfg

pytestmark = pytest.mark.gpu


def _fc1_error(pf, d, act, B, grid, min_batch, seed):
    """Error of FC1 by itself: the second FC2 matrix is the identity (times 2^12, so that the glue's own rounding is
    a small part), and what leaves the stack is FC1's output under the glue's norm."""
    ffn = max(1024, (d + 63) // 64 * 64)
    cfg = small_cfg(d=d, ffn=ffn, r=64, act=act, rate=0.3, layers=2)
    lays = [wl.make_layer(cfg, l, seed, device="cuda") for l in range(2)]
    on = torch.zeros(ffn, dtype=torch.bool, device="cuda")
    on[:d] = True                       # listed by the logit biases alone
    lay = lays[1]
    lay["p1"].zero_()
    lay["p_bias"] = torch.where(on, 1.0, -1.0).float().contiguous()
    lay["w_down"].zero_()
    lay["w_down"][torch.arange(d), torch.arange(d)] = 4096.0
    lay["b_down"] = None
    lay["b_up"] = torch.full_like(lay["b_up"], 0.5)
    x0 = wl.make_inputs(cfg, 0, seed, batch=B, device="cuda")
    ctx = pf.Context(d, ffn, 64, max_batch=B)
    ctx.set_option(pf.OPT_MFMA_MIN_BATCH, min_batch)
    ctx.set_option(pf.OPT_MFMA_GRID, grid)
    Ls = [pf.Layer.from_workload(ctx, cfg, t) for t in lays]
    x1, out = torch.empty_like(x0), torch.empty_like(x0)
    ctx.stack_step(Ls[:1], x0, x1)
    ctx.stack_step(Ls, x0, out)
    torch.cuda.synchronize()
    x = x1.double()
    up = x @ lay["w_up"].double().T
    if act == wl.ACT_RELU:
        h = torch.relu(up + 0.5)
    else:
        h = torch.relu(x @ lay["w_gate"].double().T + 0.5) * (torch.relu(up) if act == wl.ACT_DRELU else up)
    v = x + 4096.0 * h[:, :d]
    ref = v.abs() * (d ** 0.5 / v.norm(dim=1, keepdim=True))
    e = out.double().abs() - ref
    e -= ref * ((e * ref).sum(1, keepdim=True) / (ref * ref).sum(1, keepdim=True))  # the norm's own rounding
    return float(e.norm() / ref.norm())


@pytest.mark.parametrize("grid", [0, 24])  # at most 16 rows a workgroup (one 16-row pass), and more (32-row passes)
@pytest.mark.parametrize("B,d,act", [(4, 264, wl.ACT_RELU), (8, 520, wl.ACT_RELU), (5, 1032, wl.ACT_RELU),
                                     (5, 1416, wl.ACT_RELU), (8, 1544, wl.ACT_RELU), (4, 2056, wl.ACT_REGLU),
                                     (6, 3080, wl.ACT_DRELU), (3, 5128, wl.ACT_REGLU), (5, 3080, wl.ACT_RELU)])
def test_ragged_widths_no_less_accurate_than_the_vector_form(B, d, act, grid):
    """Mean error over seeds, at most that of the vector form: 1 % is what the mean of eight still varies by (each
    is a 2-norm over 1000 values and more), where the two forms are apart at all they are by 4 % and more."""
    from paper_2312_12456_amd import pf
    err = np.array([[_fc1_error(pf, d, act, B, grid, mb, 40 + s) for mb in (0, 9)] for s in range(8)])
    assert err[:, 0].mean() <= err[:, 1].mean() * 1.01, err


def _signs(ctx, B, d):
    one, out = torch.ones((B, d), device="cuda"), torch.empty((B, d), device="cuda")
    ctx.stack_glue(one, torch.zeros_like(one), out)
    return torch.sign(out).double()


@pytest.mark.parametrize("B,d,act,matrix", [(8, 1544, wl.ACT_RELU, "w_up"), (4, 2056, wl.ACT_REGLU, "w_gate"),
                                            (4, 2056, wl.ACT_REGLU, "w_up"), (5, 2080, wl.ACT_DRELU, "w_gate"),
                                            (6, 2560, wl.ACT_RELU, "w_up")])
@pytest.mark.parametrize("grid", [0, 24])
def test_infinite_weights_of_fc1(B, d, act, matrix, grid):
    """An infinite weight makes h infinite, or zero behind the ReLU, by the sign of the activation that it meets:
    y and what leaves the stack are NaN for exactly the tokens that 64 bits say."""
    from paper_2312_12456_amd import pf
    cfg = small_cfg(d=d, ffn=1024, r=64, act=act, rate=0.3, layers=2)
    lays = [wl.make_layer(cfg, l, d, device="cuda") for l in range(2)]
    lay = lays[1]
    lay["p1"].zero_()
    lay["p_bias"] = torch.ones_like(lay["p_bias"])          # every neuron is listed
    x0 = wl.make_inputs(cfg, 0, d, batch=B, device="cuda")
    clean, hit = lay[matrix].clone(), 0
    for col in (0, 3, 517, 1031, d - 1):
        lay[matrix].copy_(clean)
        lay[matrix][7, col] = float("inf")
        ctx = pf.Context(d, cfg.ffn, cfg.r, max_batch=B)
        ctx.set_option(pf.OPT_MFMA_GRID, grid)
        Ls = [pf.Layer.from_workload(ctx, cfg, t) for t in lays]
        x1, out = torch.empty_like(x0), torch.empty_like(x0)
        ctx.stack_step(Ls[:1], x0, x1)
        ctx.profile_begin()
        ctx.stack_step(Ls, x0, out)
        assert ctx.profile_end()["k_up_mfma"][0] >= 1
        torch.cuda.synchronize()
        x = x1.double()
        up, b_up = x @ lay["w_up"].double().T, lay["b_up"].double()
        if act == wl.ACT_RELU:
            h = torch.relu(up + b_up)
        else:
            h = torch.relu(x @ lay["w_gate"].double().T + b_up) * (torch.relu(up) if act == wl.ACT_DRELU else up)
        finite = torch.isfinite(h).all(1)
        hit += int((~finite).sum())
        assert torch.equal(torch.isfinite(out).all(1), finite), col
        assert bool(torch.isnan(out).all(1)[~finite].all())
        ref = _signs(ctx, B, d) * (x + h @ lay["w_down"].double() + (0 if lay["b_down"] is None else lay["b_down"].double()))
        ref = ref * (d ** 0.5 / ref.norm(dim=1, keepdim=True))
        if bool(finite.any()):
            assert (out.double() - ref)[finite].norm() < 1e-5 * ref[finite].norm()
    assert hit >= 3


@pytest.mark.parametrize("B,d,r", [(4, 1408, 72), (8, 1544, 72), (4, 4096, 72), (6, 2560, 40)])
def test_infinite_weights_of_the_hidden_layer(B, d, r):
    """An infinite weight of the predictor's hidden layer decides every logit of the tokens whose activation has its
    sign (r no multiple of 32: the output layer takes the hidden vector in fp32)."""
    from paper_2312_12456_amd import pf
    cfg = small_cfg(d=d, ffn=1024, r=r, rate=0.3, layers=2)
    lays = [wl.make_layer(cfg, l, d, device="cuda") for l in range(2)]
    lay = lays[1]
    x0 = wl.make_inputs(cfg, 0, d, batch=B, device="cuda")
    clean, hit = lay["p1"].clone(), 0
    for col in (0, 3, 517, 1031, d - 1):
        lay["p1"].copy_(clean)
        lay["p1"][5, col] = float("inf")
        ctx = pf.Context(d, cfg.ffn, r, max_batch=B)
        Ls = [pf.Layer.from_workload(ctx, cfg, t) for t in lays]
        x1, out = torch.empty_like(x0), torch.empty_like(x0)
        ctx.stack_step(Ls[:1], x0, x1)
        trace = MaskTrace(ctx, 2, cfg.ffn)
        ctx.profile_begin()
        ctx.stack_step(Ls, x0, out)
        assert ctx.profile_end()["k_glue"][0] >= 2          # the matrix-core form, behind a glue of its own
        torch.cuda.synchronize()
        t = torch.relu(x1.double() @ lay["p1"].double().T)
        hit += int(torch.isinf(t[:, 5]).sum())
        logit = t @ lay["p2"].double().T + lay["p_bias"].double()
        score = torch.sigmoid(logit)
        clear = ((score - cfg.threshold).abs() > 1e-4).all(0)
        on = torch.from_numpy(np.asarray(trace.masks()[1])).cuda()
        assert torch.equal(on[clear], (score > cfg.threshold).any(0)[clear]), col
    assert hit >= 3
