"""int4 layers of 4 to 8 tokens (FC2 takes 7 and 8 in two halves, a gated FC1 reads its input twice from 5 on) against
the same tokens one by one: the batch-1 kernels sum the same products, in lane and wave order; biases of long lists."""
import pytest
import torch

from paper_2312_12456_amd import workload as wl
from tests.util import small_cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [0, 1, 3])
@pytest.mark.parametrize("act", [wl.ACT_RELU, wl.ACT_REGLU, wl.ACT_DRELU])
@pytest.mark.parametrize("B,d,ffn", [(4, 128, 64), (5, 384, 448), (6, 1152, 1344), (7, 128, 64), (7, 1152, 1344),
                                     (8, 384, 448), (8, 2176, 1344), (7, 8448, 192), (8, 12288, 192)])
def test_int4_batch_against_single_tokens(B, d, ffn, act, split):
    from paper_2312_12456_amd import pf
    cfg = small_cfg(d=d, ffn=ffn, r=32, act=act, wtype=wl.W_INT4_G128, rate=0.3)
    lay = wl.make_layer(cfg, 0, d, device="cuda")
    x = wl.make_inputs(cfg, 0, d, batch=B, device="cuda")
    ctx = pf.Context(d, ffn, 32, max_batch=B)
    ctx.set_option(pf.OPT_DOWN_SPLIT, split)
    L = pf.Layer.from_workload(ctx, cfg, lay)
    for n in (0, 1, 63, ffn):
        idx = torch.randperm(ffn, generator=torch.Generator().manual_seed(n))[:n].sort().values.int()
        idx = torch.cat([idx, torch.zeros(ffn - n, dtype=torch.int32)]).cuda()
        count = torch.tensor([n], dtype=torch.int32, device="cuda")
        y, one = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
        ctx.sparse_ffn(L, x, idx, count, y)
        for b in range(B):
            ctx.sparse_ffn(L, x[b:b + 1], idx, count, one[b:b + 1])
        torch.cuda.synchronize()
        # at most 30 roundings of 2^-24 in each, independent: 3.3e-7 of the sums
        assert (y - one).norm() <= 2e-6 * one.norm(), n


@pytest.mark.parametrize("B,d,ffn,wtype,act", [(5, 264, 20480, wl.W_FP16, wl.ACT_RELU), (4, 72, 20480, wl.W_FP16, wl.ACT_REGLU),
                                               (1, 128, 10240, wl.W_INT4_G128, wl.ACT_RELU),
                                               (2, 256, 10240, wl.W_INT4_G128, wl.ACT_REGLU),
                                               (7, 128, 10240, wl.W_INT4_G128, wl.ACT_DRELU)])
def test_biases_of_several_rows_a_wave(B, d, ffn, wtype, act):
    """Lists that give a wave of FC1 more than one row (8192 waves, int4 4096), whose biases come by another way than the
    first row's, against 64 bits; an entry outside the layer in front and behind."""
    from paper_2312_12456_amd import pf
    cfg = small_cfg(d=d, ffn=ffn, r=8, act=act, wtype=wtype, rate=0.3)
    lay = wl.make_layer(cfg, 0, d, device="cuda")
    lay["b_up"] = torch.linspace(-2.0, 2.0, ffn, device="cuda")
    x = wl.make_inputs(cfg, 0, d, batch=B, device="cuda")

    def matrix(k):
        w = lay["w_" + k]
        if wtype == wl.W_FP16:
            return w.double()
        q = torch.stack([w & 15, w >> 4], dim=2).reshape(ffn, d).double() - 8.0
        return q * lay["s_" + k].double().repeat_interleave(128, dim=1)

    up = x.double() @ matrix("up").T
    if act == wl.ACT_RELU:
        h = torch.relu(up + lay["b_up"].double())
    else:
        h = torch.relu(x.double() @ matrix("gate").T + lay["b_up"].double()) * (torch.relu(up) if act == wl.ACT_DRELU else up)
    ctx = pf.Context(d, ffn, 8, max_batch=B)
    L = pf.Layer.from_workload(ctx, cfg, lay)
    idx = torch.arange(ffn, dtype=torch.int32, device="cuda").flip(0).contiguous()
    idx[3], idx[ffn - 5] = -1, ffn
    keep = torch.ones(ffn, dtype=torch.float64, device="cuda")
    keep[ffn - 4] = keep[4] = 0.0
    ref = (h * keep) @ matrix("down") + (lay["b_down"].double() if lay["b_down"] is not None else 0.0)
    y = torch.full_like(x, float("nan"))
    ctx.sparse_ffn(L, x, idx, torch.tensor([ffn], dtype=torch.int32, device="cuda"), y)
    torch.cuda.synchronize()
    # sums of 128 - 264 and of 20480 products: some 40 roundings of 2^-24 in a row, independent.  FC2 over int4 sums
    # h * (code + 8) and takes 8 * sum of h off again: h >= 0, so that for 10240 rows it passes sums of 8 * sum of h
    # <= 8 sqrt(10240) |h|_2 (scales apart), against a result of 4 |h|_2 (codes -7 .. 7 at random): 200 times.
    tol = (1 if wtype == wl.W_FP16 else 200) * 40 ** 0.5 * 2.0 ** -24
    assert (y.double() - ref).norm() < 2 * tol * ref.norm()
