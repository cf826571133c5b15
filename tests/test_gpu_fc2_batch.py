"""FC2 over listed fp16 rows for batches (the matrix-core form): list lengths around its 64-slot
chunks, column counts that are no multiple of its 64-column tile, every batch that runs it, and
FC1 outputs over a range that 16-bit halves cannot hold without scaling.  Against plain torch in
64 bits."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pf():
    from paper_2312_12456_amd import pf
    pf.lib()
    return pf


def _case(pf, d, ffn, n, B, spread, up_scale=1.0, b_up=None):
    g = torch.Generator(device="cuda").manual_seed(1000 * n + 10 * B + d)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    w_up = (rnd(ffn, d) * (up_scale / math.sqrt(d))).half()
    w_down = (rnd(ffn, d) / math.sqrt(d)).half()
    if b_up is None:  # magnitudes over 10^-spread .. 10^spread, in no order
        b_up = torch.where(rnd(ffn) > 0, 10.0 ** (spread * (2 * torch.rand(ffn, generator=g, device="cuda") - 1)),
                           rnd(ffn))
    b_up = b_up.float().contiguous()
    b_down = rnd(d) * 0.1
    x = rnd(B, d)
    ctx = pf.Context(d, ffn, 64, max_batch=B)
    L = pf.Layer(ctx, d, ffn, 64, w_up=w_up, w_down=w_down, b_up=b_up, b_down=b_down,
                 p1=torch.zeros(64, d, dtype=torch.half, device="cuda"),
                 p2=torch.zeros(ffn, 64, dtype=torch.half, device="cuda"))
    idx = torch.zeros(ffn, dtype=torch.int32, device="cuda")
    sel = torch.randperm(ffn, generator=g, device="cuda")[:n].sort().values
    idx[:n] = sel.int()
    count = torch.tensor([n], dtype=torch.int32, device="cuda")
    y = torch.full((B, d), float("nan"), device="cuda")
    ctx.sparse_ffn(L, x, idx, count, y)
    torch.cuda.synchronize()
    up, dn = w_up[sel].double(), w_down[sel].double()
    h = torch.relu(x.double() @ up.T + b_up[sel].double())
    ref = h @ dn + b_down.double()
    # 32-bit sums of d and n terms: 2^-24 per term, errors adding up like a random walk, 8 sigma
    mag = (x.double().abs() @ up.abs().T + b_up[sel].double().abs()) @ dn.abs() + b_down.double().abs()
    return y.double(), ref, mag * (8 * math.sqrt(d + n + 1) * 2.0 ** -24)


@pytest.mark.parametrize("B", [4, 5, 8])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 511, 512, 1000, 1024])
@pytest.mark.parametrize("d", [96, 2056, 2080])
def test_fc2_batch_list_lengths(pf, d, n, B):
    y, ref, tol = _case(pf, d, 1024, n, B, spread=0.0)
    assert bool(((y - ref).abs() <= tol).all()), float(((y - ref).abs() - tol).max())


@pytest.mark.parametrize("B", [4, 7])
@pytest.mark.parametrize("spread", [4.0, 12.0])
def test_fc2_batch_fc1_outputs_beyond_the_halves(pf, spread, B):
    """Values up to 10^12 (far above the largest half) beside values down to 10^-12."""
    y, ref, tol = _case(pf, 256, 4096, 3000, B, spread)
    assert bool(((y - ref).abs() <= tol).all())


def test_fc2_batch_scale_grows_along_the_list(pf):
    """Each chunk of the list is larger than the one before: the running scale has to follow, and
    small outputs alone (all below the smallest half) keep their relative precision."""
    n = 4096
    grow = 10.0 ** (torch.arange(n, device="cuda").double() / n * 30 - 15)
    for b in (grow, torch.full((n,), 1e-12, device="cuda")):
        y, ref, tol = _case(pf, 64, n, n, 6, 0.0, up_scale=0.0, b_up=b)
        assert bool(((y - ref).abs() <= tol).all())


def test_fc2_batch_infinite_fc1_output(pf):
    """An infinite FC1 output makes every column infinite with the sign of its weight."""
    b = torch.ones(1024, device="cuda")
    b[70] = float("inf")
    y, ref, _ = _case(pf, 64, 1024, 1024, 5, 0.0, up_scale=0.0, b_up=b)
    assert bool((y == ref).all())
