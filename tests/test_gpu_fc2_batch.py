"""FC2 over listed fp16 rows for batches, against plain torch in 64 bits.  Batches of 4 and more
with d % 32 == 0 run it on the matrix cores (at batch 4 lists of more than 256 rows per row group, the
shorter ones as the vector form does), other widths (2056 here) on the vector units: list
lengths around the 64-slot chunks, lists of several chunks per wave, column counts that are no
multiple of the 64-column tile, and FC1 outputs over ranges that 16-bit halves cannot hold.

The first tests go through FC1 and FC2 and allow for the rounding of both.  In those on FC2 alone
FC1 is exact: token b is the unit vector b, so that h[j][b] = relu(w_up[j][b] + b_up[j]), rounded
once to 32 bits."""
import math

import pytest
import torch


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


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 5, 8])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 511, 512, 1000, 1024])
@pytest.mark.parametrize("d", [96, 2056, 2080])
def test_fc2_batch_list_lengths(pf, d, n, B):
    y, ref, tol = _case(pf, d, 1024, n, B, spread=0.0)
    assert bool(((y - ref).abs() <= tol).all()), float(((y - ref).abs() - tol).max())


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 7])
@pytest.mark.parametrize("spread", [4.0, 12.0])
def test_fc2_batch_fc1_outputs_beyond_the_halves(pf, spread, B):
    """Values up to 10^12 (far above the largest half) beside values down to 10^-12."""
    y, ref, tol = _case(pf, 256, 4096, 3000, B, spread)
    assert bool(((y - ref).abs() <= tol).all())


@pytest.mark.gpu
def test_fc2_batch_infinite_fc1_output(pf):
    """An infinite FC1 output makes every column infinite with the sign of its weight."""
    b = torch.ones(1024, device="cuda")
    b[70] = float("inf")
    y, ref, _ = _case(pf, 64, 1024, 1024, 5, 0.0, up_scale=0.0, b_up=b)
    assert bool((y == ref).all())


# ---- FC2 alone -----------------------------------------------------------------------------

def _fc2_inputs(kind, n, d, B, seed=0):
    """w_up [n][B] half, b_up [n], w_down [n][d] half, and h [n][B] in 64 bits."""
    g = torch.Generator().manual_seed(7919 * seed + 31 * n + d + B)
    rnd = lambda *s: torch.randn(*s, generator=g)
    uni = lambda *s: 0.5 + torch.rand(*s, generator=g)
    off = torch.where(torch.rand(n, B, generator=g) < 0.3, -1.0, 0.0)   # switches a neuron off for a token
    w_up, b_up, w_down = torch.zeros(n, B), rnd(n) * 0.1, rnd(n, d) / math.sqrt(d)
    if kind == "relu":
        w_up = rnd(n, B)
    elif kind == "tiny":        # all below the smallest half
        w_up, b_up = off, 1e-12 * uni(n)
    elif kind == "grow":        # each chunk larger than the one before
        b_up = 10.0 ** (torch.arange(n).double() / n * 30 - 15).float() * uni(n)
    elif kind in ("gap30", "gap45", "gap100"):
        # one row in 16 is far larger than the others and has no weight in the even columns
        w_up, b_up = off, 2.0 ** -int(kind[3:]) * uni(n)
        b_up[5::16] = uni(b_up[5::16].numel())
        w_down[5::16, ::2] = 0.0
    w_up, b_up, w_down = w_up.half(), b_up.float(), w_down.half()
    h = torch.relu(w_up.float() + b_up[:, None]).double()
    return w_up, b_up, w_down, h


def _fc2_within(y, h, w_down, split):
    """Whether y [B][d] is h^T w_down as 32-bit sums give it.  On its way into a column of the
    result a product is rounded at most R times: 4 + 3 inside a chunk, once per chunk of its wave
    (8 waves and `split` row groups share the chunks), 4 in the sum of the 16 partial sums, then
    the row groups.  Each rounding is at most 2^-24 of a partial sum, i.e. of sum |h| |w|; the
    matrix cores also drop what lies 2^-24 below the largest of each 8 products, 8 more such
    steps at most.  In the 2-norm the roundings add up like independent errors."""
    ref, mag = h.T @ w_down.double(), h.T @ w_down.double().abs()
    R = 4 + 3 + math.ceil(h.shape[0] / (512.0 * split)) + 4 + split
    err = y - ref
    for cols in (slice(0, None, 2), slice(1, None, 2)):     # the "gap" inputs differ in these
        if float(err[:, cols].norm()) > math.sqrt(R) * 2.0 ** -24 * float(ref[:, cols].norm()):
            return False
    return bool((err.abs() <= (R + 8) * 2.0 ** -24 * mag).all())


def _fc2_run(pf, w_up, b_up, w_down, B, split=0, vector=False):
    n, d = w_down.shape
    ffn = (n + 63) // 64 * 64 + 64
    pad = lambda t: torch.cat([t, torch.zeros(ffn - n, *t.shape[1:], dtype=t.dtype)])
    wu = torch.zeros(ffn, d, dtype=torch.half)
    wu[:, :B] = pad(w_up)
    x = torch.zeros(B, d, device="cuda")
    for b in range(B):
        x[b, b] = 1.0
    ctx = pf.Context(d, ffn, 64, max_batch=B)
    ctx.set_option(pf.OPT_DOWN_SPLIT, split)
    if vector:
        ctx.set_option(pf.OPT_MFMA_MIN_BATCH, B + 1)
    L = pf.Layer(ctx, d, ffn, 64, w_up=wu.cuda(), w_down=pad(w_down).cuda(), b_up=pad(b_up).cuda(),
                 b_down=torch.zeros(d, device="cuda"), p1=torch.zeros(64, d, dtype=torch.half, device="cuda"),
                 p2=torch.zeros(ffn, 64, dtype=torch.half, device="cuda"))
    idx = torch.arange(ffn, dtype=torch.int32, device="cuda")
    count = torch.tensor([n], dtype=torch.int32, device="cuda")
    y = torch.full((B, d), float("nan"), device="cuda")
    ctx.sparse_ffn(L, x, idx, count, y)
    torch.cuda.synchronize()
    return y.cpu()


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 5, 8])
@pytest.mark.parametrize("n", [1, 64, 65, 300, 768, 769, 1000, 4100])
@pytest.mark.parametrize("d", [32, 96, 2080])
def test_fc2_alone_list_lengths(pf, d, n, B):
    w_up, b_up, w_down, h = _fc2_inputs("relu", n, d, B)
    for split in (0, 1, 3):
        y = _fc2_run(pf, w_up, b_up, w_down, B, split)
        assert _fc2_within(y.double(), h, w_down, split or 4), split
    if n >= 300:    # FC1 is exact in every form, so equal bits mean the vector FC2: at batch 4 for
        # lists of at most 256 rows per row group, else never
        assert torch.equal(y, _fc2_run(pf, w_up, b_up, w_down, B, 3, vector=True)) == (B == 4 and n <= 768)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["tiny", "grow", "gap30", "gap45", "gap100"])
@pytest.mark.parametrize("B", [4, 7])
def test_fc2_alone_ranges(pf, B, kind):
    """Whatever the range of h, each column is as accurate as the terms that it is made of: small
    values beside large ones that have no weight in the column keep their 24 bits."""
    w_up, b_up, w_down, h = _fc2_inputs(kind, 1500, 96, B)
    for split in (0, 1):
        assert _fc2_within(_fc2_run(pf, w_up, b_up, w_down, B, split).double(), h, w_down, split or 4), split


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 8])
@pytest.mark.parametrize("n", [300, 1500, 4100])
def test_fc2_alone_no_less_accurate_than_the_vector_form(pf, n, B):
    """The matrix cores take the place of 32-bit vector arithmetic: their error against 64 bits must
    not be larger.  Mean over seeds; the vector form's own spread between seeds is 2 %."""
    err = {False: 0.0, True: 0.0}
    for seed in range(4):
        w_up, b_up, w_down, h = _fc2_inputs("relu", n, 768, B, seed)
        ref = h.T @ w_down.double()
        for vector in err:
            y = _fc2_run(pf, w_up, b_up, w_down, B, 4, vector)
            err[vector] += float((y.double() - ref).norm() / ref.norm())
    assert err[False] <= 1.02 * err[True], err


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 8])
def test_fc2_alone_infinite_weights_and_outputs(pf, B):
    """An infinite weight or FC1 output makes a column infinite, with the sign of the product; where
    the other factor is zero, or infinities of both signs meet, it is NaN.  The rest stays finite."""
    inf = float("inf")
    w_up, b_up, w_down, h = _fc2_inputs("relu", 1500, 96, B)
    w_down[7, 3], w_down[700, 20], w_down[1400, 20], w_down[900, 50] = inf, -inf, inf, inf
    w_up[7], b_up[7] = 1.0, 2.0 ** -9           # 8 bits: the last part of h is zero
    w_up[700], b_up[700] = 1.0, 0.3
    w_up[1400], b_up[1400] = 1.0, 0.3
    w_up[900, ::2], w_up[900, 1::2] = -9.0, 2.0  # off for every other token
    h = torch.relu(w_up.float() + b_up[:, None]).double()
    for case in range(2):
        if case:
            b_up[33] = inf
            w_down[33, 5] = 0.0
            h = torch.relu(w_up.float() + b_up[:, None]).double()
        ref = torch.stack([(h[:, b:b + 1] * w_down.double()).sum(0) for b in range(B)])
        fin = torch.isfinite(ref)
        for split in (0, 1):
            y = _fc2_run(pf, w_up, b_up, w_down, B, split).double()
            assert torch.equal(torch.isnan(y), torch.isnan(ref))
            assert torch.equal(y[torch.isinf(ref)], ref[torch.isinf(ref)])
            torch.testing.assert_close(y[fin], ref[fin], rtol=0, atol=40 * 2.0 ** -24 * float(h.sum()))


@pytest.mark.parametrize("kind,n,d,B", [("relu", 1, 32, 4), ("relu", 65, 96, 5), ("relu", 4100, 2080, 8),
                                        ("tiny", 1500, 96, 4), ("grow", 1500, 96, 4), ("gap30", 1500, 96, 4),
                                        ("gap45", 1500, 96, 7), ("gap100", 1500, 96, 7)])
def test_fc2_bound_sees_lost_bits(kind, n, d, B):
    """The bound of the tests above accepts 32-bit sums and refuses h cut to 16 bits, h rounded to
    2^-34 of the largest (the "gap" inputs) and a kernel that adds nothing."""
    _, _, w_down, h = _fc2_inputs(kind, n, d, B)
    wd = w_down.double()
    sums = [(h[c:c + 64].T @ wd[c:c + 64]).float() for c in range(0, n, 64)]
    for c in range(1, len(sums)):
        sums[c] += sums[c - 1]
    assert _fc2_within(sums[-1].double(), h, w_down, 1) or len(sums) > 30     # one long chain
    assert not _fc2_within(torch.zeros(B, d).double(), h, w_down, 1)
    m, e = torch.frexp(h)
    cut = torch.ldexp(torch.floor(m * 2 ** 16) / 2 ** 16, e)
    assert not _fc2_within(cut.T @ wd, h, w_down, 1)
    if kind.startswith("gap"):
        step = float(h.max()) * 2.0 ** -34
        assert not _fc2_within((torch.round(h / step) * step).T @ wd, h, w_down, 1)
