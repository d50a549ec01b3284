"""Pre-activations of large layers next to zero: their sign is that of the 64-bit sum at the edges of the matrix, beside rows of
any size (zeros among them, with and without a bias) and where sums cancel; a row's bits do not depend on other rows.

Planted values lie within 1e-7 of zero or less for |x| |w| of 10 to 300, a hundredth of the error of an fp32 or a split
sum, so that a product's own sign is right for half of them."""
import math

import numpy as np
import pytest
import torch

import paper_2402_14212_amd as mw

pytestmark = pytest.mark.gpu


def bits_of(words, n):
    e = np.arange(n)
    return ((words[e // 64] >> (e % 64).astype(np.uint64)) & np.uint64(1)).astype(bool)


def generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def orthonormal(d_in, d_out, gen):
    return torch.linalg.qr(torch.randn(d_in, d_out, device="cuda", generator=gen))[0].t().contiguous()


def plant(x, W, rows, cols):
    """x with x[rows[i]] moved along W[cols[i]] (rows of W orthonormal) until the product of the two is a rounding error."""
    y = x.clone()
    z = (y[rows].double() * W[cols].double()).sum(1)
    y[rows] = (y[rows].double() - z[:, None] * W[cols].double()).float()
    return y


def dense_signs(W, b, x, t):
    net = mw.MoonwalkNet([W], [b], [0.3], x.shape[0])
    net.moonwalk_grad(x, t)
    assert net.memory_stats()["sign_mismatches"] == 0      # Phase III formed the same signs
    return bits_of(net.fetch_mask(0), x.shape[0] * W.shape[0]).reshape(x.shape[0], -1)


@pytest.mark.parametrize("widths,batch", [((2301, 2100), 1025), ((2048, 2049), 1025), ((2304, 2176), 1027)])
def test_last_rows_and_columns_of_a_dense_layer(widths, batch):
    """Tiles of which a few rows or columns lie in the matrix."""
    gen = generator(batch)
    d_in, d_out = max(widths), min(widths)
    W = orthonormal(d_in, d_out, gen)
    x, t = torch.randn(batch, d_in, device="cuda", generator=gen), torch.randn(batch, d_out, device="cuda", generator=gen)
    b = torch.zeros(d_out, device="cuda")
    cols = torch.cat([torch.arange(0, d_out - 8, 16, device="cuda"), torch.arange(d_out - 8, d_out, device="cuda")])
    s = (x[batch - 1].double()[None] * W[cols].double()).sum(1)
    b[cols] = -(s.float() + 2.0 * torch.abs(s.float()) * 2.0 ** -23 * torch.where(cols % 32 == 0, 1.0, -1.0))
    got = dense_signs(W, b, x, t)
    z = (x.double() @ W.double().t().contiguous() + b.double()).cpu().numpy()
    assert np.array_equal(got[-1, cols.cpu().numpy()], z[-1, cols.cpu().numpy()] > 0)
    assert np.array_equal(got[z != 0], (z > 0)[z != 0])


@pytest.mark.parametrize("bias", [None, 0.0, 0.1])
@pytest.mark.parametrize("zeros", [1, 30])
def test_beside_samples_of_zeros(bias, zeros):
    """`zeros` zero samples in every 32: they are not taken for values next to zero, and their neighbours are."""
    gen = generator(zeros)
    B, d_in, d_out = 1024, 2304, 2176
    W = orthonormal(d_in, d_out, gen)
    x, t = torch.randn(B, d_in, device="cuda", generator=gen), torch.randn(B, d_out, device="cuda", generator=gen)
    live = torch.arange(B, device="cuda")[torch.arange(B, device="cuda") % 32 >= zeros]
    cols = torch.arange(len(live), device="cuda") * 41 % d_out
    b = None if bias is None else bias * torch.randn(d_out, device="cuda", generator=gen)
    if bias:
        b[cols] = 0.0       # (the planted ones are next to zero without it)
    x = plant(x, W, live, cols)
    dead = torch.ones(B, dtype=torch.bool, device="cuda")
    dead[live] = False
    x[dead] = 0
    got = dense_signs(W, b, x, t)
    z = (x.double() @ W.double().t().contiguous()) + (0.0 if b is None else b.double())
    rows, at = live.cpu().numpy(), cols.cpu().numpy()
    z = z.cpu().numpy()
    assert np.array_equal(got[rows, at], z[rows, at] > 0)
    assert np.array_equal(got[dead.cpu().numpy()], z[dead.cpu().numpy()] > 0)


def by_row(x, w, b=None):
    """Rows times a matrix through the forward product of a 1 x 1 convolution: activations (slope one: the sums) and signs."""
    y, mask = mw.conv_forward(x.reshape(1, x.shape[0], 1, x.shape[1]), w.reshape(1, 1, *w.shape), b, 1, 0, 0, alpha=1.0, want_mask=True)
    y = y.reshape(x.shape[0], w.shape[1])
    return y, bits_of(mask.cpu().numpy().view(np.uint64), y.numel()).reshape(y.shape[0], -1)


ROWS, K, N = 25600, 1152, 128     # 200 tiles of 128 x 128


@pytest.mark.parametrize("kind", ["sizes", "tiny", "small", "large", "late", "common", "ends", "groups"])
def test_rows_of_any_kind(kind):
    """Row sizes from 2^-20 to 2^20 of their neighbours', or so small beside them that their squares underflow; all of them as small or
    as large as activations of deep networks become; columns of which the first are 2^40 smaller; sums whose halves cancel; two
    terms 30 times the others; 16 k of one sign and 16 of the other in turn (which the two groups of K each add up)."""
    gen = generator(len(kind))
    x = torch.randn(ROWS, K, device="cuda", generator=gen)
    W = torch.randn(N, K, device="cuda", generator=gen)
    k = torch.arange(K, device="cuda")
    if kind == "common":
        x, W = 1 + 0.1 * x, torch.where(k < K // 2, 1.0, -1.0) * (1 + 0.1 * W)
    elif kind == "late":
        x[:, :40] *= 2.0 ** -40
    elif kind == "ends":
        x[:, 0] = x[:, -1] = 30.0
        W[:, 0], W[:, -1] = 30.0, -30.0
    elif kind == "groups":
        x, W = x.abs(), torch.where(k // 16 % 2 == 0, 1.0, -1.0) * W.abs()
    rows = torch.arange(0, ROWS, 5, device="cuda")
    cols = rows // 5 * 37 % N
    for _ in range(2):                      # next to zero, but for the rounding of x
        w = W[cols].double()
        v = w * (k >= 40) if kind == "late" else w
        x[rows] = (x[rows].double() - (x[rows].double() * w).sum(1, keepdim=True) * v / v.pow(2).sum(1, keepdim=True)).float()
    if kind == "sizes":
        x *= torch.exp2(torch.randint(-20, 21, (ROWS, 1), device="cuda", generator=gen).float())
    if kind in ("small", "large"):
        x *= 2.0 ** (-90 if kind == "small" else 90)
    if kind == "tiny":                      # (tiles with such rows are formed again in fp32, with fp32's own signs)
        x[ROWS // 2::7] *= 2.0 ** -80
        keep = rows < ROWS // 2
        rows, cols = rows[keep], cols[keep]
    w = W.t().contiguous()
    y, got = by_row(x, w)
    z = x.double() @ w.double()
    bound = 4e-8 * math.sqrt(K) * x.double().norm(dim=1)[:, None] * w.double().norm(dim=0)[None]
    assert ((y.double() - z).abs() <= bound).all()
    assert np.array_equal(got, (y > 0).cpu().numpy())
    rows, at, z = rows.cpu().numpy(), cols.cpu().numpy(), z.cpu().numpy()
    assert np.array_equal(got[rows, at], z[rows, at] > 0)


def test_rows_that_leave_the_range_of_the_squares():
    """Rows of 2^20 to 2^70 of their neighbours' size, infinities and NaN in some: every finite row within an fp32 sum's error of the
    64-bit one, every other as infinite or NaN as IEEE says, signs those of the values."""
    gen = generator(9)
    x = torch.randn(ROWS, K, device="cuda", generator=gen) * torch.exp2(torch.randint(0, 2, (ROWS, 1), device="cuda", generator=gen)
                                                                        * torch.randint(20, 71, (ROWS, 1), device="cuda", generator=gen).float())
    w = torch.randn(K, N, device="cuda", generator=gen) * 2.0 ** 20
    x[100:ROWS // 2:997, 5] = float("inf")
    x[101:ROWS // 2:1499, 7] = float("nan")
    y, got = by_row(x, w)
    odd = ~torch.isfinite(x).all(1)
    z = x.double() @ w.double()
    bound = 4 * math.sqrt(K) * 2.0 ** -24 * x.double().norm(dim=1)[:, None] * w.double().norm(dim=0)[None]
    assert ((y.double() - z).abs() <= bound)[~odd].all()
    ref = torch.where(torch.isnan(x).any(1)[:, None], float("nan"), float("inf") * torch.sign(w[5])[None].double()).expand(ROWS, N)[odd]
    assert torch.equal(torch.isnan(y[odd]), torch.isnan(ref)) and torch.equal(torch.nan_to_num(y[odd].double()), torch.nan_to_num(ref))
    assert np.array_equal(got, (y > 0).cpu().numpy())


def test_a_row_does_not_depend_on_the_others():
    gen = generator(5)
    W = orthonormal(K, N, gen)
    live = torch.arange(0, ROWS, 3, device="cuda")
    x = plant(torch.randn(ROWS, K, device="cuda", generator=gen), W, live, live // 3 % N)
    others = torch.ones(ROWS, dtype=torch.bool, device="cuda")
    others[live] = False
    w = W.t().contiguous()
    y = by_row(x, w)[0]
    for change in (0.0, 2.0 ** -10, 2.0 ** 12):
        v = x.clone()
        v[others] *= change
        assert torch.equal(by_row(v, w)[0][live], y[live]), change


def test_weights_of_mostly_zeros():
    """Every other column of the weights a unit vector, inputs half zeros: thousands of sums that are exactly zero beside planted ones in
    dense columns. The former are the inputs themselves, the latter keep the sign of the 64-bit sum (but for one in
    a hundred that comes out as exactly zero too)."""
    gen = generator(10)
    W = orthonormal(K, N, gen)
    W[::2] = torch.eye(K, device="cuda")[: N // 2]
    x = torch.relu(torch.randn(ROWS, K, device="cuda", generator=gen))
    rows = torch.arange(0, ROWS, 7, device="cuda")
    cols = rows // 7 * 2 % N + 1
    keep = x[rows][:, : N // 2].clone()
    V = W.clone()
    V[:, : N // 2] = 0      # (moved along the part of the column that the unit vectors do not see)
    for _ in range(3):
        v = V[cols].double()
        x[rows] = (x[rows].double() - (x[rows].double() * W[cols].double()).sum(1, keepdim=True) * v / v.pow(2).sum(1, keepdim=True)).float()
    assert torch.equal(x[rows][:, : N // 2], keep)
    y, got = by_row(x, W.t().contiguous())
    assert torch.equal(y[:, ::2], x[:, : N // 2])
    z = (x[rows].double() * W[cols].double()).sum(1).cpu().numpy()
    some = (y[rows, cols] != 0).cpu().numpy()
    assert some.mean() > 0.95
    assert np.array_equal(got[rows.cpu().numpy(), cols.cpu().numpy()][some], (z > 0)[some])
    assert np.array_equal(got, (y > 0).cpu().numpy())


def test_sums_that_cancel_all_over():
    """Rows at right angles to all of W: every value is next to zero, the tile is formed again in fp32. No worse than that."""
    gen = generator(6)
    W = orthonormal(K, N, gen)
    x = torch.randn(ROWS, K, device="cuda", generator=gen)
    part = torch.arange(ROWS, device="cuda") % 2 == 0
    for _ in range(2):
        x[part] = (x[part].double() - (x[part].double() @ W.double().t().contiguous()) @ W.double()).float()
    w = W.t().contiguous()
    y, got = by_row(x, w)
    z = x.double() @ w.double()
    size = x.double().norm(dim=1)[:, None] * w.double().norm(dim=0)[None]
    assert ((y.double() - z).abs() <= 4 * math.sqrt(K) * 2.0 ** -24 * size).all()
    assert np.array_equal(got, (y > 0).cpu().numpy())


def test_last_rows_and_channels_of_a_convolution():
    """31 images of 31 x 31: 29791 rows, 96 channels: the last of 128 x 128 tiles hold 95 rows, all of them 96 columns."""
    gen = generator(7)
    B, side, C = 31, 31, 96
    x = torch.randn(B, side, side, C, device="cuda", generator=gen)
    w = torch.randn(3, 3, C, C, device="cuda", generator=gen) / math.sqrt(9 * C)
    pad = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    P = torch.cat([pad[:, u:u + side, v:v + side] for u in range(3) for v in range(3)], 3).reshape(-1, 9 * C)
    chans = torch.arange(7, C, 8, device="cuda")
    rows = P.shape[0] - 1 - chans // 8 % 5
    s = (P[rows] * w.reshape(9 * C, C)[:, chans].t().double()).sum(1)
    b = 0.1 * torch.randn(C, device="cuda", generator=gen)
    b[chans] = -(s.float() + 2.0 * torch.abs(s.float()) * 2.0 ** -23 * torch.where(chans // 8 % 2 == 0, 1.0, -1.0))
    z = (P @ w.reshape(9 * C, C).double() + b.double()).cpu().numpy()
    y, mask = mw.conv_forward(x, w, b, 1, 1, 1, alpha=0.3, want_mask=True)
    got = bits_of(mask.cpu().numpy().view(np.uint64), z.size).reshape(-1, C)
    rows, chans = rows.cpu().numpy(), chans.cpu().numpy()
    assert np.array_equal(got[rows, chans], z[rows, chans] > 0)
    assert np.array_equal(got[z != 0], (z > 0)[z != 0])


def test_signs_below_the_rounding_of_the_sum():
    """Biases that are the rounded sum itself, negated: what is left is less than half a unit in the last place of the sum."""
    gen = generator(8)
    W = orthonormal(K, N, gen)
    x = torch.randn(ROWS, K, device="cuda", generator=gen)
    cols = torch.arange(N, device="cuda")
    rows = cols * 199 + 3
    s = (x[rows].double() * W.double()).sum(1)
    b = -s.float()
    _, got = by_row(x, W.t().contiguous(), b)
    rows, cols, left = rows.cpu().numpy(), cols.cpu().numpy(), (s + b.double()).cpu().numpy()
    assert np.array_equal(got[rows, cols], left > 0)
