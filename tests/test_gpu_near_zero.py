"""Pre-activations of large layers on split operands: what comes out next to zero is formed again in 64 bits, so that its sign
is that of the 64-bit value, the same in Phase I and Phase III, beside samples of zeros (which have the bias's sign; without a bias, at the
edges of the matrix and for rows of other sizes: test_gpu_preactivations.py).

Planted: biases that bring chosen pre-activations to a few units in the last place of the sum, a hundredth of the
rounding error of a sum of two thousand terms, on either side of zero."""
import math

import numpy as np
import pytest
import torch

import paper_2402_14212_amd as mw

pytestmark = pytest.mark.gpu


def planted(sums, ulps):
    """fp32 biases that leave sums[i] + bias = ulps[i] units in the last place of sums[i]."""
    s = sums.float()
    return -(s - ulps * torch.abs(s) * 2.0 ** -23)


def bits_of(words, n):
    e = np.arange(n)
    return (words[e // 64] >> (e % 64).astype(np.uint64)) & np.uint64(1)


@pytest.mark.parametrize("widths", [(2048, 2048), (2301, 2176)])
@pytest.mark.parametrize("zero_rows", [0, 300])
def test_signs_of_a_dense_layer(widths, zero_rows):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(widths[0] + zero_rows)
    d_in, d_out = widths
    B = 1024
    W = torch.linalg.qr(torch.randn(d_in, d_out, device="cuda", generator=gen))[0].t().contiguous()
    x = torch.randn(B, d_in, device="cuda", generator=gen)
    if zero_rows:
        x[:zero_rows] = 0
    t = torch.randn(B, d_out, device="cuda", generator=gen)
    cols = torch.arange(5, d_out, 64, device="cuda")
    rows = zero_rows + (cols * 37) % (B - zero_rows)
    s = (x[rows].double() * W[cols].double()).sum(1)
    ulps = torch.where(torch.arange(len(cols), device="cuda") % 2 == 0, 3.0, -3.0)
    b = 0.1 * torch.randn(d_out, device="cuda", generator=gen)
    b[cols] = planted(s, ulps)
    net = mw.MoonwalkNet([W], [b], [0.3], B)
    net.moonwalk_grad(x, t)
    stats = net.memory_stats()          # (raises where Phase III formed another sign)
    assert stats["sign_mismatches"] == 0
    got = torch.from_numpy(bits_of(net.fetch_mask(0), B * d_out).astype(np.int64).reshape(B, d_out)).cuda().bool()
    z = x.double() @ W.double().t() + b.double()
    assert torch.equal(got[rows, cols], z[rows, cols] > 0)
    # and all others, but for those within the last rounding: of the sum and of the sum with the bias
    sure = z.abs() > 2.0 ** -22 * (z.abs() + b.double().abs() + 1e-3)
    assert torch.equal(got[sure], (z > 0)[sure])


def test_signs_of_a_convolution():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    B, side, C = 24, 64, 128
    x = torch.randn(B, side, side, C, device="cuda", generator=gen)
    w = torch.randn(3, 3, C, C, device="cuda", generator=gen) / math.sqrt(9 * C)
    w[1, 1] = torch.tril(w[1, 1])
    w[1, 1].diagonal().fill_(1.0)
    so = (side - 1) // 2 + 1
    pad = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    P = torch.cat([pad[:, u:u + 2 * so - 1:2, v:v + 2 * so - 1:2] for u in range(3) for v in range(3)], 3).reshape(-1, 9 * C)
    chans = torch.arange(3, C, 16, device="cuda")
    rows = (chans * 911) % P.shape[0]
    s = (P[rows] * w.reshape(9 * C, C)[:, chans].t().double()).sum(1)
    b = torch.zeros(C, device="cuda")
    b[chans] = planted(s, torch.where(torch.arange(len(chans), device="cuda") % 2 == 0, 3.0, -3.0))
    z = P @ w.reshape(9 * C, C).double() + b.double()
    net = mw.ConvMoonwalkNet([w], [b], [0.3], B, side, side, 2, 1)
    net.moonwalk_grad(x, torch.randn(B, so, so, C, device="cuda", generator=gen))
    assert net.memory_stats()["sign_mismatches"] == 0
    got = torch.from_numpy(bits_of(net.fetch_mask(0), z.numel()).astype(np.int64).reshape(-1, C)).cuda().bool()
    assert torch.equal(got[rows, chans], z[rows, chans] > 0)
    sure = z.abs() > 2.0 ** -22 * (z.abs() + b.double().abs() + 1e-3)
    assert torch.equal(got[sure], (z > 0)[sure])
