"""Gathered products on split operands (input cotangent and weight gradient of a convolution) against fp64, where they
can go wrong. Bound per element, that of an fp32 sum of K products in any order:
    |C - AB| <= K 2^-24 sum|a||b|
"""
import numpy as np
import pytest
import torch

from oracle import conv_oracle as CO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mw():
    import paper_2402_14212_amd as m
    m.load_library()
    return m


def draw(shape, seed):
    B, H, W, Ci, Co, k, s, p = shape
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, H, W, Ci)).astype(np.float32)
    w = (rng.standard_normal((k, k, Ci, Co)) / np.sqrt(k * k * Ci)).astype(np.float32)
    ct = rng.standard_normal((B, CO.out_size(H, k, s, p), CO.out_size(W, k, s, p), Co)).astype(np.float32)
    return rng, x, w, ct


def cuda(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def weight_gradient(mw, shape, x, ct):
    k, s, p = shape[5:]
    dw, _ = mw.conv_weight_grad(torch.from_numpy(x).cuda(), torch.from_numpy(ct).cuda(), k, k, s, p, p)
    return dw.cpu().numpy()


def check_weight_gradient(mw, shape, x, ct):
    print("weight gradient", shape, flush=True)
    k, s, p = shape[5:]
    got = weight_gradient(mw, shape, x, ct)
    x64, ct64 = x.astype(np.float64), ct.astype(np.float64)
    want = CO.conv2d_weight_grad(x64, ct64, k, s, p)
    bound = ct[..., 0].size * 2.0 ** -24 * CO.conv2d_weight_grad(np.abs(x64), np.abs(ct64), k, s, p) + 2.0 ** -149
    assert (np.abs(got - want) <= bound).all(), float((np.abs(got - want) / bound).max())
    return got


@pytest.mark.parametrize("rows", [1, 32, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("Ci,Co", [(32, 32), (96, 64), (128, 160)])
def test_weight_gradient_of_few_rows(mw, rows, Ci, Co):
    """fp32 tiles below 128 rows, split ones from there on; one slice of 256 rows, then two."""
    for k in (1, 3):
        shape = (1, 1 if k == 1 else rows, rows if k == 1 else 1, Ci, Co, k, 1, (k - 1) // 2)
        _, x, _, ct = draw(shape, rows)
        check_weight_gradient(mw, shape, x, ct)


def test_a_training_step_keeps_fp32_instructions(mw):
    """A layer whose one tap is the identity: ct_z is the output cotangent and the update of the entries below the diagonal
    is -lr x^T ct_z, bit for bit the product on fp32 instructions."""
    B, side, C, alpha, lr = 4, 8, 64, 0.25, 0.5
    rng = np.random.default_rng(2)
    x, t = cuda(*(rng.standard_normal((B, side, side, C)).astype(np.float32) for _ in range(2)))
    w, b = cuda(np.eye(C, dtype=np.float32)[None, None], np.zeros(C, np.float32))
    net = mw.ConvMoonwalkNet([w], [b], [alpha], B, side, side, 1, 0, plan=mw.PLAN_MOONWALK)
    net.sgd_step(x, t, lr)
    torch.cuda.synchronize()
    y, rows = torch.where(x > 0, x, alpha * x), B * side * side
    h, _ = mw.loss_grad(y.reshape(B, -1), t.reshape(B, -1), 1.0)
    ct = torch.where(x > 0, h.reshape(x.shape), alpha * h.reshape(x.shape))
    raw = mw.gemm_f32(mw.GEMM_TN, x.reshape(rows, C), ct.reshape(rows, C), tile=mw.TILE_64)
    below = torch.tril(torch.ones(C, C, device="cuda"), -1).bool()
    assert torch.equal(net.ws[0].reshape(C, C)[below], (-lr * raw)[below])
    net.close()
