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


def input_cotangent(mw, shape, ct, w):
    B, H, W, Ci, Co, k, s, p = shape
    h = mw.conv_input_cotangent(torch.from_numpy(ct).cuda(), torch.from_numpy(w).cuda(), (H, W), s, p, p)
    return h.cpu().numpy()


def check_input_cotangent(mw, shape, ct, w):
    print("input cotangent", shape, flush=True)
    B, H, W, Ci, Co, k, s, p = shape
    got = input_cotangent(mw, shape, ct, w)
    ct64, w64 = ct.astype(np.float64), w.astype(np.float64)
    want = CO.conv2d_input_grad(ct64, w64, s, p, (H, W))
    terms = Co * ((k + s - 1) // s) ** 2   # of the class with the most taps
    bound = terms * 2.0 ** -24 * CO.conv2d_input_grad(np.abs(ct64), np.abs(w64), s, p, (H, W)) + 2.0 ** -149
    assert (np.abs(got - want) <= bound).all(), float((np.abs(got - want) / bound).max())
    return got


# B, H, W, C_in, C_out, k, s, p: the tile the input cotangent takes
REV = [(2, 64, 64, 64, 64, 3, 1, 1),      # 64 x 64
       (6, 50, 51, 64, 128, 5, 3, 2),     # 64 x 64, nine stride classes, odd width
       (5, 58, 59, 32, 32, 5, 1, 2),      # 64 x 64 on four wavefronts, 32 channels
       (4, 65, 66, 64, 96, 3, 1, 1),      # the same, 96 channels on the long side
       (3, 75, 74, 128, 128, 3, 1, 1),    # 128 x 128
       (6, 63, 64, 128, 128, 3, 2, 1)]    # 128 x 128, four stride classes
# the tile and slices of the weight gradient
DW = [(1, 13, 17, 32, 64, 3, 1, 1),       # 64 x 64, one slice
      (5, 29, 31, 96, 64, 3, 2, 1),       # 64 x 64, several slices, the last one short
      (9, 61, 63, 128, 128, 3, 2, 1),     # 128 x 128, several slices
      (4, 40, 43, 64, 96, 5, 3, 2)]


def unfavourable(kind, rng, x):
    """An image whose values differ by many powers of two from position to position."""
    B, H, W, C = x.shape
    if kind == "empty_start":      # nothing in the first half of every image, large values after it
        x[:, :H // 2] = 0
        x[:, H // 2:] *= np.float32(2.0 ** 20)
    elif kind == "tiny_start":     # the first image far below the others
        x[0] *= np.float32(2.0 ** -30)
    elif kind == "positions":
        x *= (2.0 ** rng.integers(-20, 21, (B, H, W, 1))).astype(np.float32)
    else:                          # channels, undone by the other operand
        x *= (2.0 ** rng.integers(-20, 21, C)).astype(np.float32)
    return x


KINDS = ["plain", "empty_start", "tiny_start", "positions", "channels"]


@pytest.mark.parametrize("shape", REV)
@pytest.mark.parametrize("kind", KINDS)
def test_input_cotangent_of_unfavourable_images(mw, shape, kind):
    rng, _, w, ct = draw(shape, 5)
    if kind != "plain":
        before = ct.copy()
        unfavourable(kind, rng, ct)
        if kind == "channels":
            w = (w * (before / ct)[0, 0, 0]).astype(np.float32)
    check_input_cotangent(mw, shape, ct, w)


@pytest.mark.parametrize("shape", DW)
@pytest.mark.parametrize("kind", KINDS[:-1])
def test_weight_gradient_of_unfavourable_images(mw, shape, kind):
    rng, x, _, ct = draw(shape, 6)
    if kind != "plain":
        unfavourable(kind, rng, x)
        if kind == "positions":    # samples of very different cotangents, each unit off for half of them
            ct *= (rng.random(ct.shape) < 0.5)
            ct *= (2.0 ** rng.integers(-20, 1, ct.shape[:3] + (1,))).astype(np.float32)
    check_weight_gradient(mw, shape, x, ct)


@pytest.mark.parametrize("shape", REV)
def test_input_cotangent_of_values_that_do_not_fit(mw, shape):
    """Infinities, NaN and sums that overflow on split operands: computed again on fp32 instructions, where they belong and
    nowhere else."""
    B, H, W, Ci, Co, k, s, p = shape
    _, _, w, ct = draw(shape, 7)
    clean = input_cotangent(mw, shape, ct, w)
    bad = np.zeros(ct.shape[:3], bool)
    for (b, i, j), v in (((0, 3, 5), np.inf), ((B - 1, 0, 0), np.nan), ((B - 1, ct.shape[1] - 1, ct.shape[2] - 1), 2e38)):
        ct[b, i, j, 7] = v
        bad[b, i, j] = True
    got = input_cotangent(mw, shape, ct, w)
    reach = CO.conv2d_input_grad(bad[..., None].astype(np.float64), np.ones((k, k, 1, 1)), s, p, (H, W))[..., 0] > 0
    assert reach.any() and np.array_equal(got[~reach], clean[~reach])
    near = np.zeros(ct.shape[:3] + (1,))
    near[0, 3, 5] = 1
    at_inf = CO.conv2d_input_grad(near, np.ones((k, k, 1, 1)), s, p, (H, W))[..., 0] > 0
    assert np.isinf(got[at_inf]).all()
    with np.errstate(all="ignore"):
        ct[0, 3, 5, 7], ct[B - 1, 0, 0, 7] = 0, 0
        want = CO.conv2d_input_grad(ct.astype(np.float64), w.astype(np.float64), s, p, (H, W))
    large = (np.abs(want) > 1e30) & (np.abs(want) < 3e38)
    assert large.any() and np.allclose(got[large], want[large], rtol=1e-5)


@pytest.mark.parametrize("shape", DW)
def test_weight_gradient_of_values_that_do_not_fit(mw, shape):
    B, H, W, Ci, Co, k, s, p = shape
    _, x, _, ct = draw(shape, 8)
    clean = weight_gradient(mw, shape, x, ct)
    middle = (0, ct.shape[1] // 2, ct.shape[2] // 2)   # every tap reads inside the image there
    ct[middle][3], ct[middle][9], ct[middle][17] = np.inf, np.nan, 1e30
    got = weight_gradient(mw, shape, x, ct)
    rest = np.setdiff1d(np.arange(Co), [3, 9, 17])
    assert np.array_equal(got[..., rest], clean[..., rest])
    assert np.isinf(got[..., 3]).all() and np.isnan(got[..., 9]).all()
    want = CO.conv2d_weight_grad(x.astype(np.float64), ct.astype(np.float64)[..., 17:18], k, s, p)[..., 0]
    assert np.allclose(got[..., 17], want, rtol=1e-5, atol=1e25)


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
