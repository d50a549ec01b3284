"""Operands whose rows are no multiple of four floats long, or start anywhere: chunks that end inside a row, at the end of
the operand, and operands of less than one chunk. Against 64-bit products; the bound is that of fp32 sums,
sqrt(K) 2^-24 of the norm with a factor of four, and at least 2^-22."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2402_14212_amd as mw  # noqa: E402

SHAPES = [(1, 1, 1), (3, 2, 2), (2, 7, 5), (70, 33, 2), (130, 701, 3), (31, 5, 300), (5, 3, 1000), (33, 35, 257), (97, 130, 259),
          (100, 389, 701), (129, 131, 65), (200, 1201, 1403)]


def _operands(op, M, N, K, gap, gen):
    def one(r, c):
        # rows `gap` floats apart, what lies between them not a number: none of it may reach a result
        full = torch.full((r, c + gap), float("nan"), device="cuda")
        full[:, :c] = torch.randn(r, c, device="cuda", generator=gen)
        return full[:, :c]
    A = one(K, M) if op == "TN" else one(M, K)
    B = one(N, K) if op == "NT" else one(K, N)
    return A, B


@pytest.mark.parametrize("gap", [0, 1, 6])
@pytest.mark.parametrize("op", ["NT", "NN", "TN"])
def test_product_of_ragged_operands(op, gap):
    code = {"NT": mw.GEMM_NT, "NN": mw.GEMM_NN, "TN": mw.GEMM_TN}[op]
    for M, N, K in SHAPES:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(M + 1000 * N + K)
        A, B = _operands(op, M, N, K, gap, gen)
        ref = (A.double().t() if op == "TN" else A.double()) @ (B.double().t() if op == "NT" else B.double())
        for tile in (mw.TILE_AUTO, 1, 2, 3, 5, 6, 7):
            C = mw.gemm_f32(code, A, B, tile=tile)
            err = ((C.double() - ref).norm() / ref.norm()).item()
            assert err <= max(4 * math.sqrt(K) * 2.0 ** -24, 2.0 ** -22), (op, M, N, K, gap, tile, err)


@pytest.mark.parametrize("start", [1, 2, 3])
@pytest.mark.parametrize("op", ["NT", "NN", "TN"])
def test_operands_that_start_anywhere(op, start):
    """Rows of a multiple of four and not, every operand (and the result) `start` floats after a 16-byte boundary: the bits of
    aligned ones."""
    code = {"NT": mw.GEMM_NT, "NN": mw.GEMM_NN, "TN": mw.GEMM_TN}[op]

    def moved(t, gap):
        r, c = t.shape
        flat = torch.full((start + r * (c + gap),), float("nan"), device="cuda")
        view = flat[start:].reshape(r, c + gap)[:, :c]
        view.copy_(t)
        assert view.data_ptr() % 16 == 4 * start
        return view

    for M, N, K in [(3, 2, 2), (64, 64, 32), (33, 35, 257), (100, 388, 700), (129, 132, 64), (200, 1201, 1403), (1024, 2048, 512)]:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(M + 1000 * N + K)
        A = torch.randn((K, M) if op == "TN" else (M, K), device="cuda", generator=gen)
        B = torch.randn((N, K) if op == "NT" else (K, N), device="cuda", generator=gen)
        ref = mw.gemm_f32(code, A, B)
        for gap in (0, 4):
            got = mw.gemm_f32(code, moved(A, gap), moved(B, gap), C_out=moved(torch.zeros_like(ref), gap))
            assert torch.equal(got, ref), (op, start, M, N, K, gap)


@pytest.mark.parametrize("widths,batch", [((5, 3, 2, 1), 1), ((9, 7, 7), 3), ((66, 65, 35), 31), ((301, 299, 257), 33), ((515, 515, 259), 70)])
@pytest.mark.parametrize("alpha", [0.0, 0.3])
def test_ragged_network(widths, batch, alpha):
    """Moonwalk and backprop on the same ragged network: two ways to one gradient. Both take the signs of the same
    pre-activations, so they differ by rounding alone: at most 2^-24 a sum of K terms, times the growth of at most
    (0.3 + 1 / 0.3) / 2 < 2 a layer through the inverse, and the condition of the weights (singular values 0.8 .. 1.2)."""
    rng = np.random.default_rng(batch)
    Ws = []
    for a, b in zip(widths[:-1], widths[1:]):
        u, _, v = np.linalg.svd(rng.standard_normal((b, a)), full_matrices=False)
        Ws.append(torch.tensor((u * rng.uniform(0.8, 1.2, b)) @ v, dtype=torch.float32, device="cuda"))
    bs = [torch.tensor(0.01 * rng.standard_normal(b), dtype=torch.float32, device="cuda") for b in widths[1:]]
    x = torch.tensor(rng.standard_normal((batch, widths[0])), dtype=torch.float32, device="cuda")
    t = torch.tensor(rng.standard_normal((batch, widths[-1])), dtype=torch.float32, device="cuda")
    net = mw.MoonwalkNet(Ws, bs, [alpha] * len(Ws), batch)
    g = net.moonwalk_grad(x, t).flat.double()
    h = net.backprop_grad(x, t).flat.double()
    assert torch.isfinite(g).all()
    assert ((g - h).norm() <= 2e-5 * h.norm()).item()   # (a single sample may have no gradient at all)
    net.memory_stats()


@pytest.mark.parametrize("widths,batch,segment", [((70, 69, 67, 66, 65), 70, 0), ((300, 299, 288, 287, 64, 63), 45, 0), ((711, 700, 699), 129, 0),
                                                  ((1000, 999, 998, 997), 600, 0), ((130, 129, 128, 127, 125), 67, 2)])
@pytest.mark.parametrize("alpha", [0.0, 0.4])
def test_signs_packed_beside_the_next_layer(widths, batch, segment, alpha):
    """Widths that are and are not multiples of 32 in turn: the masks of a handle that packs them in launches of their own
    (one that keeps debugging buffers), bit for bit, padding included, and the same gradients."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(widths) + batch)
    Ws = [torch.linalg.qr(torch.randn(a, b, device="cuda", generator=gen))[0].t().contiguous() for a, b in zip(widths[:-1], widths[1:])]
    bs = [0.1 * torch.randn(b, device="cuda", generator=gen) for b in widths[1:]]
    x, t = torch.randn(batch, widths[0], device="cuda", generator=gen), torch.randn(batch, widths[-1], device="cuda", generator=gen)
    nets = [mw.MoonwalkNet(Ws, bs, [alpha] * len(Ws), batch, segment_length=segment, debug_keep=keep) for keep in (False, True)]
    grads = [net.moonwalk_grad(x, t).flat.clone() for net in nets]
    assert torch.equal(*grads)
    for i in range(len(Ws) if segment == 0 else segment):
        assert np.array_equal(nets[0].fetch_mask(i), nets[1].fetch_mask(i)), i
    nets[0].memory_stats()


@pytest.mark.parametrize("widths", [(1, 1), (3, 1), (3, 3, 1), (2, 1, 1)])
@pytest.mark.parametrize("alpha", [0.0, 0.3])
def test_weights_of_less_than_a_chunk_on_many_rows(widths, alpha):
    """Weights of one to three elements where the batch alone asks for the tiles of large outputs. Every weight is one or two in
    size, so that moonwalk and backprop differ by the rounding of the sums over the batch: 2^-24 sqrt(33000), twice."""
    batch = 33000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(widths))
    Ws = [torch.eye(b, a, device="cuda") * 2 - 0.5 for a, b in zip(widths[:-1], widths[1:])]
    bs = [torch.full((b,), 0.25, device="cuda") for b in widths[1:]]
    x, t = torch.randn(batch, widths[0], device="cuda", generator=gen), torch.randn(batch, widths[-1], device="cuda", generator=gen)
    net = mw.MoonwalkNet(Ws, bs, [alpha] * len(Ws), batch)
    g = net.moonwalk_grad(x, t).flat.double()
    h = net.backprop_grad(x, t).flat.double()
    assert net.memory_stats()["sign_mismatches"] == 0
    assert torch.isfinite(g).all() and ((g - h).norm() <= 5e-5 * h.norm()).item()


@pytest.mark.parametrize("d,batch", [(512, 128), (512, 129), (1000, 97), (992, 100), (991, 128), (1024, 100), (200, 140), (129, 300)])
def test_backprop_where_its_reverse_tile_changes(d, batch):
    """Both sides of the lines of the reverse product beside a weight gradient (rows, tiles, K), against
    the gradient in 64 bits with the signs of the handle's own pre-activations. Bound: sums of d or batch terms, four times."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + batch)
    Ws = [torch.linalg.qr(torch.randn(d, d, device="cuda", generator=gen))[0].contiguous() for _ in range(2)]
    bs = [0.1 * torch.randn(d, device="cuda", generator=gen) for _ in range(2)]
    x, t = torch.randn(batch, d, device="cuda", generator=gen), torch.randn(batch, d, device="cuda", generator=gen)
    net = mw.MoonwalkNet(Ws, bs, [0.3, 0.3], batch)
    net.moonwalk_grad(x, t)
    got = net.backprop_grad(x, t)
    ref, acts, slopes = [], [x.double()], []
    for i, (W, b) in enumerate(zip(Ws, bs)):
        words = net.fetch_mask(i)
        e = np.arange(batch * d)
        bits = torch.tensor(((words[e // 64] >> (e % 64).astype(np.uint64)) & np.uint64(1)).astype(bool), device="cuda").reshape(batch, d)
        slopes.append(torch.where(bits, 1.0, 0.3).double())
        acts.append((acts[-1] @ W.double().t().contiguous() + b.double()) * slopes[-1])
    h = (acts[-1] - t.double()) / batch
    for i in (1, 0):
        h = h * slopes[i]
        ref = [(h.t().contiguous() @ acts[i]).reshape(-1), h.sum(0)] + ref
        h = h @ Ws[i].double()
    ref = torch.cat(ref)
    bound = 4 * math.sqrt(max(d, batch)) * 2.0 ** -24
    assert ((got.flat.double() - ref).norm() <= bound * ref.norm()).item()
