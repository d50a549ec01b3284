"""The 32 x 32 tile of four 16 x 16 wavefronts: the bits of the 64 x 64 tile, at edges of its tiles, of its slices of 32 k and
of its stages of four slices, aligned and not, in every layout and through the sign packing of 16-wide rows."""
import pytest
import torch

import paper_2402_14212_amd as mw

pytestmark = pytest.mark.gpu

OPS = {"NT": mw.GEMM_NT, "NN": mw.GEMM_NN, "TN": mw.GEMM_TN}


@pytest.mark.parametrize("K", [1, 5, 31, 32, 33, 64, 100, 127, 128, 129, 160, 224, 255])
@pytest.mark.parametrize("op", ["NT", "NN", "TN"])
def test_bits_of_the_64_tile(op, K):
    # below K = 256 the automatic choice is the small tile up to 128 tiles of 64 x 64
    for M, N in [(1, 4), (15, 17), (32, 32), (33, 65), (100, 64), (257, 300)]:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(M * N + K)
        A = torch.randn((K, M) if op == "TN" else (M, K), device="cuda", generator=gen)
        B = torch.randn((N, K) if op == "NT" else (K, N), device="cuda", generator=gen)
        A = A * torch.exp2(torch.randint(-10, 11, A.shape, device="cuda", generator=gen).float())
        got, ref = mw.gemm_f32(OPS[op], A, B), mw.gemm_f32(OPS[op], A, B, tile=mw.TILE_64)
        assert torch.equal(got, ref), (op, M, N, K)


@pytest.mark.parametrize("K", [256, 257, 287, 300, 383, 384, 385, 511, 513, 640, 767, 769, 1000, 1023, 1024])
@pytest.mark.parametrize("op", ["NT", "NN", "TN"])
def test_bits_of_the_tile_that_splits_k(op, K):
    """From K = 256 to 1024, up to 128 tiles of 32 x 32, the automatic choice is the 16 x 16 tile with K split over four
    wavefronts: the bits of the 32 x 32 tile with that split."""
    for M, N in [(1, 4), (15, 17), (16, 16), (33, 65), (100, 389), (128, 1024), (129, 31)]:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(M * N + K)
        A = torch.randn((K, M) if op == "TN" else (M, K), device="cuda", generator=gen)
        B = torch.randn((N, K) if op == "NT" else (K, N), device="cuda", generator=gen)
        A = A * torch.exp2(torch.randint(-10, 11, A.shape, device="cuda", generator=gen).float())
        got, ref = mw.gemm_f32(OPS[op], A, B), mw.gemm_f32(OPS[op], A, B, tile=mw.TILE_32K4)
        assert torch.equal(got, ref), (op, M, N, K)


@pytest.mark.parametrize("side,c_in,c_out,k,stride", [(9, 32, 32, 1, 1), (17, 96, 64, 3, 2), (23, 64, 96, 5, 2), (12, 128, 32, 3, 1)])
def test_layer_of_a_small_batch(side, c_in, c_out, k, stride):
    """A layer of few images takes the small tile, many copies of them the large ones: the same image, the same bits. Only where
    neither splits K (channels that are no multiple of 128), and for the forward product of up to 64 channels, or up to 191
    tiles of 128 x 128, which is fp32 in every tile."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(side)
    x = torch.randn(2, side, side, c_in, device="cuda", generator=gen)
    w = torch.randn(k, k, c_in, c_out, device="cuda", generator=gen) / (k * k * c_in) ** 0.5
    b = torch.randn(c_out, device="cuda", generator=gen)
    y, mask = mw.conv_forward(x, w, b, stride, 0, 0, alpha=0.2, want_mask=True)
    many = 200 * 64 * 64 // y[0].numel() + 1
    assert c_out <= 64 or 2 * many * y[0].numel() // c_out < 191 * 128      # (else split operands)
    big, _ = mw.conv_forward(x.repeat(many, 1, 1, 1), w, b, stride, 0, 0, alpha=0.2, want_mask=True)
    if c_in % 64 or c_out % 64:      # (else the large batch may take a tile that splits K)
        assert torch.equal(big[:2], y) and torch.equal(big[-2:], y)
    z = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2).double().cpu(), w.permute(3, 2, 0, 1).double().cpu(), b.double().cpu(), stride)
    z = z.permute(0, 2, 3, 1)
    ref = torch.where(z > 0, z, 0.2 * z)
    assert ((y.cpu().double() - ref).norm() / ref.norm()).item() <= 4 * (k * k * c_in) ** 0.5 * 2.0 ** -24
    bits = (y.reshape(-1).cpu() > 0)
    words = mask.view(torch.int64).cpu()
    got = ((words[torch.arange(bits.numel()) // 64] >> (torch.arange(bits.numel()) % 64)) & 1).bool()
    assert torch.equal(got, bits)
