"""Products on split operands (every fp32 value as a sum of parts) against fp64, where they can go wrong: edges of the
256 x 128, 128 x 128 and 64 x 64 tiles, short and odd K, unaligned leading dimensions, and operands whose magnitudes
differ by many powers of two, from row to row and along K.

Bound per element, that of an fp32 sum of K products in any order. It holds entry by entry: a large value that meets a
zero excuses nothing.
    |C - AB| <= K 2^-24 sum|a||b|
"""
import numpy as np
import pytest
import torch

from oracle import moonwalk_oracle as O
from workloads import make_mlp

from parity import check_moonwalk

pytestmark = pytest.mark.gpu

NT, NN, TN = 0, 1, 2


@pytest.fixture(scope="module")
def mw():
    import paper_2402_14212_amd as m
    m.load_library()
    return m


def product(mw, op, A, B, pad=0, tile=0):
    """C = A B^T for A [M][K], B [N][K] through operation `op`, `pad` extra columns per stored row."""
    a, b = (A.T if op == TN else A), (B if op == NT else B.T)
    a, b = (np.pad(v, ((0, 0), (0, pad))) for v in (a, b))
    a, b = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (a, b))
    out = mw.gemm_f32(op, a[:, :a.shape[1] - pad], b[:, :b.shape[1] - pad], tile=tile)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def bound(A, B):
    a, b = np.abs(A.astype(np.float64)), np.abs(B.astype(np.float64))
    return A.shape[1] * 2.0 ** -24 * (a @ b.T) + 2.0 ** -149


def check(mw, op, A, B, pad=0):
    print("split product op=%d M=%d N=%d K=%d pad=%d" % (op, A.shape[0], B.shape[0], A.shape[1], pad), flush=True)
    got = product(mw, op, A, B, pad).astype(np.float64)
    err = np.abs(got - A.astype(np.float64) @ B.astype(np.float64).T)
    assert np.isfinite(got).all() and (err <= bound(A, B)).all(), float((err / bound(A, B)).max())
    return got


def operands(seed, M, N, K):
    rng = np.random.default_rng(seed)
    return rng, rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)


# one size for each split tile: 64 x 64, 128 x 128 and (TN) 256 x 128
SIZES = [(NT, 900, 1020, 520), (NT, 1436, 1500, 264), (NN, 900, 1020, 520), (NN, 1436, 1500, 264),
         (TN, 900, 1020, 520), (TN, 1436, 1500, 264), (TN, 2290, 2300, 260)]


@pytest.mark.parametrize("op", [NT, NN, TN])
@pytest.mark.parametrize("M,N,K,pad", [
    (832, 960, 512, 0),      # 195 tiles of 64 x 64 and the least K that takes them
    (961, 1021, 517, 0),     # odd everything: element-wise loads, remainders of rows and of a K tile
    (1408, 1536, 256, 0),    # 132 tiles of 128 x 128 and the least K of those
    (1501, 1433, 259, 0),    # odd
    (1500, 1412, 300, 1),    # an unaligned leading dimension
    (1024, 2048, 1024, 0),   # 128 tiles: from this K on
    (1024, 1024, 2044, 0),   # one round of 64 x 64 tiles up to this K
    (1024, 1024, 2048, 0),
    (130, 8448, 300, 0),     # as many tiles, mostly padding: fp32 tiles
    (2177, 2304, 256, 0),    # one row more than the tiles; TN: 256 x 128 tiles
])
def test_tile_edges(mw, op, M, N, K, pad):
    _, A, B = operands(M + K, M, N, K)
    check(mw, op, A, B, pad)


@pytest.mark.parametrize("op,M,N,K", SIZES)
@pytest.mark.parametrize("kind", ["scales", "late", "late_tiny", "late_large", "jump", "zero", "subnormal", "huge"])
def test_rows_of_other_magnitudes(mw, op, M, N, K, kind):
    rng, A, B = operands(7, M, N, K)
    rows = rng.choice(M, 60, replace=False)
    if kind == "scales":           # rows of A and B apart by many powers of two
        A *= (2.0 ** rng.integers(-60, 40, (M, 1))).astype(np.float32)
        B *= (2.0 ** rng.integers(-30, 30, (N, 1))).astype(np.float32)
    elif kind == "late":           # nothing in the first 64 (a unit that is off for all of them)
        A[rows, :64] = 0
        A[rows, 64:] *= rng.random((60, K - 64)).astype(np.float32) < 0.02
    elif kind == "late_tiny":      # nothing, then values far below those of the neighbours
        A[rows, :64] = 0
        A[rows] *= (2.0 ** rng.integers(-40, 0, (60, 1))).astype(np.float32)
    elif kind == "late_large":
        A[rows, :64] = 0
        A[rows] *= (2.0 ** rng.integers(0, 40, (60, 1))).astype(np.float32)
    elif kind == "jump":           # small values first, large ones after them
        A[rows, :64] *= (2.0 ** rng.integers(-40, -4, (60, 1))).astype(np.float32)
    elif kind == "zero":
        A[rows] = 0
        B[:128] = 0                # whole groups of rows
    elif kind == "subnormal":
        A[rows] *= np.float32(2.0 ** -130)
        A[rows] *= np.float32(2.0 ** -10)
    else:                          # sums that no longer fit once both operands are scaled up: fp32 instructions
        A *= np.float32(2.0 ** 60)
        B *= np.float32(2.0 ** 40)
    got = check(mw, op, A, B)
    # a row's result does not depend on the other rows
    other = np.full_like(A, 1e30)
    other[rows[0]] = A[rows[0]]
    assert np.array_equal(product(mw, op, other, B)[rows[0]].astype(np.float64), got[rows[0]])


def along_k(kind, M, N, K):
    """Operands whose magnitudes differ along K, so that a row's largest value says nothing about what it adds."""
    rng, A, B = operands(5, M, N, K)
    if kind == "leading":          # the first values meet nothing
        A[:, :4], A[:, 4:], B[:, :4], B[:, 4:] = 1e10, 1, 0, 1
    elif kind == "column":         # one of them does
        A[:, 37] *= np.float32(1e6)
        B[:, 37] = 0
    elif kind in ("reciprocal", "far_reciprocal"):
        s = 2.0 ** rng.integers(*((-12, 13) if kind == "reciprocal" else (-40, 41)), K)
        A, B = (A * s).astype(np.float32), (B / s).astype(np.float32)
    else:                          # samples of very different cotangents, each unit off for half of them
        A *= (2.0 ** rng.integers(-40, 1, K)).astype(np.float32)
        B *= rng.random((N, K)) < 0.5
    return A, B


@pytest.mark.parametrize("op,M,N,K", SIZES)
@pytest.mark.parametrize("kind", ["leading", "column", "reciprocal", "far_reciprocal", "samples"])
def test_magnitudes_that_differ_along_k(mw, op, M, N, K, kind):
    """Also against fp32 instructions on the same data: the largest error beside sum|a||b| is no more than twice theirs,
    or a rounding of the operands where they have none."""
    A, B = along_k(kind, M, N, K)
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    size = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64).T + 2.0 ** -149
    split, f32 = ((np.abs(product(mw, op, A, B, tile=t) - ref) / size).max() for t in (0, mw.TILE_64))
    print("%s op=%d error beside sum|a||b|: split %.3g, fp32 instructions %.3g" % (kind, op, split, f32), flush=True)
    assert split <= 2 * f32 + 2.0 ** -24 and split <= K * 2.0 ** -24


@pytest.mark.parametrize("op,M,N", [(NT, 1000, 1000), (NT, 1536, 1536), (NN, 1000, 1000), (NN, 1536, 1536), (TN, 1000, 1000),
                                    (TN, 2304, 2304)])
def test_a_single_term_is_exact(mw, op, M, N):
    """Products with one term each return the values as they are, all 24 bits of them, over fp32's range."""
    K = N
    rng, A, _ = operands(3, M, N, K)
    A *= (2.0 ** rng.integers(-120, 60, (M, K))).astype(np.float32)
    perm = rng.permutation(K)
    B = np.zeros((N, K), np.float32)
    B[np.arange(N), perm] = 1
    assert np.array_equal(product(mw, op, A, B), A[:, perm])


@pytest.mark.parametrize("op,M,N,K", SIZES)
def test_values_that_do_not_fit(mw, op, M, N, K):
    """Infinities and NaN reach exactly the results they belong to; a value next to fp32's largest stays finite."""
    _, A, B = operands(11, M, N, K)
    clean = product(mw, op, A, B)
    A[3, 200], A[65, 5], A[130, K - 1], A[200, 77], B[40, 250] = np.inf, -np.inf, np.nan, 3e38, 1e30
    got = product(mw, op, A, B)
    with np.errstate(all="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64).T
        assert np.array_equal(np.isnan(got[[3, 65, 130]]), np.isnan(ref[[3, 65, 130]]))
        assert np.array_equal(np.sign(got[[3, 65]]), np.sign(ref[[3, 65]]))
    rows = np.setdiff1d(np.arange(M), [3, 65, 130, 200])
    cols = np.setdiff1d(np.arange(N), [40])
    assert np.array_equal(got[np.ix_(rows, cols)], clean[np.ix_(rows, cols)])
    fine = np.abs(ref[200]) < 3e38
    assert fine.sum() > 100 and np.allclose(got[200][fine], ref[200][fine], rtol=1e-4)
    assert np.allclose(got[rows, 40], ref[rows, 40], rtol=1e-4)


@pytest.mark.parametrize("op", [NT, NN, TN])
@pytest.mark.parametrize("M,K", [(1024, 512), (1024, 1920), (1536, 256), (1536, 2048)])
def test_no_less_precise_than_fp32_instructions(mw, op, M, K):
    _, A, B = operands(K, M, M, K)
    f32_tile = mw.TILE_64K2 if K >= 1024 else mw.TILE_64
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    split, f32 = (np.linalg.norm(product(mw, op, A, B, tile=t) - ref) / np.linalg.norm(ref) for t in (0, f32_tile))
    print("K=%d normwise error: split %.3g, fp32 instructions %.3g" % (K, split, f32), flush=True)
    assert split <= f32


@pytest.mark.parametrize("op,M,N,K", SIZES + [(NT, 1024, 1024, 1920), (NN, 1536, 1536, 2048), (TN, 2304, 2304, 1024)])
def test_errors_have_no_common_sign(mw, op, M, N, K):
    """The mean error of a million results or more. Independent errors leave about a thousandth of their rms, of one sign
    a fifth of it; sums over samples would keep that."""
    _, A, B = operands(K, M, N, K)
    err = product(mw, op, A, B) - A.astype(np.float64) @ B.astype(np.float64).T
    rms = np.sqrt(np.mean(err * err))
    print("op=%d K=%d: mean error %.2g of its rms" % (op, K, err.mean() / rms), flush=True)
    assert abs(err.mean()) <= 0.03 * rms


@pytest.mark.parametrize("widths,alphas", [
    ((1024, 1024, 1024, 192), (0.3, 0.3, 0.3)),     # 64 x 64 tiles; the last layer is too small for split operands
    ((1023, 1022, 1021), (0.3, 0.3)),               # element-wise loads: every product in a launch of its own
    ((96, 96), (0.3,)),                             # all of it below
    ((1024, 1008, 992), (0.0, 0.0)),               # the fragment store restored in the cotangent's launch
    ((2816, 2752), (0.3,)),                         # 128 x 128 tiles
])
def test_phase3_in_two_launches(mw, widths, alphas):
    """The activation and the cotangent of a layer in launches of their own: against the oracle on the same signs, and
    with the same bits as the unfused path."""
    wl = make_mlp(list(widths), 776, list(alphas), seed=3, reseed_interval=0, name="split")
    nets = [mw.MoonwalkNet.from_workload(wl, fuse=f) for f in (True, False)]
    res = [net.moonwalk_grad(net.x, net.t) for net in nets]
    torch.cuda.synchronize()
    check_moonwalk(nets[0], wl, res[0])
    for i in range(wl.depth):
        assert torch.equal(res[0].dW[i], res[1].dW[i]), i
        assert O.normwise_rel_err(res[0].db[i].cpu().numpy(), res[1].db[i].cpu().numpy()) < 1e-5
    for net in nets:
        net.close()


@pytest.mark.parametrize("widths,kernels", [
    ((1024, 1024, 1024), 5),     # activation and cotangent twice (the second with the first weight gradient), one left
    ((1023, 1022, 1021), 6),     # every product by itself
    ((96, 96, 96), 3),           # one kernel for both products
])
def test_every_phase3_kernel_is_counted(mw, widths, kernels):
    wl = make_mlp(list(widths), 776, [0.3, 0.3], seed=3, reseed_interval=0, name="split")
    net = mw.MoonwalkNet.from_workload(wl)
    net.moonwalk_grad(net.x, net.t)
    torch.cuda.synchronize()
    assert net.profile_launches()["phase3"] == kernels
    net.close()
