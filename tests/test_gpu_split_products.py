"""Products on split operands (two fp16 halves per fp32 value) against fp64, where they can go wrong: edges of the
256 x 128, 128 x 128 and 64 x 64 tiles, short and odd K, unaligned leading dimensions, and rows whose first values (the
sample that chooses a row's scale) say little about the rest.

Bound per element. A value v of a row with largest magnitude m is represented to 2^-23 |v|, or, where its lower half
falls under fp16's subnormal spacing, to 2^-25 after scaling; a row is scaled so that m is at least 2^-4 (else fp32
instructions repeat it), so that is 2^-21 m at worst. With the dropped product of the lower halves (2^-22) and K sums
rounded to 2^-24:
    |C - AB| <= (2^-21 + K 2^-24) sum|a||b| + 2^-21 (max|a| sum|b| + max|b| sum|a|)
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
    K = A.shape[1]
    return (2.0 ** -21 + K * 2.0 ** -24) * (a @ b.T) + 2.0 ** -21 * (np.outer(a.max(1), b.sum(1)) + np.outer(a.sum(1), b.max(1))) + 2.0 ** -149


def check(mw, op, A, B, pad=0):
    print("split product op=%d M=%d N=%d K=%d pad=%d" % (op, A.shape[0], B.shape[0], A.shape[1], pad), flush=True)
    got = product(mw, op, A, B, pad).astype(np.float64)
    err = np.abs(got - A.astype(np.float64) @ B.astype(np.float64).T)
    assert np.isfinite(got).all() and (err <= bound(A, B)).all(), float((err / bound(A, B)).max())
    return got


def operands(seed, M, N, K):
    rng = np.random.default_rng(seed)
    return rng, rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)


@pytest.mark.parametrize("op", [NT, NN, TN])
@pytest.mark.parametrize("M,N,K,pad", [
    (640, 640, 128, 0),      # 100 tiles of 64 x 64: the least grid and the least K that take split operands
    (700, 612, 160, 0),      # remainders of rows and of a K tile
    (637, 705, 131, 0),      # odd everything: element-wise loads
    (1280, 2052, 192, 1),    # 128 x 128 tiles, an unaligned leading dimension
    (2049, 2304, 256, 0),    # one row more than the tiles
    (4096, 4100, 136, 0),    # TN: 256 x 128 tiles
])
def test_tile_edges(mw, op, M, N, K, pad):
    _, A, B = operands(M + K, M, N, K)
    check(mw, op, A, B, pad)


@pytest.mark.parametrize("op", [NT, NN, TN])
@pytest.mark.parametrize("kind", ["scales", "late", "late_tiny", "late_large", "jump", "zero", "subnormal"])
def test_rows_the_sample_says_little_about(mw, op, kind):
    M, N, K = 640, 704, 320
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
    elif kind == "jump":           # small in the sample, large after it
        A[rows, :64] *= (2.0 ** rng.integers(-40, -4, (60, 1))).astype(np.float32)
    elif kind == "zero":
        A[rows] = 0
        B[:128] = 0                # whole groups of rows
    else:
        A[rows] *= np.float32(2.0 ** -130)
        A[rows] *= np.float32(2.0 ** -10)
    got = check(mw, op, A, B)
    # a row's result does not depend on the rows beside it in the tile beyond its aligned group of 32
    other = A.copy()
    keep = 32 * (rows[0] // 32)
    other[:keep] = 1e30 if keep else other[:keep]
    assert np.array_equal(product(mw, op, other, B)[keep:keep + 32].astype(np.float64), got[keep:keep + 32])


@pytest.mark.parametrize("op", [NT, NN, TN])
def test_values_that_do_not_fit(mw, op):
    """Infinities and NaN reach exactly the results they belong to; a value next to fp32's largest stays finite."""
    M, N, K = 640, 704, 320
    _, A, B = operands(11, M, N, K)
    clean = product(mw, op, A, B)
    A[3, 200], A[65, 5], A[130, 319], A[200, 77], B[40, 300] = np.inf, -np.inf, np.nan, 3e38, 1e30
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
@pytest.mark.parametrize("K", [128, 512, 2048])
def test_no_less_precise_than_fp32_instructions(mw, op, K):
    _, A, B = operands(K, 1024, 768, K)
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    split, f32 = (np.linalg.norm(product(mw, op, A, B, tile=t) - ref) / np.linalg.norm(ref) for t in (0, mw.TILE_64))
    print("K=%d normwise error: split %.3g, fp32 instructions %.3g" % (K, split, f32), flush=True)
    assert split <= f32


@pytest.mark.parametrize("widths,alphas", [
    ((1152, 1024, 1024, 192), (0.3, 0.3, 0.3)),     # 64 x 64 tiles; the last layer is too small for split operands
    ((1029, 1027, 1025), (0.3, 0.3)),               # element-wise loads: every product in a launch of its own
    ((96, 96), (0.3,)),                             # all of it below
    ((1088, 1056, 1024), (0.0, 0.0)),               # the fragment store restored in the cotangent's launch
    ((2176, 2112), (0.3,)),                         # 128 x 128 tiles
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
