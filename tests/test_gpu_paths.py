"""Kernels at the edges of their tiles and of their dispatch (needs a GPU):
products of small integers, which are exact in every type, and the pivoted QR
and the orthonormalization against the FP64 oracle."""

import numpy as np
import pytest
import torch

from oracle import dense as OD
from paper_1502_05366_amd import workloads as W
from tests.helpers import orth_err, pivot_prefix

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_1502_05366_amd as R
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return R


def dev(x, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")


def padded(x, dtype, ld, off=0):
    """x on the GPU with rows ld apart, off elements into its buffer."""
    buf = torch.zeros(x.shape[0] * ld + off, dtype=dtype, device="cuda")
    v = torch.as_strided(buf, x.shape, (ld, 1), off)
    v.copy_(torch.as_tensor(x))
    return v


# ---- FP64 / FP32 passes with A in registers --------------------------------
# K = 16 (tile kernel), 17 and 31 (one full k-step and a tail), l around the
# column blocks, rows around a tile; row strides and first elements that are
# not multiples of 16 bytes
@pytest.mark.parametrize("m,n,l,pad,off", [
    (70, 16, 5, 0, 0), (129, 17, 16, 0, 0), (63, 31, 17, 1, 0), (257, 33, 32, 0, 1),
    (300, 65, 33, 3, 1), (128, 640, 48, 0, 0), (511, 96, 79, 2, 3), (65, 1029, 81, 1, 1),
    (4099, 130, 113, 0, 0), (1023, 258, 225, 5, 0), (40, 5000, 96, 0, 1)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_pass_edges(R, m, n, l, pad, off, dtype):
    A = W.integer_matrix(m, n, seed=m + n)
    Xn = W.integer_matrix(n, l, seed=l + 1)
    Xm = W.integer_matrix(m, l, seed=l + 2)
    Ad = padded(A, dtype, n + pad, off)
    Y = R.pass_(Ad, dev(Xn, dtype)).cpu().numpy()
    Z = R.pass_(Ad, dev(Xm, dtype), trans=True).cpu().numpy()
    # every partial sum is an integer below 2^24: exact in FP32 and FP64
    assert np.array_equal(Y.astype(np.float64), A @ Xn)
    assert np.array_equal(Z.astype(np.float64), A.T @ Xm)


# the unrolled steps of the shortest k-steps (one and two column blocks, at least
# seven steps): their operands come from lane swaps in FP64
@pytest.mark.parametrize("m,n,l", [(300, 1000, 16), (130, 333, 9), (1000, 2049, 32)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_pass_short_steps(R, m, n, l, dtype):
    A = W.integer_matrix(m, n, seed=m + n)
    Xn = W.integer_matrix(n, l, seed=l + 1)
    Xm = W.integer_matrix(m, l, seed=l + 2)
    Ad = dev(A, dtype)
    Y = R.pass_(Ad, dev(Xn, dtype)).cpu().numpy()
    Z = R.pass_(Ad, dev(Xm, dtype), trans=True).cpu().numpy()
    assert np.array_equal(Y.astype(np.float64), A @ Xn)
    assert np.array_equal(Z.astype(np.float64), A.T @ Xm)


# 16 column blocks (the most accumulators), as one column tile and as two
@pytest.mark.parametrize("m,n,l", [(700, 500, 241), (257, 640, 250), (700, 500, 449),
                                   (300, 777, 500), (500, 700, 512)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_pass_widest_tiles(R, m, n, l, dtype):
    A = W.integer_matrix(m, n, seed=m + n)
    Xn = W.integer_matrix(n, l, seed=l + 1)
    Xm = W.integer_matrix(m, l, seed=l + 2)
    Ad = dev(A, dtype)
    Y = R.pass_(Ad, dev(Xn, dtype)).cpu().numpy()
    Z = R.pass_(Ad, dev(Xm, dtype), trans=True).cpu().numpy()
    assert np.array_equal(Y.astype(np.float64), A @ Xn)
    assert np.array_equal(Z.astype(np.float64), A.T @ Xm)


# ---- BF16 / FP8 passes ------------------------------------------------------
# reductions shorter than a k-step and with a remainder, rows around a tile and
# one more tile than compute units, l around the column blocks (288 / 289: one
# and two column groups)
@pytest.mark.parametrize("m,n,l", [(31, 33, 1), (255, 64, 15), (257, 129, 17), (130, 500, 32),
                                   (600, 250, 97), (66000, 96, 33), (96, 66000, 33),
                                   (300, 300, 288), (290, 310, 289), (64, 4100, 575)])
@pytest.mark.parametrize("kind", ["bf16", "f8"])
def test_narrow_pass_edges(R, m, n, l, kind):
    A = W.integer_matrix(m, n, seed=m + n)
    # (a largest entry of 7 in every column: the FP8 scales are powers of two)
    Xn = np.clip(W.integer_matrix(n, l, seed=l + 1), -7, 7)
    Xm = np.clip(W.integer_matrix(m, l, seed=l + 2), -7, 7)
    Xn[0, :] = 7.0
    Xm[0, :] = 7.0
    ld = (n + 15) // 16 * 16
    if kind == "bf16":
        Ad = padded(A, torch.bfloat16, ld)
        Y = R.pass_(Ad, dev(Xn, torch.float32))
        Z = R.pass_(Ad, dev(Xm, torch.float32), trans=True)
    else:
        Ad = padded(torch.as_tensor(A).to(torch.float8_e4m3fn).view(torch.uint8).numpy(),
                    torch.uint8, ld)
        sc = torch.ones(n, dtype=torch.float32, device="cuda")
        Y = R.pass_f8(Ad, sc, dev(Xn, torch.float32))
        Z = R.pass_f8(Ad, sc, dev(Xm, torch.float32), trans=True)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), A @ Xn)
    assert np.array_equal(Z.cpu().numpy().astype(np.float64), A.T @ Xm)


# few row tiles: column tiles of two blocks and up, splits of two steps and up, pairs
# of row tile and split that do not fill the eight XCDs
@pytest.mark.parametrize("m,n,l", [(1000, 1000, 250), (1024, 1024, 32), (300, 5000, 100),
                                   (5000, 300, 220), (513, 2049, 576), (256, 700, 300),
                                   (2600, 450, 130)])
@pytest.mark.parametrize("kind", ["bf16", "f8"])
def test_narrow_pass_few_tiles(R, m, n, l, kind):
    A = W.integer_matrix(m, n, seed=m + n)
    Xn = np.clip(W.integer_matrix(n, l, seed=l + 1), -7, 7)
    Xm = np.clip(W.integer_matrix(m, l, seed=l + 2), -7, 7)
    Xn[0, :] = 7.0
    Xm[0, :] = 7.0
    ld = (n + 15) // 16 * 16
    if kind == "bf16":
        Ad = padded(A, torch.bfloat16, ld)
        Y = R.pass_(Ad, dev(Xn, torch.float32))
        Z = R.pass_(Ad, dev(Xm, torch.float32), trans=True)
    else:
        Ad = padded(torch.as_tensor(A).to(torch.float8_e4m3fn).view(torch.uint8).numpy(),
                    torch.uint8, ld)
        sc = torch.ones(n, dtype=torch.float32, device="cuda")
        Y = R.pass_f8(Ad, sc, dev(Xn, torch.float32))
        Z = R.pass_f8(Ad, sc, dev(Xm, torch.float32), trans=True)
    # (exact: integers, every partial sum below 2^24)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), A @ Xn)
    assert np.array_equal(Z.cpu().numpy().astype(np.float64), A.T @ Xm)


# results scaled and added to C over every column block: X of two FP8 terms (the
# second of them exact here: its product is zero) and scales of powers of two
@pytest.mark.parametrize("m,n,l", [(300, 260, 31), (257, 400, 250), (130, 1000, 288)])
def test_f8_pass_adds_scaled_results(R, m, n, l):
    g = np.random.default_rng(m + l)
    A = W.integer_matrix(m, n, seed=m + n)
    ld = (n + 15) // 16 * 16
    Ad = padded(torch.as_tensor(A).to(torch.float8_e4m3fn).view(torch.uint8).numpy(),
                torch.uint8, ld)
    s = 2.0 ** g.integers(-3, 4, n)
    # (a largest entry of 7 times a power of two in every column of diag(s) X and X)
    Xn = np.clip(W.integer_matrix(n, l, seed=l + 1), -7, 7)
    Xm = np.clip(W.integer_matrix(m, l, seed=l + 2), -7, 7)
    Xn[0, :] = 7.0
    Xm[0, :] = 7.0
    t = 2.0 ** g.integers(-2, 3, l)
    sd = dev(s, torch.float32)
    Y = R.pass_f8(Ad, sd, dev(Xn * t / s[:, None], torch.float32), split=True)
    Z = R.pass_f8(Ad, sd, dev(Xm * t, torch.float32), trans=True, split=True)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), A @ (Xn * t))
    assert np.array_equal(Z.cpu().numpy().astype(np.float64), s[:, None] * (A.T @ (Xm * t)))


# ---- orth: dependent columns and the second pass's test ----------------------
# one and several column blocks (l around 16 and 64), the last block ragged;
# every third column repeats the one before it
@pytest.mark.parametrize("rows,l", [(200, 15), (64, 16), (1000, 17), (333, 63), (5000, 65),
                                    (2000, 256)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_orth_dependent_columns(R, rows, l, dtype):
    g = np.random.default_rng(rows + l)
    Y = g.standard_normal((rows, l)).astype(np.float32).astype(np.float64)
    Y[:, 2::3] = Y[:, 1::3][:, :Y[:, 2::3].shape[1]]
    Q, Rm, info = R.orth(dev(Y, dtype), seed=11)
    Q, Rm = Q.cpu().numpy().astype(np.float64), Rm.cpu().numpy()
    assert int(info.cpu()[0]) == R.INFO_ORTH_FALLBACK
    # orthonormal and spanning Y, to the rounding of the basis: l entries of a
    # column, each to an ulp or so of its type
    eps = np.finfo(np.float64 if dtype == torch.float64 else np.float32).eps
    assert orth_err(Q) < 16 * np.sqrt(l) * eps
    assert np.abs(Q @ (Q.T @ Y) - Y).max() < 64 * l * eps * np.abs(Y).max()
    assert np.abs(Q @ Rm - Y).max() < 64 * l * eps * np.abs(Y).max()


# ---- pivoted QR ---------------------------------------------------------------
# rows around the multiples of 16 that a lane can hold, columns around one, two
# and three per group of 16 lanes on 256 compute units, and beyond (in LDS)
@pytest.mark.parametrize("r,c,k", [(1, 1, 1), (32, 31, 20), (33, 33, 33), (64, 1025, 40),
                                   (129, 2000, 100), (209, 300, 209), (256, 700, 256),
                                   (20, 8193, 12), (40, 16385, 10), (24, 24576, 6),
                                   (24, 24577, 6)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_cpqr_edges(R, r, c, k, dtype):
    g = np.random.default_rng(r * 7 + c)
    B = g.standard_normal((r, c)) * g.uniform(0.05, 10.0, c)[None, :]
    B = B.astype(np.float32).astype(np.float64)
    J, T, pv, info = R.cpqr(dev(B.T, dtype), r, k)
    J, T, pv = J.cpu().numpy(), T.cpu().numpy(), pv.cpu().numpy()
    f = OD.cpqr(B, k)
    # up to a near tie the pivots are the oracle's
    npre = pivot_prefix(f['pivot_norms'], f['second_norms'], 1e-8)
    npre = k if c == k == npre + 1 else npre
    assert np.array_equal(J[:npre], f['J'][:npre])
    assert np.allclose(pv[:npre], f['pivot_norms'][:npre], rtol=1e-11)
    if npre == k:
        To = OD.solve_upper(f['S11'], f['S12'])
        assert np.abs(T - To).max(initial=0) <= 1e-9 * max(1.0, np.abs(To).max(initial=0))
    assert np.array_equal(np.sort(J), np.arange(c))
    assert np.all(np.diff(J[k:]) > 0)
    assert int(info.cpu()[0]) & R.INFO_BARRIER == 0


def test_cpqr_ties_take_the_lowest_column(R):
    """Equal columns in different lanes, waves and workgroups."""
    g = np.random.default_rng(2)
    r, c = 40, 9000
    B = 0.1 * g.standard_normal((r, c))
    x, y = 9.0 * g.standard_normal((2, r))
    B[:, [8999, 4100, 77, 70, 66]] = x[:, None]
    B[:, [8000, 300, 299]] = 0.5 * y[:, None]
    J, T, pv, info = R.cpqr(dev(B.T), r, 2)
    assert J.cpu().numpy()[:2].tolist() == [66, 299]


# ---- the block Jacobi split over workgroups ------------------------------------
# one more column than the single-workgroup limit, around the blocks of 16, an odd
# number of blocks, both row layouts (l <= 256 and above), the largest
@pytest.mark.parametrize("l", [65, 80, 81, 112, 256, 257, 400, 576])
def test_small_svd_split(R, l):
    g = np.random.default_rng(l)
    U0 = np.linalg.qr(g.standard_normal((l, l)))[0]
    V0 = np.linalg.qr(g.standard_normal((l, l)))[0]
    so = np.logspace(0, -3, l)
    Rh = np.linalg.qr((U0 * so) @ V0.T)[1]
    S, Uh, Vh, info = R.small_svd(dev(Rh), l)
    S, Uh, Vh = S.cpu().numpy(), Uh.cpu().numpy(), Vh.cpu().numpy()
    assert int(info.cpu()[0]) == 0
    # the rounding of l rotations per column and sweep, of the size of sigma_1
    bound = 50 * l * np.finfo(np.float64).eps
    assert np.abs(S - so).max() <= bound
    assert orth_err(Uh) <= bound * 1e3 and orth_err(Vh) <= bound     # (Uh: w_j / sigma_j)
    assert np.abs(Rh @ Vh - Uh * S[None, :]).max() <= bound


@pytest.mark.parametrize("l", [70, 112, 256])
def test_split_and_whole_pairs_give_the_same_bits(R, l):
    """svd splits the block pairs; beside a pivoted QR (decompose) each has one
    workgroup: the sums have the same order."""
    g = torch.Generator(device="cuda").manual_seed(l)
    A = torch.randn((700, 400), dtype=torch.float64, device="cuda", generator=g)
    k, p = l - 10, 10
    U, S, V, info = R.svd(A, k, p, 1, 5)
    D = R.decompose(A, k, p, 1, 5)
    assert int(info.cpu()[0]) == 0
    for x, y in ((U, D["U"]), (S, D["S"]), (V, D["V"])):
        assert torch.equal(x, y)


def test_split_jacobi_on_four_streams(R):
    g = torch.Generator(device="cuda").manual_seed(9)
    As = [torch.randn((1500, 1200), dtype=torch.float64, device="cuda", generator=g)
          for _ in range(4)]
    alone = [R.svd(A, 560, 16, 0, 3) for A in As]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in As]
    beside = []
    for A, s in zip(As, streams):
        with torch.cuda.stream(s):
            beside.append(R.svd(A, 560, 16, 0, 3))
    torch.cuda.synchronize()
    for x, y in zip(alone, beside):
        assert int(y[3].cpu()[0]) == 0
        for u, v in zip(x[:3], y[:3]):
            assert torch.equal(u, v)
