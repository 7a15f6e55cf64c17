"""The workloads by which this library's speed is followed.

``listed()`` names them, ``draw()`` gives more of the same ranges, ``prepare()``
makes what a program holds before a call (inputs on the device, a batch plan),
``run()`` is one pass through the public entry points of
``paper_1502_05366_amd``, ``work()`` the bytes and operations that the pass
cannot do without, and ``exact()`` the floating-point results from plain torch
in FP64.

The decompositions of an FP64 A are whole calls.  With A in FP32, BF16 or FP8
the products with A are followed on their own: they are the part of such a
call that depends on the storage type (everything after them is FP64).
"""

import math

import numpy as np
import torch

import paper_1502_05366_amd as R

DEV = "cuda"
SEED = 0x5EED0000            # seed of the Gaussian sketches


# ------------------------------------------------------------------- cases --

def listed():
    return [
        # the smallest call: a plain rank-20 SVD of a matrix that fits the caches;
        # launches and latencies count (the paper's own synthetic test matrix)
        dict(name="svd_small", op="svd", m=2000, n=1000, k=20, p=10, q=1, decay="exp"),
        # many components of a mid-size matrix: the sample is wider than one
        # column block of the orthonormalization, the small SVD is 576 x 576
        dict(name="svd_wide", op="svd", m=16384, n=8192, k=512, p=64, q=1, decay="inv"),
        # SVD + ID + CUR of a large slowly decaying matrix in one call (the
        # benchmark's configuration)
        dict(name="decompose_large", op="decompose", m=20000, n=10000, k=200, p=20, q=2,
             decay="inv"),
        # row and column selection of an ordinary matrix with odd sizes
        dict(name="cur_odd", op="cur", m=5003, n=3001, k=90, p=11, q=1, decay="inv"),
        # rank found on the fly: blocks of 32 until the residual is below tol
        dict(name="qb_adaptive", op="qb", m=20000, n=10000, b=32, M=10, q=1, tol=0.07,
             decay="inv"),
        # a training step through the SVD: forward, then the gradient of
        # sum(S) + ||A - Q Q^T A||_F^2
        dict(name="svd_train", op="grad", m=8192, n=4096, k=64, p=16, q=2, vectors=False,
             decay="inv"),
        # thousands of uneven small FP32 problems in one call
        dict(name="batch", op="batch", count=4096, mmax=2048, nmax=1024, kmax=64, p=8, q=1,
             sizes=0xC0FFEE04),
        # the two products of a power step, A in FP32
        dict(name="pass_f32", op="pass", dtype="f32", m=20000, n=10000, l=220),
        # the same with a narrow sample (bound by reading A)
        dict(name="pass_f32_narrow", op="pass", dtype="f32", m=20000, n=10000, l=30),
        # A in BF16
        dict(name="pass_bf16", op="pass", dtype="bf16", m=20000, n=10000, l=220),
        # A in BF16, the largest: many components of a large matrix
        dict(name="pass_bf16_wide", op="pass", dtype="bf16", m=65536, n=32768, l=576),
        # A in FP8 E4M3 with column scales; the last projection keeps two terms
        dict(name="pass_f8_wide", op="pass", dtype="f8", m=65536, n=32768, l=576),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the whole range of the listed ones (evenly in
    their logarithm), not rounded to anything."""
    op = rng.choice(["svd", "svd", "decompose", "cur", "qb", "grad", "batch", "pass", "pass",
                     "pass", "pass"])
    if op == "pass":
        dtype = rng.choice(["f32", "f32", "bf16", "f8"])
        top = (20000, 10000, 220) if dtype == "f32" else (65536, 32768, 576)
        return dict(op=op, dtype=dtype, m=_log(rng, 1000, top[0]), n=_log(rng, 1000, top[1]),
                    l=_log(rng, 16, top[2]))
    if op == "batch":
        return dict(op=op, count=_log(rng, 64, 2048), mmax=_log(rng, 256, 2048),
                    nmax=_log(rng, 256, 1024), kmax=_log(rng, 8, 64), p=8, q=rng.choice([0, 1]),
                    sizes=rng.randrange(1 << 30))
    if op == "qb":
        m, n = _log(rng, 1500, 20000), _log(rng, 1000, 10000)
        return dict(op=op, m=m, n=n, b=rng.choice([8, 16, 20, 32, 48]), M=rng.randint(3, 8),
                    q=rng.choice([0, 1]), tol=0.0, decay="inv")
    if op == "grad":
        return dict(op=op, m=_log(rng, 500, 8192), n=_log(rng, 400, 4096),
                    k=_log(rng, 8, 64), p=rng.randint(4, 16), q=rng.choice([1, 2]),
                    vectors=rng.choice([False, True]), decay="inv")
    if op == "svd":
        m, n = _log(rng, 600, 16384), _log(rng, 600, 8192)
        return dict(op=op, m=m, n=n, k=_log(rng, 10, 500), p=rng.randint(5, 64),
                    q=rng.choice([0, 1, 1, 2]), decay="inv")
    return dict(op=op, m=_log(rng, 600, 20000), n=_log(rng, 600, 10000), k=_log(rng, 10, 200),
                p=rng.randint(5, 20), q=rng.choice([1, 1, 2]), decay="inv")


# ------------------------------------------------------------------ inputs --

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _orthonormal(g, rows, r):
    """rows x r with orthonormal columns (Gaussian, orthonormalized twice)."""
    X = torch.randn(rows, r, dtype=torch.float64, device=DEV, generator=g)
    for _ in range(2):
        L = torch.linalg.cholesky(X.T @ X)
        X = torch.linalg.solve_triangular(L, X.T.contiguous(), upper=False).T.contiguous()
    return X


def _spectrum_matrix(seed, m, n, decay):
    """FP64 A = U diag(s) V^T + noise, s_j = 1/j ("inv") or 10^(-j/10) ("exp")
    over the first min(m, n, 1280) components, noise N(0, 1e-6^2) ("inv")."""
    g = _gen(seed)
    r = min(m, n, 1280)
    j = torch.arange(1, r + 1, dtype=torch.float64, device=DEV)
    s = 1.0 / j if decay == "inv" else 10.0 ** (-j / 10.0)
    U, V = _orthonormal(g, m, r), _orthonormal(g, n, r)
    A = (U * s) @ V.T
    if decay == "inv":
        A += 1e-6 * torch.randn(m, n, dtype=torch.float64, device=DEV, generator=g)
    return A


def _pass_inputs(case, seed):
    """A in its storage type (rows padded to 16 bytes), the column scales of an
    FP8 A, and the skinny operands of A X and A^T X (FP32, columns of norm ~1)."""
    m, n, l, dtype = case["m"], case["n"], case["l"], case["dtype"]
    g = _gen(seed)
    r = min(m, n, 256)
    j = torch.arange(1, r + 1, dtype=torch.float32, device=DEV)
    P = torch.randn(m, r, device=DEV, generator=g) / j
    A = torch.matmul(P, torch.randn(r, n, device=DEV, generator=g))
    X = torch.randn(n, l, device=DEV, generator=g) / math.sqrt(n)
    W = torch.randn(m, l, device=DEV, generator=g) / math.sqrt(m)
    scales = None
    if dtype == "bf16":
        St = torch.zeros(m, (n + 7) // 8 * 8, dtype=torch.bfloat16, device=DEV)
        St[:, :n] = A
        A = St[:, :n]
    elif dtype == "f8":
        scales = A.abs().amax(dim=0) / 448.0
        A /= scales
        St = torch.zeros(m, (n + 15) // 16 * 16, dtype=torch.uint8, device=DEV)
        St[:, :n] = A.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
        A = St[:, :n]
    return A, scales, X, W


def _batch_sizes(case):
    """m ~ U{64..mmax}, n ~ U{64..nmax}, k ~ U{4..kmax}."""
    g = np.random.Generator(np.random.PCG64(case["sizes"]))
    m = g.integers(64, case["mmax"] + 1, size=case["count"]).astype(np.int64)
    n = g.integers(64, case["nmax"] + 1, size=case["count"]).astype(np.int64)
    k = g.integers(4, case["kmax"] + 1, size=case["count"])
    return m, n, np.minimum(k, np.minimum(m, n)).astype(np.int32)


def _batch_matrices(case, seed):
    """The FP32 matrices, one by one: Gaussian factors, s_j = exp(-j/8)."""
    g = _gen(seed)
    s = torch.exp(-torch.arange(1, 321, device=DEV) / 8.0)
    for m, n in zip(*_batch_sizes(case)[:2]):
        r = min(int(m), int(n), 320)
        P = torch.randn(int(m), r, device=DEV, generator=g)
        yield (P * (s[:r] / math.sqrt(float(m) * float(n)))) @ torch.randn(r, int(n), device=DEV,
                                                                           generator=g)


def _cotangents(case, seed):
    g = _gen(seed + 0x10000)
    m, n, k = case["m"], case["n"], case["k"]
    return (torch.randn(m, k, dtype=torch.float64, device=DEV, generator=g),
            torch.randn(n, k, dtype=torch.float64, device=DEV, generator=g))


def prepare(case, seed):
    op = case["op"]
    if op == "pass":
        A, scales, X, W = _pass_inputs(case, seed)
        return dict(case=case, A=A, scales=scales, X=X, W=W)
    if op == "batch":
        plan = R.BatchPlan(*_batch_sizes(case), case["p"], case["q"])
        buf = torch.zeros(plan.a_elems, dtype=torch.float32, device=DEV)
        for i, A in enumerate(_batch_matrices(case, seed)):
            m, n = A.shape
            off, ld = int(plan.a_off[i]), int(plan.lda[i])
            buf[off:off + m * ld].view(m, ld)[:, :n] = A
        return dict(case=case, plan=plan, A=buf, out=plan.outputs())
    state = dict(case=case, A=_spectrum_matrix(seed, case["m"], case["n"], case["decay"]))
    if op == "grad":
        state["A"].requires_grad_(True)
        state["one"] = torch.ones(case["k"], dtype=torch.float64, device=DEV)
        if case["vectors"]:
            state["dU"], state["dV"] = _cotangents(case, seed)
    return state


# --------------------------------------------------------------------- run --

def run(state):
    c, A = state["case"], state["A"]
    op = c["op"]
    if op == "pass":
        if c["dtype"] == "f8":
            return [R.pass_f8(A, state["scales"], state["X"]),
                    R.pass_f8(A, state["scales"], state["W"], trans=True),
                    R.pass_f8(A, state["scales"], state["W"], trans=True, split=True)]
        return [R.pass_(A, state["X"]), R.pass_(A, state["W"], trans=True)]
    if op == "batch":
        return state["plan"].run(A, SEED, state["out"])
    if op == "qb":
        return R.qb(A, c["b"], c["M"], c["q"], c["tol"], SEED)
    k, p, q = c["k"], c["p"], c["q"]
    if op == "svd":
        return R.svd(A, k, p, q, SEED)
    if op == "cur":
        return R.cur(A, k, p, q, SEED)
    if op == "decompose":
        out = R.decompose(A, k, p, q, SEED)
        return {x: out[x] for x in ("U", "S", "V", "J", "T", "Jr", "Ucur", "info")}
    U, S, V, r2 = R.svd_diff(A, k, p, q, SEED)
    if c["vectors"]:
        (dA,) = torch.autograd.grad([U, S, V], [A], [state["dU"], state["one"], state["dV"]])
    else:
        (dA,) = torch.autograd.grad([S, r2], [A], [state["one"], torch.ones_like(r2)])
    return [U.detach(), S.detach(), V.detach(), r2.detach(), dA]


# -------------------------------------------------------------------- work --

def _svd_flops(m, n, k, l, q):
    """Products with A, the orthonormalizations (QR of the tall factors), U and V."""
    return (2.0 * (2 * q + 2) * m * n * l + (q + 1) * 2.0 * (m + n) * l * l
            + 2.0 * (m + n) * l * k)


def work(case):
    op = case["op"]
    if op == "batch":
        b = f = 0.0
        for m, n, k in zip(*_batch_sizes(case)):
            m, n, k = int(m), int(n), int(k)
            l = min(k + case["p"], m, n)
            b += 4.0 * m * n + 4.0 * (m + n) * k + 8.0 * k
            f += _svd_flops(m, n, k, l, case["q"])
        return dict(bytes=b, flops=f)
    m, n = case["m"], case["n"]
    if op == "pass":
        l = case["l"]
        a = {"f32": 4.0, "bf16": 2.0, "f8": 1.0}[case["dtype"]]
        reps = 4 if case["dtype"] == "f8" else 2        # the two-term product counts twice
        outs = m + 2 * n if case["dtype"] == "f8" else m + n
        return dict(bytes=a * m * n + 4.0 * l * (m + n) + 4.0 * l * outs,
                    flops=reps * 2.0 * m * n * l)
    if op == "qb":
        b, M, q = case["b"], case["M"], case["q"]
        if case["tol"] > 0:                             # s_j = 1/j: tail norm below tol
            M = min(M, math.ceil(1.0 / case["tol"] ** 2 / b) + 1)
        f = sum((2 * q + 3) * 2.0 * m * n * b + 4.0 * m * (i * b) * b for i in range(M))
        return dict(bytes=8.0 * (2.0 * m * n + (m + n) * b * M), flops=f)
    k, q = case["k"], case["q"]
    l = min(k + case["p"], m, n)
    f = _svd_flops(m, n, k, l, q)
    if op == "grad":
        # forward products with the residual, adjoint products, terms of dA
        f = 2.0 * m * n * l * ((2 * q + 3) + (2 * q + 1) + (2 * q + 2))
        return dict(bytes=8.0 * (2.0 * m * n + (m + n) * k), flops=f)
    out = 0.0
    if op in ("svd", "decompose"):
        out += (m + n) * k
    if op == "decompose":
        out += n * k
    if op in ("cur", "decompose"):
        f += 4.0 * k * (l * n + k * m) + k * k * n      # pivoted QRs, interpolation
    return dict(bytes=8.0 * (m * n + out), flops=f)


# ------------------------------------------------------------------- exact --
# Plain torch in FP64.  Singular vectors have no sign of their own: None.

def _mul32(c, const):
    """High and low words of the 32 x 32-bit products (int64 tensors)."""
    p = c * const                                       # wraps modulo 2^64
    return (p >> 32) & 0xFFFFFFFF, p & 0xFFFFFFFF


def _sketch(n, l, sid=0, batch=0):
    """The n x l sketch of the library's documentation: entry (i, j) = normal
    number j*n + i of the Philox4x32-10 stream `sid` (Box-Muller)."""
    pairs = torch.arange((n * l + 1) // 2, dtype=torch.int64, device=DEV)
    c0, c1 = pairs & 0xFFFFFFFF, pairs >> 32
    c2, c3 = torch.full_like(c0, sid), torch.full_like(c0, batch)
    k0, k1 = SEED & 0xFFFFFFFF, SEED >> 32
    for _ in range(10):
        h0, l0 = _mul32(c0, 0xD2511F53)
        h1, l1 = _mul32(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u1 = ((c0 >> 5).double() * 67108864.0 + (c1 >> 6).double() + 1.0) * 2.0 ** -53
    u2 = ((c2 >> 5).double() * 67108864.0 + (c3 >> 6).double()) * 2.0 ** -53
    rad, th = torch.sqrt(-2.0 * torch.log(u1)), 6.283185307179586 * u2
    z = torch.stack([rad * torch.cos(th), rad * torch.sin(th)], dim=1).reshape(-1)[:n * l]
    return z.view(l, n).T.contiguous()


def _basis(A, l, q, batch=0, orth=None):
    orth = orth or (lambda Y: torch.linalg.qr(Y)[0])
    Y = A @ _sketch(A.shape[1], l, batch=batch)
    for _ in range(q):
        Y = A @ orth(A.T @ orth(Y))
    return orth(Y)


def _pivoted_qr(B, k):
    """k greedy steps on the columns of B: the order, and S11^{-1} S12."""
    W, piv = B.clone(), []
    Qs = torch.zeros(B.shape[0], k, dtype=B.dtype, device=B.device)
    left = torch.ones(B.shape[1], dtype=torch.bool, device=B.device)
    for t in range(k):
        j = int(torch.where(left, W.square().sum(0), -1.0).argmax())
        piv.append(j)
        left[j] = False
        v = W[:, j].clone()
        v -= Qs @ (Qs.T @ v)
        v /= torch.linalg.vector_norm(v)
        Qs[:, t] = v
        W -= v[:, None] * (v @ W)
    rest = torch.nonzero(left).reshape(-1)
    J = torch.cat([torch.tensor(piv, device=B.device), rest])
    S = Qs.T @ B[:, J]
    T = torch.linalg.solve_triangular(torch.triu(S[:, :k]), S[:, k:].contiguous(), upper=True)
    return J, T


def _cur_core(A, J, T, k):
    Jr = _pivoted_qr(A[:, J[:k]].T.contiguous(), k)[0][:k]
    Qt, Rt = torch.linalg.qr(A[Jr, :].T.contiguous())
    M = Qt[J[:k]] + T @ Qt[J[k:]]
    return torch.linalg.solve_triangular(Rt, M.T.contiguous(), upper=True).T.contiguous()


def _svals(B, k):
    return torch.from_numpy(np.linalg.svd(torch.linalg.qr(B.T)[1].cpu().numpy(),
                                          compute_uv=False)[:k])


def _exact_pass(case, seed):
    A, scales, X, W = _pass_inputs(case, seed)
    m, n = case["m"], case["n"]
    Y = torch.empty(m, case["l"], dtype=torch.float64, device=DEV)
    Z = torch.zeros(n, case["l"], dtype=torch.float64, device=DEV)
    for r in range(0, m, 8192):
        B = A[r:r + 8192]
        if case["dtype"] == "f8":
            B = B.contiguous().view(torch.float8_e4m3fn).to(torch.float32).double() \
                * scales.double()
        else:
            B = B.double()
        Y[r:r + 8192] = B @ X.double()
        Z += B.T @ W[r:r + 8192].double()
    return [Y, Z, Z] if case["dtype"] == "f8" else [Y, Z]


def _exact_batch(case, seed):
    def orth(Y):
        for _ in range(2):
            L = torch.linalg.cholesky_ex(Y.T @ Y)[0]
            Y = torch.linalg.solve_triangular(L, Y.T.contiguous(), upper=False).T
        return Y.contiguous()

    ks = _batch_sizes(case)[2]
    lmax = int(ks.max()) + case["p"]
    Rs = torch.zeros(case["count"], lmax, lmax, dtype=torch.float64, device=DEV)
    for i, A in enumerate(_batch_matrices(case, seed)):
        A = A.double()
        l = min(int(ks[i]) + case["p"], *A.shape)
        B = _basis(A, l, case["q"], batch=i, orth=orth).T @ A
        Rs[i, :l, :l] = B @ orth(B.T.contiguous())
    s = np.linalg.svd(Rs.cpu().numpy(), compute_uv=False)
    return [None, torch.from_numpy(np.concatenate([s[i, :k] for i, k in enumerate(ks)])), None,
            None]


def _exact_qb(case, seed):
    A = _spectrum_matrix(seed, case["m"], case["n"], case["decay"])
    b, Qs, Bs, res = case["b"], [], [], 0.0

    def orth(Y):
        Q, Rr = torch.linalg.qr(Y)
        return Q * torch.sign(torch.diagonal(Rr))

    for i in range(case["M"]):
        Q = orth(A @ _sketch(A.shape[1], b, sid=5, batch=i))
        for _ in range(case["q"]):
            Q = orth(A @ orth(A.T @ Q))
        if Qs:
            P = torch.cat(Qs, dim=1)
            Q = Q - P @ (P.T @ Q)
        Q = orth(Q)
        B = Q.T @ A
        A -= Q @ B
        Qs.append(Q)
        Bs.append(B)
        res = float(torch.linalg.vector_norm(A))
        if res < case["tol"]:
            break
    return [torch.cat(Qs, dim=1), torch.cat(Bs), res, A, None]


def _exact_grad(case, seed):
    k, l = case["k"], min(case["k"] + case["p"], case["m"], case["n"])
    A = _spectrum_matrix(seed, case["m"], case["n"], case["decay"]).requires_grad_(True)
    Q = _basis(A, l, case["q"])
    B = Q.T @ A
    S = torch.linalg.svdvals(torch.linalg.qr(B.T)[1])[:k]
    r2 = (A - Q @ B).square().sum()
    (dA,) = torch.autograd.grad([S.sum() + r2], [A])
    return [None, S.detach(), None, r2.detach(), dA]


def exact(case, seed):
    op = case["op"]
    if op == "pass":
        return _exact_pass(case, seed)
    if op == "batch":
        return _exact_batch(case, seed)
    if op == "qb":
        return _exact_qb(case, seed)
    if op == "grad":
        return None if case["vectors"] else _exact_grad(case, seed)
    k = case["k"]
    A = _spectrum_matrix(seed, case["m"], case["n"], case["decay"])
    l = min(k + case["p"], case["m"], case["n"])
    B = _basis(A, l, case["q"]).T @ A
    if op == "svd":
        return [None, _svals(B, k), None, None]
    J, T = _pivoted_qr(B, k)
    U = _cur_core(A, J, T, k)
    if op == "cur":
        return [None, None, U, None]
    return dict(U=None, S=_svals(B, k), V=None, J=None, T=T, Jr=None, Ucur=U, info=None)
