"""GPU parity of Newton directions on a formed sub-sampled Hessian (dense problems of a few hundred weights): every strip
count per thread, features below, at and above the strips of eight and the 16- and 64-feature tiles, one and several row
chunks, padded weights and rows, and the shapes on either side of what the form serves."""
import numpy as np
import pytest
import torch

from paper_1802_09113_amd.binding import Context
from tests.gpu_util import Pair, rel_err

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32

# n, p, C, nS, ldw, ldx.  Class pairs C (C - 1) / 2; the form's limit is some 32 000 (fp64) / 70 000 (fp32) elements
CASES = [
    (300, 1, 2, 40, None, None),          # one weight
    (400, 8, 33, 64, None, None),         # 528 class pairs, one strip a row
    (400, 9, 12, 1, 13, None),            # one row, two strips a row, padded weights
    (700, 16, 6, 67, None, 19),           # one feature tile, padded rows
    (900, 33, 5, 300, None, None),        # three feature tiles, chunks that the CG kernel adds itself
    (4000, 54, 7, 1500, None, None),      # fp32: nine strips a thread; fp64: too many blocks, the matrix-free form
    (1000, 40, 7, 200, 7, None),          # fp32: six strips a thread, blocks in fp32
    (2000, 50, 3, 2000, 3, 50),           # every row
    (5000, 64, 4, 4999, None, None),      # whole tiles; twelve and more chunks
    (1500, 65, 3, 700, 5, 67),            # two feature blocks, one of them one feature wide
    (900, 130, 2, 500, None, None),       # binary, three feature blocks
    (700, 176, 2, 333, None, None),       # binary, fp64: the widest served
    (800, 264, 2, 120, None, 265),        # binary, fp32: the widest served; fp64: not
    (600, 273, 2, 90, None, None),        # binary, not served
]
MATRIX_FREE = {F32: {(273, 2)}, F64: {(273, 2), (264, 2), (8, 33), (54, 7), (40, 7)}}       # p, C


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,C,nS,ldw,ldx", CASES)
def test_direction_on_the_formed_hessian(n, p, C, nS, ldw, ldx, dtype):
    g = np.random.default_rng(1000 * p + C)
    X = g.standard_normal((n, p)) / np.sqrt(p)
    labels = g.integers(0, C, n).astype(np.int32)
    pair = Pair(dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.05), dtype, ldw=ldw, ldx=ldx)
    Wh, Wd = pair.block(0.5 * g.standard_normal((p, C - 1)))
    S = g.integers(0, n, nS)                       # a multiset
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    # Features of norm one: the data term has eigenvalues of at most max(1, p / nS), lambda is 0.05, so the rounding of a product
    # (a few 1e-16, or the 6e-8 of fp32 operands) is amplified by some tens in the direction and by the condition number, at
    # most a few hundred, in the scalars of an iteration; observed 1e-13 / 1.2e-7.
    tol = 1e-10 if dtype == F64 else 2e-6
    for theta, T in [(1e-30, 5), (0.2, 9)]:
        print(f"[case] direction n={n} p={p} C={C} nS={nS} dtype={dtype} theta={theta}", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, theta, T)
        if theta < 1e-20 and np.min(ref["rnorm"]) < 1e-6 * np.linalg.norm(Gh):
            ref = pair.oracle.cg(Wh, S, Gh, 1e-3, T)        # a handful of weights: converged within the budget
            theta = 1e-3
        out = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert pair.gpu.ssn_direction_form() == (1 if (p, C) in MATRIX_FREE[dtype] else 2)
        assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"])
        np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=100 * tol if dtype == F32 else tol)
        np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=100 * tol, atol=tol * np.linalg.norm(Gh))
        np.testing.assert_allclose(out["sHs"], ref["sHs"], rtol=100 * tol)
        assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
        again = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert torch.equal(again["p"][:, : C - 1], out["p"][:, : C - 1])
    pair.close()


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
def test_formed_hessian_and_an_indefinite_product(dtype):
    """lambda = 0 and rows of zeros: H_S is zero, s^T H s is not positive, the direction is the steepest descent."""
    n, p, C = 200, 20, 4
    X = np.zeros((n, p))
    X[0] = 1.0
    labels = (np.arange(n) % C).astype(np.int32)
    pair = Pair(dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.0), dtype)
    Wh, Wd = pair.block(np.ones((p, C - 1)))
    S = np.arange(10, 60)
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    ref = pair.oracle.cg(Wh, S, Gh, 1e-4, 6)
    out = pair.gpu.ssn_cg(Gd, 1e-4, 6)
    torch.cuda.synchronize()
    assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"]) == (1, 2)
    np.testing.assert_array_equal(pair.host(out["p"]), -Gh)
    pair.close()


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("theta", [-1.0, 0.0])
def test_formed_hessian_and_a_tolerance_that_is_never_met(theta, dtype):
    """||r|| <= theta ||g|| does not hold for a theta of zero or below while a residual is left: all T products are made."""
    n, p, C, nS, T = 500, 40, 3, 200, 6
    g = np.random.default_rng(5)
    X = g.standard_normal((n, p)) / np.sqrt(p)
    pair = Pair(dict(layout="dense", X=X, labels=g.integers(0, C, n).astype(np.int32), n=n, p=p, C=C, K=C - 1, lam=0.05), dtype)
    Wh, Wd = pair.block(0.1 * g.standard_normal((p, C - 1)))
    S = g.permutation(n)[:nS]
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    ref, out = pair.oracle.cg(Wh, S, Gh, theta, T), pair.gpu.ssn_cg(Gd, theta, T)
    torch.cuda.synchronize()
    assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"]) == (T, 0)
    assert rel_err(pair.host(out["p"]), ref["p"]) <= (1e-10 if dtype == F64 else 2e-6)
    pair.close()


def test_formed_hessian_and_products_below_the_normal_numbers():
    """Data of 1e-78: s^T H s of about 1e-312 is a subnormal number with some eleven digits, whose reciprocal overflows; the steps
    ||r||^2 / s^T H s are ordinary ones of 1e156.  Sums of fp64 products to 1e-12, then three iterations."""
    n, p, C, nS = 300, 24, 3, 150
    g = np.random.default_rng(6)
    X = 1e-78 * g.standard_normal((n, p))
    pair = Pair(dict(layout="dense", X=X, labels=g.integers(0, C, n).astype(np.int32), n=n, p=p, C=C, K=C - 1, lam=0.0), F64)
    Wh, Wd = pair.block(np.zeros((p, C - 1)))
    S = g.permutation(n)[:nS]
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    ref, out = pair.oracle.cg(Wh, S, Gh, 1e-4, 3), pair.gpu.ssn_cg(Gd, 1e-4, 3)
    torch.cuda.synchronize()
    assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"]) == (3, 0)
    np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=1e-7)
    assert rel_err(pair.host(out["p"]) * 1e-78, ref["p"] * 1e-78) <= 1e-7
    pair.close()


def _exact_direction(H, g, theta, T):
    """Alg. 2 on a formed matrix, in fp64."""
    p, r = torch.zeros_like(g), -g
    s, best, g0 = r.clone(), -g, g.norm()
    least = g0
    for _ in range(T):
        Hs = H @ s
        rr = r @ r
        alpha = rr / (s @ Hs)
        p, r = p + alpha * s, r - alpha * Hs
        if r.norm() <= least:
            least, best = r.norm(), p.clone()
        if r.norm() <= theta * g0:
            break
        s = r + (r @ r) / rr * s
    return best


@pytest.mark.parametrize("n,p,K,nS,T,lam,bound", [(100000, 8, 31, 1000, 10, 1e-3, 1.6e-7), (60000, 54, 6, 20000, 10, 1e-3, 1.5e-7),
                                                  (300000, 50, 3, 300000, 24, 1e-3, 1.1e-7)])
def test_rounding_of_fp32_directions(n, p, K, nS, T, lam, bound):
    """fp32 directions against fp64 ones of the same fp32 data, mean over four data sets: what forming H_S costs in precision.
    Sums over the sample's rows (up to 300000) and products are carried in fp64: 1.2e-7, 1.3e-7 and 0.7e-7 in this order, as
    matrix-free products leave (1.2e-7, 1.1e-7, 0.8e-7); with fp32 sums and products it was 3.4e-7, 1.9e-7 and 1.5e-7."""
    errors = []
    for seed in range(4):
        g = torch.Generator(device="cuda")
        g.manual_seed(77 * seed + p)
        X = torch.randn(n, p, generator=g, device="cuda", dtype=F32)
        score = X @ torch.randn(p, K + 1, generator=g, device="cuda") / np.sqrt(p)
        labels = (score + torch.randn(n, K + 1, generator=g, device="cuda")).argmax(1).to(torch.int32)
        W = (0.1 * torch.randn(p, K, generator=g, device="cuda")).contiguous()
        S = torch.sort(torch.randperm(n, generator=g, device="cuda")[:nS]).values.to(torch.int32)
        ctx = Context(labels, K + 1, lam, X=X)
        G, _ = ctx.ssn_gradient(W)
        ctx.ssn_hess_prepare(W, S)
        out = ctx.ssn_cg(G, 1e-4, T)["p"][:, :K].double()
        torch.cuda.synchronize()
        Xs = X[S.long()].double()
        P = torch.softmax(torch.cat([Xs @ W.double(), torch.zeros(nS, 1, device="cuda", dtype=F64)], 1), 1)[:, :K]
        H = torch.zeros(K, p, K, p, device="cuda", dtype=F64)
        for a in range(K):
            for b in range(a, K):
                q = P[:, a] * ((1.0 if a == b else 0.0) - P[:, b])
                H[a, :, b, :] = Xs.T.contiguous() @ (Xs * q[:, None])
                H[b, :, a, :] = H[a, :, b, :]
        H = H.reshape(K * p, K * p) / nS + lam * torch.eye(K * p, device="cuda", dtype=F64)
        ref = _exact_direction(H, G[:, :K].double().T.reshape(-1), 1e-4, T).reshape(K, p).T
        errors.append(float((out - ref).norm() / ref.norm()))
        ctx.close()
    print(f"[case] rounding n={n} p={p} K={K} nS={nS}: {np.mean(errors):.3e}", flush=True)
    assert np.mean(errors) <= bound
