"""GPU parity of Newton directions on CSR samples in the sample's row space: samples around the tiles of 16, 32 and 64 rows
and the change of the product's share at 1024, weight columns around the class tiles of 16, columns below, at and above
the length that makes one frequent, empty rows, repeated rows, padded weights, and samples on either side of what the form
serves; the form that served a direction is asked for."""
import numpy as np
import pytest
import torch

from tests.gpu_util import Pair, rel_err

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32

# n, p, mean row length, C, nS, ldw, sample with repeats
CASES = [
    (60, 300, 12, 2, 1, None, False),
    (900, 4000, 20, 2, 333, 3, True),             # one weight column, padded
    (200, 900, 20, 3, 63, 4, False),
    (200, 900, 20, 17, 64, None, False),          # whole class tile, whole row tile
    (300, 700, 30, 18, 65, 19, True),             # a class more, a row more
    (400, 3000, 25, 34, 130, None, True),         # three class tiles
    (900, 20000, 15, 20, 500, None, False),       # support far wider than the sample
    (1300, 2500, 12, 5, 1024, None, False),
    (1300, 2500, 12, 5, 1025, 6, True),           # shares of 128 rows, the last one half of it padding
    (2500, 4000, 8, 3, 1930, None, False),        # sixteen shares, the last one of 64 rows
    (2500, 4000, 8, 6, 2048, None, True),         # the largest sample served
    (2500, 4000, 8, 6, 2049, None, True),         # not served
]


def _matrix(n, p, mean, g):
    """Rows of distinct columns whose frequencies fall like 1/rank: a few columns in most rows, many in one or two.
    Every eleventh row is empty."""
    w = 1.0 / np.arange(1, p + 1)
    w /= w.sum()
    rows, vals = [], []
    for i in range(n):
        m = 0 if i % 11 == 5 else int(np.clip(g.poisson(mean), 1, p))
        c = np.unique(g.choice(p, size=m, p=w)) if m else np.zeros(0, dtype=np.int64)
        v = g.standard_normal(c.size)
        rows.append(c)
        vals.append(v / max(np.linalg.norm(v), 1e-30))
    rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    return rowptr.astype(np.int64), np.concatenate(rows).astype(np.int32), np.concatenate(vals)


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,mean,C,nS,ldw,repeats", CASES)
def test_direction_in_the_row_space(n, p, mean, C, nS, ldw, repeats, dtype):
    g = np.random.default_rng(n + 7 * p + C)
    rowptr, colidx, vals = _matrix(n, p, mean, g)
    labels = g.integers(0, C, n).astype(np.int32)
    d = dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.01)
    pair = Pair(d, dtype, ldw=ldw)
    K = C - 1
    Wh, Wd = pair.block(0.3 * g.standard_normal((p, K)))
    S = np.sort(g.integers(0, n, nS) if repeats else g.permutation(n)[:nS])
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    # Rows of norm one and lambda = 0.01: H_S has eigenvalues between lambda and about 0.3, so a product's rounding (1e-16,
    # or the 6e-8 of fp32 operands) is amplified at most some thirtyfold; observed 1e-14 / 1.2e-7.
    tol = 1e-10 if dtype == F64 else 2e-6
    form = 3 if nS > 2048 else 4
    more = 14 if C == 2 else 4 if nS > 1200 else 0      # with one weight column or many rows the form pays from more products on
    for theta, T in [(1e-4, 6 + more), (0.2, 9 + more)]:
        print(f"[case] direction n={n} p={p} C={C} nS={nS} dtype={dtype} theta={theta}", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, theta, T)
        out = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert pair.gpu.ssn_direction_form() == form
        assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"])
        np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=100 * tol)
        np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=100 * tol, atol=tol * np.linalg.norm(Gh))
        np.testing.assert_allclose(out["sHs"], ref["sHs"], rtol=100 * tol)
        assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
        again = pair.gpu.ssn_cg(Gd, theta, T)
        pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
        anew = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert torch.equal(again["p"][:, :K], out["p"][:, :K]) and torch.equal(anew["p"][:, :K], out["p"][:, :K])
    # the right-hand side in the rows' span, no column outside the sample's: what cancels in r.r is largest here
    u = g.standard_normal((nS, K))
    R = np.zeros((p, K))
    for i, s in enumerate(S):
        e = slice(rowptr[s], rowptr[s + 1])
        R[colidx[e]] += np.outer(vals[e], u[i])
    Gh, Gd = pair.block(R)
    ref = pair.oracle.cg(Wh, S, Gh, 1e-4, 5 + more)
    out = pair.gpu.ssn_cg(Gd, 1e-4, 5 + more)
    torch.cuda.synchronize()
    assert out["iters"] == ref["iters"] and pair.gpu.ssn_direction_form() == form
    assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
    pair.close()


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
def test_steps_with_directions_in_the_row_space(dtype):
    """Alg. 1 (the next sample's Gram matrix is made beside the line search) against the oracle."""
    g = np.random.default_rng(3)
    n, p, C, nS = 700, 5000, 4, 150
    rowptr, colidx, vals = _matrix(n, p, 40, g)
    labels = g.integers(0, C, n).astype(np.int32)
    pair = Pair(dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.01), dtype)
    Wh, Wd = pair.block(0.1 * g.standard_normal((p, C - 1)))
    S = np.stack([np.sort(g.permutation(n)[:nS]) for _ in range(4)]).astype(np.int32)
    W_ref, log_ref, _ = pair.oracle.ssn(Wh, S, theta=1e-4, T=10)
    log, _ = pair.gpu.ssn_solve(Wd, pair.idx(S), theta=1e-4, T=10)
    torch.cuda.synchronize()
    assert pair.gpu.ssn_direction_form() == 4
    np.testing.assert_allclose([r["f"] for r in log], log_ref[:, 0], rtol=1e-10 if dtype == F64 else 1e-6)
    assert rel_err(pair.host(Wd), W_ref) <= (1e-8 if dtype == F64 else 1e-5)
    pair.close()
