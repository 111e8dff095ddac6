"""GPU parity on CSR rows that store a column more than once (its values add up): a column of nearly every row, of a handful
of rows and of one row, stored two and three times, in samples with and without repeated rows, for one and several weight
columns, and in whole iterations.  Results are the oracle's and the same bits on repetition."""
import numpy as np
import pytest
import torch

from tests.gpu_util import TOL, Pair, rel_err, rel_scalar

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


def _matrix(n, p, mean, g):
    """Columns 0 and 1 are in almost every row; column 0 is stored twice, column 1 three times in two rows of three, column 2
    twice in a dozen rows, column 3 twice in one row."""
    rows, vals = [], []
    for i in range(n):
        c = np.sort(g.choice(np.arange(4, p), size=int(g.integers(1, 2 * mean)), replace=False))
        if i % 19 != 7:
            c = np.concatenate([[0, 0], [1] * (3 if i % 3 else 1), c])
        if i % (n // 12) == 3:
            c = np.concatenate([c, [2, 2]])
        if i == n // 2:
            c = np.concatenate([c, [3, 3]])
        c = np.sort(c)
        v = g.standard_normal(c.size)
        rows.append(c)
        vals.append(v / np.linalg.norm(v))
    rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    return rowptr.astype(np.int64), np.concatenate(rows).astype(np.int32), np.concatenate(vals)


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,mean,C,nS,repeats", [(400, 5000, 20, 5, 200, False), (900, 3000, 25, 20, 300, True), (1400, 9000, 15, 4, 1200, True),
                                                   (700, 4000, 30, 2, 150, False)])
def test_columns_stored_more_than_once(n, p, mean, C, nS, repeats, dtype):
    g = np.random.default_rng(n + C)
    rowptr, colidx, vals = _matrix(n, p, mean, g)
    labels = g.integers(0, C, n).astype(np.int32)
    K = C - 1
    pair = Pair(dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=C, K=K, lam=0.01), dtype)
    Wh, Wd = pair.block(0.3 * g.standard_normal((p, K)))
    print(f"[case] repeated columns n={n} C={C} nS={nS} dtype={dtype}", flush=True)
    G_ref, f_ref = pair.oracle.gradient(Wh)
    G, f = pair.gpu.ssn_gradient(Wd)
    torch.cuda.synchronize()
    assert rel_scalar(f, f_ref) <= TOL[dtype] / 10 and rel_err(pair.host(G), G_ref) <= TOL[dtype] / 10
    S = np.sort(g.integers(0, n, nS)) if repeats else np.sort(g.permutation(n)[:nS])
    Gh, Gd = pair.block(G_ref)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    Vh, Vd = pair.block(g.standard_normal((p, K)))
    HV = pair.gpu.ssn_hess_apply(Vd)
    torch.cuda.synchronize()
    assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= TOL[dtype] / 10
    # rows of norm one, lambda 0.01: a product's rounding (1e-16 / 6e-8) is amplified at most some thirtyfold; observed 3e-7 in fp32
    tol = 1e-10 if dtype == F64 else 5e-6
    for theta, T in [(1e-4, 5), (0.2, 20)]:
        ref, out = pair.oracle.cg(Wh, S, Gh, theta, T), pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"])
        assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
        for _ in range(3):
            pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
            again = pair.gpu.ssn_cg(Gd, theta, T)
            torch.cuda.synchronize()
            assert torch.equal(again["p"][:, :K], out["p"][:, :K])
    Ss = np.stack([np.sort(g.permutation(n)[:nS]) for _ in range(3)]).astype(np.int32)
    W0h, W0d = pair.block(0.1 * g.standard_normal((p, K)))
    _, log_ref, _ = pair.oracle.ssn(W0h, Ss, theta=1e-3, T=8)
    log, _ = pair.gpu.ssn_solve(W0d, pair.idx(Ss), theta=1e-3, T=8)
    torch.cuda.synchronize()
    np.testing.assert_allclose([r["f"] for r in log], log_ref[:, 0], rtol=1e-9 if dtype == F64 else 1e-4)
    pair.close()
