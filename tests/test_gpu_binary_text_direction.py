"""GPU parity of Newton directions on CSR samples with one weight column (three launches per product): samples of less than a
wave of pieces, columns of one piece, of more pieces than a wave and than the steps behind it, more pieces than the largest
grid has threads, samples without an entry, padded weights, repeated rows, a zero gradient."""
import numpy as np
import pytest
import torch

from tests.gpu_util import Pair, rel_err

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32

# n, p, entries per row, nS (None: rows without an entry only), ldw, repeats
CASES = [
    (60, 300, 6, 5, None, False),
    (300, 40, 8, 200, 2, True),
    (5000, 50, 8, 4700, None, False),             # columns of seventy pieces: beyond a wave
    (30000, 6, 4, 25000, 3, True),                # of four hundred: two steps behind the wave
    (2600, 400000, 130, 2500, None, False),       # 300 000 pieces: a second trip of the largest grid
    (400, 900, 10, None, None, False),
]


def _matrix(n, p, per, g):
    """Every eleventh row is empty; half of a row's columns among the first few, half anywhere."""
    rows, vals = [], []
    for i in range(n):
        m = 0 if i % 11 == 5 else per
        few = g.integers(0, min(p, 3 * per), m - m // 2 if p < 1000 else 0)
        c = np.unique(np.concatenate([few, g.integers(0, p, m // 2 if p < 1000 else m)]).astype(np.int64))
        v = g.standard_normal(c.size)
        rows.append(c)
        vals.append(v / max(np.linalg.norm(v), 1e-30))
    rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    return rowptr.astype(np.int64), np.concatenate(rows).astype(np.int32), np.concatenate(vals)


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,per,nS,ldw,repeats", CASES)
def test_direction_with_one_weight_column(n, p, per, nS, ldw, repeats, dtype):
    g = np.random.default_rng(n + 7 * p)
    rowptr, colidx, vals = _matrix(n, p, per, g)
    labels = g.integers(0, 2, n).astype(np.int32)
    pair = Pair(dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=2, K=1, lam=0.01), dtype, ldw=ldw)
    Wh, Wd = pair.block(0.3 * g.standard_normal((p, 1)))
    S = np.arange(5, n, 11) if nS is None else np.sort(g.integers(0, n, nS) if repeats else g.permutation(n)[:nS])
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    # Rows of norm one and lambda = 0.01: H_S has eigenvalues between lambda and about 0.3, so a product's rounding (1e-16,
    # or the 6e-8 of fp32 operands) is amplified at most some thirtyfold; observed 9e-8 in fp32.
    # (theta 9e-6: below what is left to the row space of the sample)
    tol = 1e-10 if dtype == F64 else 2e-6
    for theta, T in [(9e-6, 5), (9e-6, 1), (0.2, 9)]:
        print(f"[case] binary direction n={n} p={p} nS={nS} dtype={dtype} theta={theta} T={T}", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, theta, T)
        out = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"])
        # (a sample without an entry has no pieces to sum)
        assert pair.gpu.ssn_direction_form() == (3 if nS is None else 5) or theta > 1e-5 and pair.gpu.ssn_direction_form() == 4
        np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=100 * tol)
        np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=100 * tol, atol=tol * np.linalg.norm(Gh))
        np.testing.assert_allclose(out["sHs"], ref["sHs"], rtol=100 * tol)
        assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
        again = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert torch.equal(again["p"][:, :1], out["p"][:, :1])
    zero = pair.gpu.ssn_cg(torch.zeros_like(Gd), 9e-6, 3)
    torch.cuda.synchronize()
    assert zero["iters"] == 0 and not zero["p"][:, :1].any()
    pair.close()
