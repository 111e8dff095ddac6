"""GPU products on CSR data with infinite numbers in the right operand: a row or a column that stores no such entry is not touched
by it, one that does has the infinity arithmetic gives over its stored entries, and predictions follow.  Rows and columns of
every length around the rounds the kernels take their entries in (their last round is filled up with repeats of an entry,
which must not count, not even as zero times infinity)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import Pair

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


def _same(a, ref, tol):
    assert np.array_equal(np.isnan(a), np.isnan(ref)) and np.array_equal(np.isinf(a), np.isinf(ref))
    inf, fin = np.isinf(ref), np.isfinite(ref)
    assert np.array_equal(a[inf], ref[inf])
    np.testing.assert_allclose(a[fin], ref[fin], rtol=tol, atol=tol * np.max(np.abs(ref[fin])))


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 9, 19, 40])
def test_infinite_numbers_stay_where_they_are_stored(K, dtype):
    g = np.random.default_rng(K)
    lengths = np.concatenate([np.arange(0, 70), [90, 127, 128, 129, 200, 255, 256, 257, 300]])
    n, p = lengths.size, 400 + lengths.size       # row i's last entry is column 400 + i, which no other row stores
    rows = [np.append(np.sort(g.choice(400, size=m - 1, replace=False)), 400 + i) if m else np.zeros(0, int) for i, m in enumerate(lengths)]
    rowptr, colidx = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64), np.concatenate(rows).astype(np.int32)
    vals = g.uniform(0.5, 1.5, colidx.size)
    labels = g.integers(0, K + 1, n).astype(np.int32)
    pair = Pair(dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=K + 1, K=K, lam=0.0), dtype)
    nd = np.float64 if dtype == F64 else np.float32
    X = np.zeros((n, p))
    for i, c in enumerate(rows):
        X[i, c] = vals[rowptr[i]:rowptr[i + 1]].astype(nd)
    W = g.standard_normal((p, K))
    # one class with weights of +inf, one (from three columns on) with weights of -inf, in the last columns of some rows
    hot = {int(rows[i][-1]) for i in range(1, n, 4)}
    W[list(hot), 0] = np.inf
    if K > 2:
        W[[int(rows[i][-1]) for i in range(2, n, 9)], K - 1] = -np.inf
    Wh, Wd = pair.block(W)
    print(f"[case] infinite weights K={K} dtype={dtype}", flush=True)
    pred, _ = pair.gpu.ssn_predict(Wd)
    Z = np.zeros((n, K + 1))
    for i, c in enumerate(rows):
        if c.size:
            Z[i, :K] = X[i, c] @ Wh[c]
    assert not np.isnan(Z).any()
    top = np.sort(Z, axis=1)
    with np.errstate(invalid="ignore"):
        clear = (top[:, -1] == np.inf) | (top[:, -1] - top[:, -2] > 1e-3)
    assert np.array_equal(pred.cpu().numpy()[clear], np.argmax(Z, axis=1)[clear])
    # the product: probabilities of finite weights, an operand with infinities
    W0h, W0d = pair.block(0.01 * g.standard_normal((p, K)))
    V = g.standard_normal((p, K))
    V[[400 + 3, 400 + 9, 400 + 17], 1] = np.inf
    Vh, Vd = pair.block(V)
    S = np.arange(n)
    HV = pair.gpu.ssn_hessvec(W0d, pair.idx(S), Vd)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore", over="ignore"):
        E = np.exp(X @ W0h)
        P = E / (1.0 + E.sum(axis=1, keepdims=True))
        Zv = np.zeros((n, K))
        for i, c in enumerate(rows):
            if c.size:
                Zv[i] = X[i, c] @ Vh[c]
        U = P * Zv - P * (P * Zv).sum(axis=1, keepdims=True)
        ref = np.zeros((p, K))
        for i, c in enumerate(rows):
            ref[c] += np.outer(X[i, c], U[i])
        ref = ref / n + 0.0 * Vh
    _same(pair.host(HV), ref, 1e-10 if dtype == F64 else 1e-4)
    pair.close()
