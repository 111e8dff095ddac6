"""GPU parity of the column-sorted gather (X^T U on CSR rows) at every number of weight columns a lane can hold: one, two and
four per lane, whole and overlapping last lanes, with columns of one, of up to four, of around eight and of hundreds of
entries (pieces end at every 64th), padded result rows, and a matrix whose last piece is the end of the entry list."""
import numpy as np
import pytest
import torch

from tests.gpu_util import TOL, Pair, rel_err

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


def _columns(n, g):
    """CSR matrix whose column j has counts[j] entries in distinct rows."""
    counts = np.concatenate([[n, n - 1, 130, 129, 128, 127, 65, 64, 63, 0, 17, 16, 15, 9, 8, 7, 5, 4, 3, 2],
                             np.ones(300, int), [0, 0], g.integers(1, 6, 200), g.integers(1, 40, 60), [1]])
    p = counts.size
    rows = np.concatenate([np.sort(g.permutation(n)[:c]) for c in counts])
    cols = np.repeat(np.arange(p), counts)
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(n + 1, np.int64)
    np.add.at(rowptr, rows + 1, 1)
    return np.cumsum(rowptr), cols[order].astype(np.int32), g.standard_normal(rows.size), p


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("K,pad", [(1, 0), (2, 0), (3, 1), (4, 0), (5, 0), (6, 2), (7, 0), (8, 1), (9, 0), (16, 0), (19, 0), (21, 0),
                                   (32, 0), (33, 3), (63, 0)])
def test_gather_at_every_split_of_the_weight_columns(K, pad, dtype):
    g = np.random.default_rng(K)
    n = 300
    rowptr, colidx, vals, p = _columns(n, g)
    labels = g.integers(0, K + 1, n).astype(np.int32)
    d = dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals / 4, labels=labels, n=n, p=p, C=K + 1, K=K, lam=1e-3)
    pair = Pair(d, dtype, ldw=K + pad)
    Wh, Wd = pair.block(0.1 * g.standard_normal((p, K)))
    print(f"[case] gather K={K} dtype={dtype}", flush=True)
    G, f = pair.gpu.ssn_gradient(Wd)
    G_ref, f_ref = pair.oracle.gradient(Wh)
    torch.cuda.synchronize()
    assert rel_err(pair.host(G), G_ref) <= TOL[dtype] / 10
    if pad:
        assert torch.isnan(Wd[:, K:]).all()
    S = g.permutation(n)[:70]
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    Vh, Vd = pair.block(g.standard_normal((p, K)))
    HV = pair.gpu.ssn_hess_apply(Vd)
    torch.cuda.synchronize()
    assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= TOL[dtype] / 10
    pair.close()
