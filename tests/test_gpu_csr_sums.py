"""How far fp32 gradients on CSR data are from fp64: what the order of the sums leaves.  A row's products are added in two sums
of four per round of a lane, a column's in pieces of 64 entries, two sums of four products each time."""
import numpy as np
import pytest
import torch

from tests.gpu_util import Pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,per,K,bound", [(3000, 300, 200, 9, 7.4e-8), (3000, 300, 200, 5, 7.7e-8), (1500, 3000, 450, 9, 5.3e-8),
                                             (1500, 3000, 450, 2, 6.7e-8)])
def test_rounding_of_fp32_gradients(n, p, per, K, bound):
    """All values positive, so the rounding of every addition is one of the whole sum's size.  Relative errors of the gradient over
    four data sets, in the mean: 6.8e-8, 7.0e-8, 4.9e-8 and 6.2e-8 in this order; with one chain of every second product (a
    piece: two chains of 32) 7.9e-8, 8.1e-8, 5.6e-8 and 7.0e-8.  The bounds lie between."""
    errors = []
    for seed in range(4):
        g = np.random.default_rng(seed * 100 + K)
        w = 1.0 / np.arange(1, p + 1) ** 0.7
        w /= w.sum()
        rows = [np.unique(g.choice(p, size=per, p=w)) for _ in range(n)]
        rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
        colidx = np.concatenate(rows).astype(np.int32)
        vals = np.abs(g.standard_normal(colidx.size)).astype(np.float32) / np.float32(np.sqrt(per))
        labels = g.integers(0, K + 1, n).astype(np.int32)
        d = dict(layout="csr", rowptr=rowptr, colidx=colidx, vals=vals, labels=labels, n=n, p=p, C=K + 1, K=K, lam=1e-3)
        pair = Pair(d, torch.float32)
        Wh, Wd = pair.block(0.3 * g.standard_normal((p, K)))
        G, _ = pair.gpu.ssn_gradient(Wd)
        torch.cuda.synchronize()
        ref = pair.oracle.gradient(Wh)[0]
        errors.append(np.linalg.norm(pair.host(G) - ref) / np.linalg.norm(ref))
        pair.close()
    print(f"[case] sums n={n} p={p} K={K}: {np.mean(errors):.3e}", flush=True)
    assert np.mean(errors) <= bound
