"""GPU products on a column-sorted view that is built again with more entries than it was allocated for, in the capacity the
first build left: rows of exactly eight entries, and samples whose entry lists end at each of the last places of it."""
import numpy as np
import pytest
import torch

from tests.gpu_util import TOL, Pair, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("view", ["filter", "sort"])
def test_samples_up_to_the_capacity_of_the_first(view, dtype, monkeypatch):
    """An array grown for N entries has room for N + N / 8 + 64: 8000 rows of eight entries, 72064 then, are followed by
    samples of 9007 and 9008 rows, 72056 and 72064 entries."""
    if view == "sort":
        monkeypatch.setenv("SSN_CSR_VIEW", "sort")
    g = np.random.default_rng(8)
    n, p, C, per = 9100, 5000, 4, 8
    colidx = np.concatenate([np.sort(g.choice(p, size=per, replace=False)) for _ in range(n)]).astype(np.int32)
    d = dict(layout="csr", rowptr=np.arange(n + 1, dtype=np.int64) * per, colidx=colidx, vals=g.standard_normal(n * per),
             labels=g.integers(0, C, n).astype(np.int32), n=n, p=p, C=C, K=C - 1, lam=0.01)
    pair = Pair(d, dtype)
    Wh, Wd = pair.block(0.1 * g.standard_normal((p, C - 1)))
    Vh, Vd = pair.block(g.standard_normal((p, C - 1)))
    for nS in (8000, 9007, 9008):
        print(f"[case] entry list view={view} dtype={dtype} nS={nS}", flush=True)
        S = g.permutation(n)[:nS]
        HV = pair.gpu.ssn_hessvec(Wd, pair.idx(S), Vd)
        torch.cuda.synchronize()
        assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= TOL[dtype] / 10
    pair.close()
