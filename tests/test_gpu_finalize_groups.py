"""GPU parity of directions and gradients where the sums behind the products change the elements per workgroup (2048, 8192,
16384), with an incomplete last group, and where a workgroup takes several groups (above 65536 elements)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import TOL, Pair, rel_err

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32

# n, p, C, nS, ldw
CASES = [
    (900, 682, 4, 300, None),            # 2046
    (900, 2048, 2, 300, None),           # 2048
    (900, 910, 10, 300, 10),             # 8190
    (900, 2048, 5, 300, None),           # 8192
    (900, 8192, 3, 300, None),           # 16384
    (900, 1639, 11, 300, 12),            # 16390
    (500, 6561, 11, 200, None),          # 65610: two groups in some workgroups
]


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,C,nS,ldw", CASES)
def test_groups_of_elements(n, p, C, nS, ldw, dtype):
    g = np.random.default_rng(p + C)
    X = g.standard_normal((n, p), dtype=np.float32).astype(np.float64) / np.sqrt(p)
    labels = g.integers(0, C, n).astype(np.int32)
    pair = Pair(dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.01), dtype, ldw=ldw)
    Wh, Wd = pair.block(0.5 * g.standard_normal((p, C - 1)))
    print(f"[case] groups n={n} p={p} C={C} dtype={dtype}", flush=True)
    G_ref, _ = pair.oracle.gradient(Wh)
    G, _ = pair.gpu.ssn_gradient(Wd)
    torch.cuda.synchronize()
    assert rel_err(pair.host(G), G_ref) <= TOL[dtype]
    S = np.sort(g.permutation(n)[:nS])
    Gh, Gd = pair.block(G_ref)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    # Rows of norm one and lambda = 0.01: H_S has eigenvalues between lambda and about 0.1, so a product's rounding (1e-16, or
    # the 6e-8 of fp32 operands) is amplified at most some tenfold; observed 1.3e-7 in fp32
    tol = 1e-10 if dtype == F64 else 2e-6
    ref, out = pair.oracle.cg(Wh, S, Gh, 1e-4, 6), pair.gpu.ssn_cg(Gd, 1e-4, 6)
    torch.cuda.synchronize()
    assert (out["iters"], out["flags"]) == (ref["iters"], ref["flags"])
    assert rel_err(pair.host(out["p"]), ref["p"]) <= tol
    pair.close()
