"""Device memory that directions in the row space of a CSR sample take: the dense copy of the frequent columns has a row for each
of them, and there are no more than the sample has columns."""
import numpy as np
import pytest
import torch

from paper_1802_09113_amd.binding import Context

pytestmark = pytest.mark.gpu


def test_long_rows_over_few_columns():
    """2048 rows of some 3000 entries over 4000 columns: 6 million entries would make 24 000 columns of 256 entries (390 MB), but
    all 4000 columns are 66 MB beside 34 MB of the Gram matrix and 2 MB of vectors; allocations are an eighth larger."""
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    n, p, C, nS, T = 2100, 4000, 5, 2048, 30
    mask = torch.rand(n, p, generator=g, device="cuda") < 0.75
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(mask.sum(1), 0).to(torch.int32)
    colidx = mask.nonzero()[:, 1].to(torch.int32)
    vals = torch.randn(colidx.numel(), generator=g, device="cuda", dtype=torch.float64) / 50.0
    labels = torch.randint(0, C, (n,), generator=g, device="cuda", dtype=torch.int32)
    ctx = Context(labels, C, 0.01, csr=(rowptr, colidx, vals), p=p)
    W = 0.1 * torch.randn(p, C - 1, generator=g, device="cuda", dtype=torch.float64)
    S = torch.sort(torch.randperm(n, generator=g, device="cuda")[:nS]).values.to(torch.int32)
    G, _ = ctx.ssn_gradient(W)
    ctx.ssn_hess_prepare(W, S)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    print("[case] row space workspace", flush=True)
    out = ctx.ssn_cg(G, 1e-4, T)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    print(f"[case] {used / 1e6:.0f} MB", flush=True)
    assert 60e6 < used < 250e6             # (below: the row space did not serve it)
    # against Alg. 2 on the dense rows
    X = torch.zeros(n, p, device="cuda", dtype=torch.float64)
    X[mask] = vals
    Xs = X[S.long()]
    P = torch.softmax(torch.cat([Xs @ W, torch.zeros(nS, 1, device="cuda", dtype=torch.float64)], 1), 1)[:, : C - 1]
    pd, r = torch.zeros_like(W), -G[:, : C - 1]
    s, rr = r.clone(), (r * r).sum()
    g0, least, best = rr.sqrt(), rr.sqrt(), r.clone()
    for _ in range(T):
        Z = Xs @ s
        U = P * Z - P * (P * Z).sum(1, keepdim=True)
        H = Xs.T.contiguous() @ U / nS + 0.01 * s
        alpha = rr / (s * H).sum()
        pd, r = pd + alpha * s, r - alpha * H
        new = (r * r).sum()
        if new.sqrt() <= least:
            least, best = new.sqrt(), pd.clone()
        if new.sqrt() <= 1e-4 * g0:
            break
        s, rr = r + new / rr * s, new
    assert float((out["p"][:, : C - 1] - best).norm() / best.norm()) <= 1e-9
    ctx.close()
