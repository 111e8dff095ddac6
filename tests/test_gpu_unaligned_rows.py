"""Two-kernel dense path on rows that are aligned to their element only: 16-byte loads from the width on where two trips
of them fit (128 fp32, 64 fp64 features), element loads below, and a workgroup per row block on few or wide rows.  Every
mode against the oracle; the widths put the end of the last whole trip at, before and behind the end of a row."""
import numpy as np
import pytest
import torch

from paper_1802_09113_amd import synth
from tests.gpu_util import TOL, Pair, rel_err, rel_scalar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,K", [(203, 63, 18), (203, 64, 18), (203, 65, 18), (203, 127, 18), (203, 128, 18), (203, 129, 18),
                                   (1003, 331, 23), (203, 513, 18), (203, 2051, 3), (8203, 2051, 3), (203, 2051, 18)])
def test_rows_of_any_alignment(n, p, K, dtype):
    g = np.random.default_rng(3)
    d = dict(layout="dense", n=n, p=p, C=K + 1, K=K, lam=1e-2, X=g.standard_normal((n, p), dtype=np.float32),
             labels=g.integers(0, K + 1, size=n).astype(np.int32))
    pair = Pair(d, dtype, xoff=1)
    tol = TOL[dtype]
    print(f"[case] unaligned rows n={n} p={p} K={K} dtype={dtype}", flush=True)
    Wh, Wd = pair.block(synth.probe(p, K, sub=1, scale=0.02))
    G_ref, f_ref = pair.oracle.gradient(Wh)
    assert rel_scalar(pair.gpu.ssn_objective(Wd), f_ref) <= tol
    G, f = pair.gpu.ssn_gradient(Wd)
    torch.cuda.synchronize()
    assert rel_scalar(f, f_ref) <= tol and rel_err(pair.host(G), G_ref) <= tol
    pred, _ = pair.gpu.ssn_predict(Wd)
    flips = int(np.count_nonzero(pred.cpu().numpy() != pair.oracle.predict(Wh)))
    assert flips <= (0 if dtype == torch.float64 else max(1, n // 500))
    Vh, Vd = pair.block(synth.probe(p, K, sub=2))
    S = synth.sample_rows(n, 100)
    HV = pair.gpu.ssn_hessvec(Wd, pair.idx(S), Vd)
    torch.cuda.synchronize()
    assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= tol
    # a step far too long: up to sixteen weight columns its trials go over the margins of both operands
    Gh, Gd = pair.block(G_ref)
    Ph, Pd = pair.block(-2e3 * G_ref)
    ref = pair.oracle.linesearch(Wh, Ph, Gh, f_ref, imax=60)
    out = pair.gpu.ssn_linesearch(Wd, Pd, Gd, pair.gpu.ssn_objective(Wd), imax=60)
    assert out["alpha"] == ref["alpha"] and rel_scalar(out["f_new"], ref["f_new"]) <= tol
    pair.close()
