"""Two-kernel dense path on rows that are aligned to their element only: 16-byte loads or element loads by width, rows and
class tiles, a workgroup per row block on few or wide rows.  Every mode against the oracle; the widths put the end of the
last whole trip, and of the last whole tile of 64 features, at, before and behind the end of a row."""
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
    _check(n, p, K, dtype, 1, 100)


# One weight tile (K <= 16) and a wave per row block, which the shapes above do not reach: 1301 and 1087 features on more
# than 512 row blocks (two row blocks per trip if aligned, one if not), 1031 on more than 1024 (fp64 takes the 16-byte loads
# from there on).  Two tiles: 575 features end 63 behind a trip and a tile; 2051 row blocks are a round more for 16-byte
# loads in fp64 than for element loads, 513 are not.  The sample is every row where products shall take these forms too.
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("off", [0, 1], ids=["off0", "off1"])
@pytest.mark.parametrize("n,p,K,nS", [(8209, 1301, 3, 8209), (8209, 1300, 3, 8209), (8209, 1087, 10, 300), (16401, 1031, 3, 16401),
                                      (8209, 575, 18, 8209), (32801, 68, 18, 32801), (8209, 68, 18, 8209)])
def test_wave_per_row_block(n, p, K, nS, off, dtype):
    _check(n, p, K, dtype, off, nS, path=1)


# Shapes of the one-pass path, whose line search still forms the margins of both operands with the two-kernel path's rows
# kernel: one tile (2 K <= 16) of 16-byte or element loads, two tiles, and a workgroup per row block
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("off", [0, 1], ids=["off0", "off1"])
@pytest.mark.parametrize("n,p,K", [(1003, 331, 3), (1003, 127, 3), (16401, 131, 3), (16401, 127, 3), (8209, 577, 3), (1003, 577, 3),
                                   (1003, 191, 12)])
def test_margins_of_one_pass_shapes(n, p, K, off, dtype):
    _check(n, p, K, dtype, off, 100, path=2)


def _check(n, p, K, dtype, off, nS, path=None):
    g = np.random.default_rng(3)
    d = dict(layout="dense", n=n, p=p, C=K + 1, K=K, lam=1e-2, X=g.standard_normal((n, p), dtype=np.float32),
             labels=g.integers(0, K + 1, size=n).astype(np.int32))
    pair = Pair(d, dtype, xoff=off)
    assert path is None or pair.gpu.ssn_dense_path() == path
    tol = TOL[dtype]
    print(f"[case] rows n={n} p={p} K={K} nS={nS} off={off} dtype={dtype}", flush=True)
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
    S = synth.sample_rows(n, nS)
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
