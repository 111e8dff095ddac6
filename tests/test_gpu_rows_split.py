"""GPU parity of the rows kernels where a workgroup shares a row block (two, four, eight and sixteen waves): row counts on
either side of each change of form, features at the first trip of a wave and with tails, one and two class tiles, padded
rows and weights, and a sample of repeated rows."""
import numpy as np
import pytest
import torch

from tests.gpu_util import TOL, Pair, rel_err, rel_scalar

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32

# n, p, C, ldx, ldw.  256 compute units: forms change at 512, 640, 1088, 1536, 2048 and 2560 row blocks of sixteen
CASES = [
    (2000, 127, 19, None, None),          # a wave per row block
    (2000, 128, 19, None, 20),            # four waves, one trip each at most
    (8192, 259, 18, 260, None),           # eight waves, a tail
    (8193, 130, 21, None, None),          # four
    (10300, 255, 18, 256, None),          # two
    (10300, 256, 18, None, None),         # four
    (17409, 140, 25, None, None),         # two
    (24577, 128, 18, None, None),         # two class tiles: a wave per row block
    (24577, 1100, 3, None, 3),            # one class tile: two
    (17410, 1281, 19, None, None),        # two class tiles: fp64 two, fp32 four
    (24600, 2050, 18, 2051, None),        # fp64 two, fp32 four
    (25000, 2305, 9, None, 9),            # one class tile: four
    (20000, 2307, 3, None, None),         # fp64 two, fp32 four
    (32784, 513, 18, 520, None),          # fp64 four, fp32 a wave per row block
    (32784, 1280, 2, None, None),         # binary kernels next to it: one weight column
    (32784, 1281, 3, None, None),         # four
    # weights in registers: from 64 million elements and 16384 rows (fp32), 37.5 million and 28000 (fp64) on
    (28000, 1536, 17, None, 18),          # fp64: sixteen weight columns, one slice of whole windows
    (28010, 1345, 9, 1346, None),         # fp64: the last window moved back; margins of two operands in one tile
    (28001, 2049, 4, None, None),         # fp64: odd rows of any alignment, two slices
    (16384, 4096, 3, None, None),         # fp32: two slices of whole windows
    (28001, 2301, 3, 2303, 3),            # one slice in fp32, two in fp64, windows far back
]


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,p,C,ldx,ldw", CASES)
def test_rows_shared_by_a_workgroup(n, p, C, ldx, ldw, dtype):
    g = np.random.default_rng(n + p)
    X = g.standard_normal((n, p), dtype=np.float32).astype(np.float64) / np.sqrt(p)
    labels = g.integers(0, C, n).astype(np.int32)
    pair = Pair(dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=0.01), dtype, ldx=ldx, ldw=ldw)
    pair.oracle.threads = True
    Wh, Wd = pair.block(0.5 * g.standard_normal((p, C - 1)))
    print(f"[case] rows n={n} p={p} C={C} dtype={dtype}", flush=True)
    f = pair.gpu.ssn_objective(Wd)
    G, fg = pair.gpu.ssn_gradient(Wd)
    G_ref, f_ref = pair.oracle.gradient(Wh)
    pred, acc = pair.gpu.ssn_predict(Wd)
    torch.cuda.synchronize()
    assert rel_scalar(f, f_ref) <= TOL[dtype] / 10 and rel_scalar(fg, f_ref) <= TOL[dtype] / 10
    assert rel_err(pair.host(G), G_ref) <= TOL[dtype]
    Z = np.concatenate([pair.oracle.X @ Wh, np.zeros((n, 1))], axis=1)
    ref = np.argmax(Z, axis=1)
    top = np.sort(Z, axis=1)
    clear = top[:, -1] - top[:, -2] > 1e-4                # elsewhere rounding may decide in fp32
    assert np.array_equal(pred.cpu().numpy()[clear], ref[clear])
    assert abs(acc - float(np.mean(ref == labels))) <= float(np.mean(~clear)) + 1e-12
    if 2 * (C - 1) <= 16:                                 # a line search that backs off: the margins of both operands
        Ph, Pd = pair.block(-40.0 * G_ref)
        Gh, Gd = pair.block(G_ref)
        ls, ref_ls = pair.gpu.ssn_linesearch(Wd, Pd, Gd, f, imax=6), pair.oracle.linesearch(Wh, Ph, Gh, f_ref, imax=6)
        assert ls["alpha"] == ref_ls["alpha"] and rel_scalar(ls["f_new"], ref_ls["f_new"]) <= TOL[dtype]
    S = g.integers(0, n, min(n, 3000))
    Vh, Vd = pair.block(g.standard_normal((p, C - 1)))
    HV = pair.gpu.ssn_hessvec(Wd, pair.idx(S), Vd)
    torch.cuda.synchronize()
    assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= TOL[dtype]
    pair.close()
