"""Passes over p x K weight blocks at the sizes where they change form: contiguous, 16-byte aligned blocks that give every
thread of the launch a vector (fp64: all of more than 65 536 elements; fp32: multiples of 1024 from there on, and all of
1 048 576 and more) go as 16-byte vectors in one share per workgroup, the others element by element.  CSR data of few rows, so
that the block passes are what the calls consist of.  Against the oracle, and axpy against its own arithmetic."""
import numpy as np
import pytest
import torch

from paper_1802_09113_amd import synth
from tests.gpu_util import TOL, Pair, rel_err, rel_scalar

pytestmark = pytest.mark.gpu
F64, F32 = torch.float64, torch.float32


def _data(n, p, C):
    g = np.random.default_rng(11)
    lens = g.integers(0, 9, size=n)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    colidx = np.concatenate([np.sort(g.choice(p, size=k, replace=False)) for k in lens]).astype(np.int32)
    return dict(layout="csr", n=n, p=p, C=C, K=C - 1, lam=1e-2, labels=g.integers(0, C, size=n).astype(np.int32),
                rowptr=rowptr, colidx=colidx, vals=g.standard_normal(colidx.size))


# 65536 elements (one per thread, element by element), one more, shares that end inside a round of four vectors per thread,
# one and two million elements, packed and padded
@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("p,C,pad", [(65536, 2, 0), (65537, 2, 0), (21847, 4, 0), (10923, 8, 0), (131075, 2, 0), (65539, 20, 0),
                                     (65539, 20, 1), (400001, 6, 0)])
def test_block_passes(p, C, pad, dtype):
    _check(p, C, pad, 0, dtype)


# Shares of several rounds (from 2 097 154 elements in fp64, 4 194 308 in fp32) with every length of tail behind the last
# whole vector; the smallest vector pass of fp32 (66560 elements, without a tail) and the element-wise size behind it;
# packed blocks that start one element behind a 16-byte boundary
@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("p,C,shift", [(5000000, 2, 0), (5000001, 2, 0), (5000002, 2, 0), (5000003, 2, 0), (1700003, 4, 0),
                                       (66560, 2, 0), (66561, 2, 0), (66560, 2, 1), (1400001, 4, 1)])
def test_block_passes_over_several_rounds(p, C, shift, dtype):
    _check(p, C, 0, shift, dtype)


def _check(p, C, pad, shift, dtype):
    n, d = 60, _data(60, p, C)
    pair = Pair(d, dtype, ldw=C - 1 + pad)
    if shift:
        plain = pair.block

        def shifted(host):
            r, t = plain(host)
            flat = torch.empty(shift + t.numel(), dtype=t.dtype, device=t.device)
            flat[shift:].copy_(t.flatten())
            return r, flat[shift:].view(t.shape)
        pair.block = shifted
    tol = TOL[dtype]
    print(f"[case] block p={p} C={C} pad={pad} shift={shift} dtype={dtype}", flush=True)
    Wh, Wd = pair.block(synth.probe(p, C - 1, sub=1, scale=0.3))
    G_ref, f_ref = pair.oracle.gradient(Wh)
    G, f = pair.gpu.ssn_gradient(Wd)
    assert rel_scalar(f, f_ref) <= tol and rel_err(pair.host(G), G_ref) <= tol
    assert rel_scalar(pair.gpu.ssn_objective(Wd), f_ref) <= tol
    # another block in the same buffer: nothing of the last one's norm is left
    Vh, Vd = pair.block(synth.probe(p, C - 1, sub=2, scale=0.1))
    Wd.copy_(Vd)
    assert rel_scalar(pair.gpu.ssn_gradient(Wd)[1], pair.oracle.objective(Vh)) <= tol
    S = synth.sample_rows(n, 20)
    Gh, Gd = pair.block(G_ref)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    out, ref = pair.gpu.ssn_cg(Gd, 1e-12, 6), pair.oracle.cg(Vh, S, Gh, 1e-12, 6)
    k = min(3, out["iters"], ref["iters"])
    np.testing.assert_allclose(out["alpha"][:k], ref["alpha"][:k], rtol=1e-9 if dtype == F64 else 1e-3)
    # the line search forms both products and the norms of W, P and their product; a step far too long backs off
    Ph, Pd = pair.block(-2e3 * G_ref)
    G1, f1 = pair.oracle.gradient(Vh)
    G1h, G1d = pair.block(G1)
    ls_ref = pair.oracle.linesearch(Vh, Ph, G1h, f1, imax=60)
    ls = pair.gpu.ssn_linesearch(Wd, Pd, G1d, pair.gpu.ssn_objective(Wd), imax=60)
    assert ls["alpha"] == ls_ref["alpha"] and rel_scalar(ls["f_new"], ls_ref["f_new"]) <= 10 * tol
    pair.gpu.ssn_axpy(-0.37, Pd, Wd)
    torch.cuda.synchronize()
    # one rounding of the result and at most two of the sum
    want = -0.37 * Ph + Vh
    eps = np.finfo(np.float64 if dtype == F64 else np.float32).eps
    assert np.all(np.abs(pair.host(Wd) - want) <= eps * (np.abs(want) + np.finfo(np.float64).eps / eps * 2 * (np.abs(Ph) + np.abs(Vh))))
    pair.close()
