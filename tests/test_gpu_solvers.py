"""GPU parity of the iterations: CG (Alg. 2), line search (Alg. 3), the SSN loop (Alg. 1), and the C-ABI
error paths.  Iterations are followed step by step against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1802_09113_amd import binding, synth
from paper_1802_09113_amd.binding import Context, SsnError
from tests.gpu_util import TOL, Pair, rel_err, rel_scalar, workload

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
DTYPES = [F64, F32]


@pytest.fixture(scope="module")
def tiny():
    return workload(0, 2000)


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
@pytest.mark.parametrize("cfg,n", [(0, 2000), (1, 3001), (4, 403)])
def test_cg_follows_the_oracle_step_by_step(cfg, n, dtype):
    d = workload(cfg, n)
    pair = Pair(d, dtype)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = synth.sample_rows(n, d["nS"])
    G_ref, _ = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)                      # both sides start from the same right-hand side
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    # trajectory tolerance: CG amplifies rounding differences step by step
    ttol = 1e-8 if dtype == F64 else 5e-3
    for theta, T in [(1e-4, 10), (0.3, 10), (1e-30, 3)]:
        print(f"[case] cg cfg={cfg} dtype={dtype} theta={theta} T={T}", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, theta, T)
        out = pair.gpu.ssn_cg(Gd, theta, T)
        torch.cuda.synchronize()
        assert out["iters"] == ref["iters"]
        assert out["flags"] == ref["flags"]
        np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=ttol)
        np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=ttol)
        np.testing.assert_allclose(out["sHs"], ref["sHs"], rtol=ttol)
        assert rel_scalar(out["rel_res"], ref["rel_res"]) <= ttol
        assert rel_err(pair.host(out["p"]), ref["p"]) <= ttol
        # the returned direction satisfies what it reports: ||H p + g|| / ||g|| = rel_res
        Hp = pair.gpu.ssn_hess_apply(out["p"])
        torch.cuda.synchronize()
        res = np.linalg.norm(pair.host(Hp) + Gh) / np.linalg.norm(Gh)
        assert rel_scalar(res, out["rel_res"]) <= (1e-7 if dtype == F64 else 2e-2)
    pair.close()


def _shape_problem(n, p, C, lam, seed):
    """Seeded dense stand-in of a given shape (N(0,1) features, labels from a random linear model)."""
    g = np.random.default_rng(seed)
    X = g.standard_normal((n, p))
    Wt = g.standard_normal((p, C))
    labels = np.argmax(X @ Wt / np.sqrt(p) + g.gumbel(size=(n, C)), axis=1).astype(np.int32)
    return dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=lam, nS=n, T=10, iters=1, name="shape")


@pytest.mark.parametrize("n,p,C,lam,theta,T", [(1500, 48, 11, 1e-3, 1e-9, 150), (640, 1000, 2, 1e-2, 1e-8, 300)],
                         ids=["drive_like", "gisette_like_binary"])
def test_full_newton_with_a_long_cg(n, p, C, lam, theta, T):
    # the FullNewton variant of Sec. 4 (|S| = n, exact gradient and Hessian) with a CG budget far beyond
    # the usual 10 products, on the two shapes the paper runs long CG on (11 classes / 48 features, and
    # the binary case K = 1)
    d = _shape_problem(n, p, C, lam, seed=41)
    pair = Pair(d, F64)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = np.arange(n, dtype=np.int32)
    G_ref, _ = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    print(f"[case] full newton long cg n={n} p={p} C={C} T={T}", flush=True)
    ref = pair.oracle.cg(Wh, S, Gh, theta, T)
    out = pair.gpu.ssn_cg(Gd, theta, T)
    torch.cuda.synchronize()
    assert ref["flags"] & 1 and out["flags"] & 1                     # both reach the tolerance
    assert abs(out["iters"] - ref["iters"]) <= 2                      # long recurrences drift by rounding
    assert out["rel_res"] <= theta and ref["rel_res"] <= theta
    k = min(out["iters"], ref["iters"], 25)
    np.testing.assert_allclose(out["alpha"][:k], ref["alpha"][:k], rtol=1e-6)
    assert rel_err(pair.host(out["p"]), ref["p"]) <= 1e-7               # the Newton direction itself
    # one exact Newton iteration through the driver
    W0h, W0d = pair.block(np.zeros((pair.p, pair.K)))
    Wn, log_ref, _ = pair.oracle.ssn(W0h, S[None, :], theta=theta, T=T)
    recs, done = pair.gpu.ssn_solve(W0d, pair.idx(S)[None, :].contiguous(), theta=theta, T=T)
    torch.cuda.synchronize()
    assert done == 1 and recs[0]["alpha"] == log_ref[0, 4]
    assert rel_err(pair.host(W0d), Wn) <= 1e-7
    pair.close()


def test_csr_cg_best_iterate_when_the_residual_goes_up_and_down():
    # on this sample the residual norm of Alg. 2 rises every other product, so the best-iterate memory
    # (kept lazily on the CSR path) is exercised in both directions, including a best iterate that is not
    # the last one
    d = workload(4, 403)
    pair = Pair(d, F64)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = synth.sample_rows(403, 100)
    G_ref, _ = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    for T in (30, 11, 4):
        print(f"[case] csr cg lazy best iterate T={T}", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, 1e-30, T)
        assert np.any(np.diff(ref["rnorm"]) > 0)
        out = pair.gpu.ssn_cg(Gd, 1e-30, T)
        torch.cuda.synchronize()
        assert out["iters"] == ref["iters"] == T
        np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=1e-7)
        assert rel_scalar(out["rel_res"], ref["rel_res"]) <= 1e-7
        assert rel_err(pair.host(out["p"]), ref["p"]) <= 1e-7
    pair.close()


def _small_csr(n, p, C, seed, empty_rows):
    """Seeded CSR stand-in: 1-6 entries per row at random columns, rows in empty_rows without entries."""
    g = np.random.default_rng(seed)
    rowptr = [0]
    cols, vals = [], []
    for i in range(n):
        k = 0 if i in empty_rows else int(g.integers(1, 7))
        c = np.sort(g.choice(p, size=k, replace=False))
        cols.extend(c.tolist())
        vals.extend(g.standard_normal(k).tolist())
        rowptr.append(len(cols))
    labels = g.integers(0, C, size=n).astype(np.int32)
    return {"name": "small_csr", "layout": "csr", "n": n, "p": p, "C": C, "K": C - 1, "lam": 1e-2,
            "rowptr": np.array(rowptr, dtype=np.int64), "colidx": np.array(cols, dtype=np.int32),
            "vals": np.array(vals, dtype=np.float64), "labels": labels, "nnz": len(cols)}


@pytest.mark.parametrize("ldw", [None, 8], ids=["packed", "padded_blocks"])
def test_csr_cg_keeps_its_vectors_on_the_sample_columns(ldw):
    # On the CSR path Alg. 2 runs on the columns the sample touches; every other coordinate follows g through
    # three scalars.  Cases: a sample that touches a few of the columns, one whose rows are all empty (H_S =
    # lambda I, the direction is -g / lambda after one product), one that touches every column, and a sample
    # with a repeated row.  Each is followed against the oracle, which knows nothing of this.
    n, p, C = 300, 500, 4
    empty = set(range(0, 40))
    d = _small_csr(n, p, C, seed=77, empty_rows=empty)
    pair = Pair(d, F64, ldw=ldw)
    Wh, Wd = pair.block(synth.probe(p, C - 1, sub=3, scale=0.2))
    G_ref, _ = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    samples = {
        "few_columns": np.array([50, 60, 70, 80, 90, 100], dtype=np.int32),
        "empty_rows_only": np.array([1, 5, 9, 30], dtype=np.int32),
        "every_column": np.arange(n, dtype=np.int32),
        "repeated_row": np.array([45, 45, 200, 45, 7, 210], dtype=np.int32),
    }
    touched = np.unique(d["colidx"]).size
    for name, S in samples.items():
        # budgets below the rank of the sampled term (4 distinct rows x 3 classes in the last case): past
        # convergence the trajectory is rounding noise on both sides
        for theta, T in ((1e-30, 8 if name == "repeated_row" else 12), (1e-3, 40), (1e-30, 0)):
            if name == "empty_rows_only" and theta == 1e-30 and T > 0:
                theta = 1e-10        # the residual after the one product is rounding noise: stop there on both sides
            print(f"[case] csr support cg {name} theta={theta} T={T} ldw={ldw}", flush=True)
            pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
            ref = pair.oracle.cg(Wh, S, Gh, theta, T)
            out = pair.gpu.ssn_cg(Gd, theta, T)
            torch.cuda.synchronize()
            assert out["iters"] == ref["iters"]
            assert out["flags"] == ref["flags"]
            np.testing.assert_allclose(out["alpha"], ref["alpha"], rtol=1e-8)
            assert rel_err(pair.host(out["p"]), ref["p"]) <= 1e-8
            if name == "empty_rows_only":
                if T > 0:
                    assert out["iters"] == 1 and out["rel_res"] <= 1e-14
                    assert rel_err(pair.host(out["p"]), -Gh / d["lam"]) <= 1e-12
                continue
            np.testing.assert_allclose(out["rnorm"], ref["rnorm"], rtol=1e-8)
            assert rel_scalar(out["rel_res"], ref["rel_res"]) <= 1e-8
    assert touched < p          # some columns are touched by no row at all: always outside the support
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_cg_zero_budget_and_zero_gradient(tiny, dtype):
    pair = Pair(tiny, dtype)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = synth.sample_rows(2000, 100)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    Gh, Gd = pair.block(pair.oracle.gradient(Wh)[0])
    out = pair.gpu.ssn_cg(Gd, 1e-4, 0)
    torch.cuda.synchronize()
    assert out["iters"] == 0
    np.testing.assert_array_equal(pair.host(out["p"]), -Gh)
    Zh, Zd = pair.block(np.zeros((pair.p, pair.K)))
    out = pair.gpu.ssn_cg(Zd, 1e-4, 5)
    torch.cuda.synchronize()
    assert out["iters"] == 0 and np.all(pair.host(out["p"]) == 0)
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_linesearch_matches_oracle(tiny, dtype):
    pair = Pair(tiny, dtype)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=2, scale=0.5))
    G_ref, f_ref = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    f = pair.gpu.ssn_objective(Wd)
    for stretch, imax in [(1.0, 10), (300.0, 40), (5000.0, 40), (-1.0, 3)]:
        Ph, Pd = pair.block(-stretch * Gh)
        print(f"[case] linesearch stretch={stretch} dtype={dtype}", flush=True)
        ref = pair.oracle.linesearch(Wh, Ph, Gh, f_ref, imax=imax)
        out = pair.gpu.ssn_linesearch(Wd, Pd, Gd, f, imax=imax)
        assert out["ok"] == ref["ok"] and out["n_eval"] == ref["n_eval"]
        assert out["alpha"] == ref["alpha"]
        assert rel_scalar(out["f_new"], ref["f_new"]) <= TOL[dtype]
    assert out["ok"] == 0 and out["n_eval"] == 5         # the ascent direction is never accepted
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_ssn_fixed_schedule_tiny_config(tiny, dtype):
    d = tiny
    pair = Pair(d, dtype)
    test = workload(0, 2000, part="test")
    tpair = Pair(test, dtype)
    S_all = synth.sample_schedule(2000, d["nS"], d["iters"])
    W0h, W0d = pair.block(np.zeros((pair.p, pair.K)))
    Wref, log_ref, done_ref = pair.oracle.ssn(W0h, S_all, theta=1e-4, T=d["T"])
    recs, done = pair.gpu.ssn_solve(W0d, torch.from_numpy(S_all).cuda(), theta=1e-4, T=d["T"], test=tpair.gpu)
    torch.cuda.synchronize()
    assert done == done_ref == d["iters"]
    f_gpu = np.array([r["f"] for r in recs])
    ftol = 1e-8 if dtype == F64 else 1e-3
    np.testing.assert_allclose(f_gpu, log_ref[:, 0], rtol=ftol)
    assert f_gpu[0] == pytest.approx(np.log(pair.C), rel=TOL[dtype])
    assert np.all(np.diff(f_gpu) < 0)
    assert [r["cg_iters"] for r in recs] == [int(x) for x in log_ref[:, 2]]
    assert [r["alpha"] for r in recs] == list(log_ref[:, 4])
    assert rel_err(pair.host(W0d), Wref) <= (1e-7 if dtype == F64 else 2e-2)
    acc_ref = tpair.oracle.accuracy(Wref)
    assert abs(recs[-1]["test_acc"] - acc_ref) <= 1e-3
    _, acc_now = tpair.gpu.ssn_predict(W0d)
    assert acc_now == recs[-1]["test_acc"]
    pair.close()
    tpair.close()


@pytest.mark.parametrize("nS", [400, 12], ids=["accepted_then_rejected", "rejected_with_some_accepted"])
def test_ssn_gradient_look_ahead_changes_no_number(tiny, nS):
    # By default the first line-search trial is evaluated by the gradient pass and an accepted trial hands its
    # gradient to the next iteration.  With 400 sampled rows the first six first trials are accepted and the rest
    # rejected; with 12 the direction is poor, most first trials are rejected and a few accepted, so the
    # look-ahead is switched off and on again.
    # Either way the run is the oracle's, and the same as with the look-ahead turned off.
    d = tiny
    pair = Pair(d, F64)
    iters = 10
    S_all = synth.sample_schedule(2000, nS, iters)
    W0h, Wa = pair.block(np.zeros((pair.p, pair.K)))
    _, Wb = pair.block(np.zeros((pair.p, pair.K)))
    Wref, log_ref, done_ref = pair.oracle.ssn(W0h, S_all, theta=1e-4, T=d["T"])
    Sd = torch.from_numpy(S_all).cuda()
    ra, done_a = pair.gpu.ssn_solve(Wa, Sd, theta=1e-4, T=d["T"])
    rb, done_b = pair.gpu.ssn_solve(Wb, Sd, theta=1e-4, T=d["T"], lookahead=False)
    torch.cuda.synchronize()
    assert done_a == done_b == done_ref == iters
    alphas = list(log_ref[:, 4])
    assert alphas.count(1.0) >= 2 and min(alphas) < 1.0      # the schedule does exercise both outcomes
    for recs, W in ((ra, Wa), (rb, Wb)):
        assert [r["alpha"] for r in recs] == alphas
        assert [r["cg_iters"] for r in recs] == [int(x) for x in log_ref[:, 2]]
        np.testing.assert_allclose([r["f"] for r in recs], log_ref[:, 0], rtol=1e-9)
        np.testing.assert_allclose([r["gnorm"] for r in recs], log_ref[:, 1], rtol=1e-7)
        assert rel_err(pair.host(W), Wref) <= 1e-7
    assert [r["ls_evals"] for r in ra] == [r["ls_evals"] for r in rb]
    assert rel_err(pair.host(Wa), pair.host(Wb)) <= 1e-10
    pair.close()


@pytest.mark.parametrize("nS", [40, 403], ids=["small_sample_backtracking", "all_rows_unit_steps"])
@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_ssn_on_the_sparse_layout(dtype, nS):
    # Alg. 1 end to end on CSR data: on that path CG runs on the columns the sample touches, the slope comes from
    # the support's partial sums plus the off-support scalars, and the regulariser of a trial point from the pass
    # that writes it -- none of which the oracle knows about.  With and without the gradient look-ahead.
    n = 403
    d = workload(4, n)
    pair = Pair(d, dtype)
    iters = 6
    S_all = synth.sample_schedule(n, nS, iters)     # 40 rows: every first trial is rejected; all rows: most are accepted
    S_all[2, :5] = S_all[2, 5]                      # a sample with a repeated row
    W0h, Wa = pair.block(np.zeros((pair.p, pair.K)))
    _, Wb = pair.block(np.zeros((pair.p, pair.K)))
    Wref, log_ref, done_ref = pair.oracle.ssn(W0h, S_all, theta=1e-4, T=d["T"])
    Sd = torch.from_numpy(S_all).cuda()
    ra, done_a = pair.gpu.ssn_solve(Wa, Sd, theta=1e-4, T=d["T"])
    rb, done_b = pair.gpu.ssn_solve(Wb, Sd, theta=1e-4, T=d["T"], lookahead=False)
    torch.cuda.synchronize()
    assert done_a == done_b == done_ref == iters
    ftol, gtol, wtol = (1e-9, 1e-7, 1e-7) if dtype == F64 else (1e-3, 2e-2, 2e-2)
    for recs, W in ((ra, Wa), (rb, Wb)):
        assert [r["alpha"] for r in recs] == list(log_ref[:, 4])
        # in fp32 the theta test of Alg. 2 can fall on the other side of a near-tie: one product more or less
        slack = 0 if dtype == F64 else 1
        assert all(abs(r["cg_iters"] - int(x)) <= slack for r, x in zip(recs, log_ref[:, 2]))
        np.testing.assert_allclose([r["f"] for r in recs], log_ref[:, 0], rtol=ftol)
        np.testing.assert_allclose([r["gnorm"] for r in recs], log_ref[:, 1], rtol=gtol)
        assert rel_err(pair.host(W), Wref) <= wtol
    assert rel_err(pair.host(Wa), pair.host(Wb)) <= (1e-10 if dtype == F64 else 1e-4)
    pair.close()


@pytest.mark.parametrize("T", [0, 1, 3])
def test_ssn_with_tiny_cg_budgets_and_an_odd_number_of_steps(tiny, T):
    # T = 0: Alg. 2 returns its initial p_best = -g and the iteration is a steepest-descent step with back-tracking;
    # T = 1, 3: the shortest loops of the two-launch CG.  Three iterations: the iterate ends in the solver's own
    # buffer and has to be copied back into the caller's block.
    d = tiny
    pair = Pair(d, F64, ldw=8)                                # padded blocks: K = 2 of 8 columns in use
    S_all = synth.sample_schedule(2000, d["nS"], 3)
    W0h, W0d = pair.block(np.zeros((pair.p, pair.K)))
    Wref, log_ref, done_ref = pair.oracle.ssn(W0h, S_all, theta=1e-4, T=T)
    recs, done = pair.gpu.ssn_solve(W0d, torch.from_numpy(S_all).cuda(), theta=1e-4, T=T)
    torch.cuda.synchronize()
    assert done == done_ref == 3
    assert [r["alpha"] for r in recs] == list(log_ref[:, 4])
    assert [r["cg_iters"] for r in recs] == [int(x) for x in log_ref[:, 2]]
    np.testing.assert_allclose([r["f"] for r in recs], log_ref[:, 0], rtol=1e-10)
    assert rel_err(pair.host(W0d), Wref) <= 1e-9
    assert torch.isnan(W0d[:, pair.K:]).all()                 # the padding columns of the caller's block are untouched
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_ssn_with_sub_sampled_gradient(tiny, dtype):
    # Alg. 1 with eq. (2a) and eq. (2b): 20 % of the rows for g, 5 % for H
    d = tiny
    pair = Pair(d, dtype)
    iters = 6
    S_all = synth.sample_schedule(2000, d["nS"], iters)
    Sg_all = np.stack([synth.sample_rows(2000, 400, seed=900 + k) for k in range(iters)]).astype(np.int32)
    W0h, W0d = pair.block(np.zeros((pair.p, pair.K)))
    Wref, log_ref, done_ref = pair.oracle.ssn_sg(W0h, Sg_all, S_all, theta=1e-4, T=d["T"])
    recs, done = pair.gpu.ssn_solve(W0d, torch.from_numpy(S_all).cuda(), theta=1e-4, T=d["T"],
                                    Sg_all=torch.from_numpy(Sg_all).cuda())
    torch.cuda.synchronize()
    assert done == done_ref == iters
    f_gpu = np.array([r["f"] for r in recs])
    np.testing.assert_allclose(f_gpu, log_ref[:, 0], rtol=1e-8 if dtype == F64 else 1e-3)
    np.testing.assert_allclose([r["gnorm"] for r in recs], log_ref[:, 1], rtol=1e-7 if dtype == F64 else 2e-2)
    assert [r["cg_iters"] for r in recs] == [int(x) for x in log_ref[:, 2]]
    assert [r["alpha"] for r in recs] == list(log_ref[:, 4])
    assert rel_err(pair.host(W0d), Wref) <= (1e-7 if dtype == F64 else 2e-2)
    pair.close()


def test_work_follows_the_stream_it_is_given(tiny):
    # a context created on a side stream (default priority) and one moved there with ssn_set_stream: the
    # library's launches are ordered with other work on that stream, not with the default stream
    d = tiny
    side = torch.cuda.Stream()
    X = torch.from_numpy(d["X"]).cuda()
    labels = torch.from_numpy(d["labels"]).cuda()
    pair = Pair(d, F64)                                              # oracle side (its GPU context is not used)
    Wh = synth.probe(pair.p, pair.K, sub=1, scale=0.2)
    S = synth.sample_rows(2000, 100)
    Sd = torch.from_numpy(S).cuda()
    G_ref, f_ref = pair.oracle.gradient(Wh)
    HV_ref = pair.oracle.hessvec(Wh, S, Wh)
    torch.cuda.synchronize()
    ctx_a = Context(labels, d["C"], d["lam"], X=X, stream=side.cuda_stream)
    ctx_b = Context(labels, d["C"], d["lam"], X=X)
    ctx_b.ssn_set_stream(side.cuda_stream)
    for ctx in (ctx_a, ctx_b):
        with torch.cuda.stream(side):
            W = torch.zeros((pair.p, pair.K), dtype=F64, device="cuda")
            W.copy_(torch.from_numpy(Wh).cuda(), non_blocking=True)  # produced on the side stream ...
            G, f = ctx.ssn_gradient(W)                               # ... and consumed there by the library
            HV = ctx.ssn_hessvec(W, Sd, W)
            out = HV * 2.0                                           # torch work queued behind the library's
        side.synchronize()
        assert rel_scalar(f, f_ref) <= 1e-10
        assert rel_err(G.cpu().numpy(), G_ref) <= 1e-10
        assert rel_err(out.cpu().numpy(), 2.0 * HV_ref) <= 1e-10
        ctx.close()
    pair.close()


def test_products_replay_from_a_hip_graph():
    # ssn_hess_apply and ssn_gradient (without f) allocate nothing and never wait for the device once the
    # sample is prepared, so a caller may capture them in a HIP graph; every replay is checked against the
    # eager result on fresh inputs, with eager work between the replays
    d = workload(1, 3001)
    pair = Pair(d, F64)
    side = torch.cuda.Stream()
    pair.gpu.ssn_set_stream(side.cuda_stream)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = synth.sample_rows(3001, d["nS"])
    Sd = pair.idx(S)
    V = pair.gpu.new_block()
    HV = pair.gpu.new_block()
    G = pair.gpu.new_block()
    with torch.cuda.stream(side):
        pair.gpu.ssn_hess_prepare(Wd, Sd)
        V.copy_(pair.block(synth.probe(pair.p, pair.K, sub=20))[1])
        pair.gpu.ssn_hess_apply(V, HV)                               # warm-up outside the capture
        pair.gpu.ssn_gradient(Wd, G, want_f=False)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pair.gpu.ssn_hess_apply(V, HV)
        pair.gpu.ssn_gradient(Wd, G, want_f=False)
    G_ref, _ = pair.oracle.gradient(Wh)
    for rep in range(4):
        Vh, Vd = pair.block(synth.probe(pair.p, pair.K, sub=30 + rep))
        print(f"[case] graph replay {rep}", flush=True)
        with torch.cuda.stream(side):
            V.copy_(Vd)
            HV.zero_()
            G.zero_()
            graph.replay()
        side.synchronize()
        assert rel_err(pair.host(HV), pair.oracle.hessvec(Wh, S, Vh)) <= 1e-10
        assert rel_err(pair.host(G), G_ref) <= 1e-10
        with torch.cuda.stream(side):                                # eager work between replays
            eager = pair.gpu.ssn_hess_apply(V)
        side.synchronize()
        assert torch.equal(eager[:, : pair.K], HV[:, : pair.K])
    pair.close()


def test_error_paths(tiny):
    d = tiny
    dev = "cuda"
    X = torch.from_numpy(d["X"]).to(dev)
    labels = torch.from_numpy(d["labels"]).to(dev)
    bad = labels.clone()
    bad[123] = d["C"]
    with pytest.raises(SsnError) as e:
        Context(bad, d["C"], 1e-3, X=X)
    assert e.value.status == binding.SSN_E_BAD_LABEL
    bad[123] = -1
    with pytest.raises(SsnError) as e:
        Context(bad, d["C"], 1e-3, X=X)
    assert e.value.status == binding.SSN_E_BAD_LABEL
    with pytest.raises(SsnError) as e:
        Context(labels, 1, 1e-3, X=X)
    assert e.value.status == binding.SSN_E_INVALID_ARG
    with pytest.raises(SsnError) as e:
        Context(labels, d["C"], -1.0, X=X)
    assert e.value.status == binding.SSN_E_INVALID_ARG
    with pytest.raises(SsnError) as e:
        Context(labels, 40, 1e-3, X=X)           # K = 39 > 32 on the dense path
    assert e.value.status == binding.SSN_E_UNSUPPORTED
    ctx = Context(labels, d["C"], 1e-3, X=X)
    W = torch.zeros((ctx.p, ctx.K), dtype=torch.float64, device=dev)
    V = torch.ones_like(W)
    with pytest.raises(SsnError) as e:
        ctx.ssn_hess_apply(V)
    assert e.value.status == binding.SSN_E_NOT_PREPARED
    with pytest.raises(SsnError) as e:
        ctx.ssn_cg(V, 1e-4, 3)
    assert e.value.status == binding.SSN_E_NOT_PREPARED
    for badS in ([0, 5, 2000], [-1, 3]):
        with pytest.raises(SsnError) as e:
            ctx.ssn_hess_prepare(W, torch.tensor(badS, dtype=torch.int32, device=dev))
        assert e.value.status == binding.SSN_E_BAD_INDEX
    # a failed prepare leaves the context unprepared, a good one repairs it
    with pytest.raises(SsnError):
        ctx.ssn_hess_apply(V)
    ctx.ssn_hess_prepare(W, torch.tensor([1, 2, 3], dtype=torch.int32, device=dev))
    ctx.ssn_hess_apply(V)
    # NaN weights surface as a status, not as a silent NaN
    Wn = W.clone()
    Wn[0, 0] = float("nan")
    with pytest.raises(SsnError) as e:
        ctx.ssn_objective(Wn)
    assert e.value.status == binding.SSN_E_NONFINITE
    L = binding.lib()
    assert L.ssn_objective(None, None, None) == binding.SSN_E_INVALID_ARG
    assert L.ssn_destroy(None) == binding.SSN_E_INVALID_ARG
    ctx.close()
    # CSR: column index out of range, broken rowptr
    rp = torch.tensor([0, 2, 3], dtype=torch.int32, device=dev)
    ci = torch.tensor([0, 7, 2], dtype=torch.int32, device=dev)
    vals = torch.ones(3, dtype=torch.float64, device=dev)
    lab2 = torch.tensor([0, 1], dtype=torch.int32, device=dev)
    with pytest.raises(SsnError) as e:
        Context(lab2, 2, 0.0, csr=(rp, ci, vals), p=5)
    assert e.value.status == binding.SSN_E_BAD_INDEX
    rp_bad = torch.tensor([0, 3, 2], dtype=torch.int32, device=dev)
    with pytest.raises(SsnError) as e:
        Context(lab2, 2, 0.0, csr=(rp_bad, ci, vals), p=8)
    assert e.value.status == binding.SSN_E_INVALID_ARG
    ok = Context(lab2, 2, 0.0, csr=(rp, ci, vals), p=8)
    ok.close()


@pytest.mark.parametrize("cfg,n", [(0, 2000), (1, 3001), (2, 1003), (4, 403)],
                         ids=["narrow", "one_pass", "two_kernel", "csr"])
def test_results_are_deterministic(cfg, n):
    # every reduction has a fixed order on every path (the CSR transposed product gathers by column
    # instead of scattering with atomics), so two runs give the same bits
    d = workload(cfg, n)
    pair = Pair(d, F64)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.2))
    Vh, Vd = pair.block(synth.probe(pair.p, pair.K, sub=2))
    Sd = pair.idx(synth.sample_rows(n, max(100, d["nS"])))
    runs = []
    for _ in range(2):
        print(f"[case] determinism cfg={cfg} n={n}", flush=True)
        f = pair.gpu.ssn_objective(Wd)
        G, _ = pair.gpu.ssn_gradient(Wd)
        HV = pair.gpu.ssn_hessvec(Wd, Sd, Vd)
        out = pair.gpu.ssn_cg(G, 1e-6, 8, want_trace=True)
        torch.cuda.synchronize()
        runs.append((f, G.clone(), HV.clone(), out["p"].clone(), np.array(out["alpha"] + out["rnorm"] + out["sHs"])))
    assert runs[0][0] == runs[1][0]
    for k in (1, 2, 3):
        assert torch.equal(runs[0][k][:, : pair.K], runs[1][k][:, : pair.K]), k
    assert np.array_equal(runs[0][4], runs[1][4])
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_text_results_are_the_same_in_every_context(dtype):
    # One set of stored entries over the whole vocabulary: every context that is made on it, and every call, gives the
    # same bits (its column-sorted view neither drops nor moves an entry), and a gradient is that of the oracle.  So two
    # runs whose results on text differ by an entry's worth were given different entries.
    n = 3000
    d = workload(4, n)
    S_all = synth.sample_schedule(n, 150, 2)
    runs = []
    for k in range(3):
        pair = Pair(d, dtype)
        print(f"[case] text context {k} n={n} nnz={d['vals'].size} dtype={dtype}", flush=True)
        W0h, W = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.01))
        for _ in range(2):
            G, f = pair.gpu.ssn_gradient(W)
            run = W.clone()
            log, _ = pair.gpu.ssn_solve(run, torch.from_numpy(S_all).cuda(), theta=1e-4, T=10)
            torch.cuda.synchronize()
            runs.append((f, [(r["f"], r["alpha"], r["gnorm"]) for r in log], G.clone(), run))
        if k == 0:
            G_ref, f_ref = pair.oracle.gradient(W0h)
            assert rel_scalar(f, f_ref) <= TOL[dtype] and rel_err(pair.host(G), G_ref) <= TOL[dtype]
        pair.close()
    for r in runs[1:]:
        assert r[:2] == runs[0][:2]
        assert torch.equal(r[2], runs[0][2]) and torch.equal(r[3], runs[0][3])


def _ill_conditioned_shape(n, p, C, lam, seed, spread):
    """Dense stand-in whose columns differ in scale by e^(2 spread): with a small lambda CG needs its whole budget."""
    g = np.random.default_rng(seed)
    X = g.standard_normal((n, p)) * np.exp(g.uniform(-spread, spread, size=p))
    Wt = g.standard_normal((p, C))
    labels = np.argmax(X @ Wt / np.sqrt(p) + g.gumbel(size=(n, C)), axis=1).astype(np.int32)
    return dict(layout="dense", X=X, labels=labels, n=n, p=p, C=C, K=C - 1, lam=lam, nS=n, T=1000, iters=1, name="ill")


@pytest.mark.parametrize("n,p,C,lam,spread", [(50000, 48, 11, 1e-7, 2.5), (6000, 5000, 2, 1e-5, 1.0)],
                         ids=["drive_shape", "gisette_shape"])
def test_cg_budget_of_1000_products_at_the_full_shapes(n, p, C, lam, spread):
    # Sec. 4 runs T = 1000 on the 50000 x 48, C = 11 and the 6000 x 5000, C = 2 data sets with |S| = n.  On these
    # ill-conditioned stand-ins CG uses the whole budget.  Two long CG runs in floating point do not stay together
    # product by product, so what is compared: the first products step by step; that the residual the library
    # reports for its direction (carried by recurrences over 1000 products: H s_k, s_k^T H s_k and r_k are never
    # recomputed) is the residual that direction really has, measured with the oracle's product; and that the
    # direction is as good as the oracle's.  The oracle's row loops run on all cores here (its OpenMP build).
    from oracle.oracle import Problem
    d = _ill_conditioned_shape(n, p, C, lam, 41, spread)
    pair = Pair(d, F64)
    pair.oracle = Problem(d["labels"], C, lam, X=d["X"], threads=True)
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=1, scale=0.1))
    S = np.arange(n, dtype=np.int32)
    G_ref, _ = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    gn = np.linalg.norm(Gh)
    pair.gpu.ssn_hess_prepare(Wd, pair.idx(S))
    for T in (300, 1000):
        print(f"[case] long cg n={n} p={p} C={C} T={T}: oracle", flush=True)
        ref = pair.oracle.cg(Wh, S, Gh, 1e-12, T)
        print("[case] ... gpu", flush=True)
        out = pair.gpu.ssn_cg(Gd, 1e-12, T)
        torch.cuda.synchronize()
        assert out["iters"] == ref["iters"] == T and out["flags"] == ref["flags"] == 0
        np.testing.assert_allclose(out["alpha"][:30], ref["alpha"][:30], rtol=1e-6)
        np.testing.assert_allclose(out["rnorm"][:30], ref["rnorm"][:30], rtol=1e-6)
        true_res = np.linalg.norm(pair.oracle.hessvec(Wh, S, pair.host(out["p"])) + Gh) / gn
        print(f"[info] T={T} reported {out['rel_res']:.6e} true {true_res:.6e} oracle {ref['rel_res']:.6e}", flush=True)
        assert rel_scalar(out["rel_res"], true_res) <= 1e-6
        assert out["rel_res"] <= 3.0 * ref["rel_res"]
    pair.close()


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
@pytest.mark.parametrize("cfg,n,p,nS,w0", [(0, 2000, None, 12, 0.0), (1, 3001, None, 150, 0.0), (2, 1003, None, 50, 0.0),
                                          (3, 5003, None, 50, 0.0), (4, 403, None, 40, 0.0), (5, 1003, 700, 60, 0.01)],
                         ids=["tiny", "image_like", "wide", "tall_narrow", "sparse", "binary"])
def test_line_search_on_cached_margins_takes_the_same_decisions(cfg, n, p, nS, w0, dtype):
    # Back-tracking trials evaluated from X W + alpha X P (one pass over the data, then n x 2K numbers per trial)
    # against the same run with every trial a pass over the data (Alg. 3 as written), and against the oracle.
    # Small samples give poor directions, so these schedules back-track a lot.
    d = synth.make(cfg, n=n, p=p)
    pair = Pair(d, dtype)
    # (the image-like and wide schedules start at zero, where they back-track five times at once; from there two
    # runs only stay together for a few iterations -- see tests/test_gpu_fixed_schedule.py -- hence three of them)
    iters = 3 if cfg in (1, 2) else 6
    S_all = synth.sample_schedule(n, nS, iters)
    W0h, Wa = pair.block(synth.probe(pair.p, pair.K, sub=7, scale=w0))
    _, Wb = pair.block(synth.probe(pair.p, pair.K, sub=7, scale=w0))
    Sd = torch.from_numpy(S_all).cuda()
    print(f"[case] cached margins cfg={cfg} dtype={dtype}", flush=True)
    ra, _ = pair.gpu.ssn_solve(Wa, Sd, theta=1e-4, T=d["T"])
    rb, _ = pair.gpu.ssn_solve(Wb, Sd, theta=1e-4, T=d["T"], margin_cache=False)
    torch.cuda.synchronize()
    Wref, log_ref, _ = pair.oracle.ssn(W0h, S_all, theta=1e-4, T=d["T"])
    assert sum(r["ls_evals"] for r in ra) >= iters + 3                 # the cache was in use
    assert [r["alpha"] for r in ra] == [r["alpha"] for r in rb]
    assert [r["ls_evals"] for r in ra] == [r["ls_evals"] for r in rb]
    f64 = dtype == F64
    np.testing.assert_allclose([r["f"] for r in ra], [r["f"] for r in rb], rtol=1e-9 if f64 else 1e-4)
    assert rel_err(pair.host(Wa), pair.host(Wb)) <= (1e-8 if f64 else 1e-3)
    # (the oracle comparison is left to the other tests for the two degenerate starts at zero)
    if cfg not in (1, 2) and [r["alpha"] for r in ra] == list(log_ref[:, 4]):
        np.testing.assert_allclose([r["f"] for r in ra], log_ref[:, 0], rtol=1e-6 if f64 else 2e-3)
    # one search by itself: trials, step and value are Alg. 3's
    Wh, Wd = pair.block(synth.probe(pair.p, pair.K, sub=2, scale=0.3))
    G_ref, f_ref = pair.oracle.gradient(Wh)
    Gh, Gd = pair.block(G_ref)
    for stretch in (2e3, 2e5, 2e7, 2e9):                                # far too long: several reductions
        Ph, Pd = pair.block(-stretch * G_ref)
        ref = pair.oracle.linesearch(Wh, Ph, Gh, f_ref, imax=60)
        if ref["n_eval"] >= 3:
            break
    out = pair.gpu.ssn_linesearch(Wd, Pd, Gd, pair.gpu.ssn_objective(Wd), imax=60)
    assert ref["n_eval"] >= 3
    assert out["alpha"] == ref["alpha"] and out["n_eval"] == ref["n_eval"] and out["ok"] == ref["ok"]
    assert rel_scalar(out["f_new"], ref["f_new"]) <= TOL[dtype]
    pair.close()


def test_solve_without_back_tracking_takes_no_margin_cache():
    # the cache is n x 2 K values (192 MB here); a solve whose first trials are all accepted never looks at it
    n, p, K = 300000, 64, 40
    g = np.random.default_rng(6)
    vals = g.standard_normal(n)
    d = dict(layout="csr", n=n, p=p, C=K + 1, K=K, lam=1.0, rowptr=np.arange(n + 1, dtype=np.int64),
             colidx=g.integers(0, p, size=n).astype(np.int32), vals=vals, labels=g.integers(0, K + 1, size=n).astype(np.int32))
    pair = Pair(d, F64)
    S_all = synth.sample_schedule(n, 2000, 3)
    Sd = torch.from_numpy(S_all).cuda()
    _, W = pair.block(np.zeros((p, K)))
    G, _ = pair.gpu.ssn_gradient(W)                          # the whole matrix's view and the other workspaces
    pair.gpu.ssn_hess_prepare(W, Sd[0].contiguous())
    pair.gpu.ssn_cg(G, 1e-4, 10)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    print("[case] solve without back-tracking", flush=True)
    log, _ = pair.gpu.ssn_solve(W, Sd, theta=1e-4, T=10)
    torch.cuda.synchronize()
    assert [r["ls_evals"] for r in log] == [1, 1, 1]
    assert free - torch.cuda.mem_get_info()[0] < n * 2 * K * 8 // 2
    pair.close()


@pytest.mark.parametrize("lookahead", [True, False], ids=["look_ahead", "no_look_ahead"])
@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32"])
def test_margins_kept_from_gradient_passes_change_nothing(dtype, lookahead):
    # The second run finds the margin cache of the first, so its gradient passes leave X W there and a search that backs
    # off adds X P only; the first forms both products at its first back-off.  Same bits.
    n, nS, iters = 403, 40, 6
    pair = Pair(workload(4, n), dtype)
    Sd = torch.from_numpy(synth.sample_schedule(n, nS, iters)).cuda()
    runs = []
    for k in range(3):
        print(f"[case] kept margins run={k} dtype={dtype} lookahead={lookahead}", flush=True)
        _, W = pair.block(np.zeros((pair.p, pair.K)))
        log, _ = pair.gpu.ssn_solve(W, Sd, theta=1e-4, T=10, lookahead=lookahead)
        torch.cuda.synchronize()
        runs.append(([(r["f"], r["alpha"], r["ls_evals"], r["cg_iters"]) for r in log], W.clone()))
    evals = [r[2] for r in runs[0][0]]
    assert sum(e > 1 for e in evals) >= 2                    # iterations that backed off
    for r in runs[1:]:
        assert r[0] == runs[0][0] and torch.equal(r[1], runs[0][1])
    pair.close()
