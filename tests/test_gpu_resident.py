"""Resident runs (one cooperative launch for a whole run, iterates in operand
order): one step against an FP64 product at the edges of the tiles, whole
runs of every method against exact densities, and the launch sequence's
outcomes on trivial, truncated, diverging and cut-off runs and on batches
with teams of every size."""
import math

import numpy as np
import pytest

import oracle
from workloads import dense_instance
from tests.gpu_helpers import print_case

pytestmark = pytest.mark.gpu

U = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "bf16x3": 2.0 ** -24}
D_TOL = {"fp64": 1e-11, "fp32": 2e-5, "bf16x3": 2e-4}
# 1, a 16-block and its neighbours, whole tiles of every edge (32, 48, 64,
# 80), one past them, several tiles, an odd K split over the four waves, and
# (1900) FP64's single chain per wave
SIZES = (1, 2, 15, 16, 17, 32, 33, 47, 48, 49, 64, 65, 80, 81, 96, 129, 161, 240, 307, 520, 900,
         1900)


def _step_bound(prec, n):
    """|error| of an element of one step X1 = S or 2 X - S, S = X X, for rows
    of norm at most 1: n roundings of partial sums of at most 1 each, four
    more for the polynomial and the store; BF16x3 drops |L||L'| and the
    remainders of the two splits (2^-18 of |x||x'| each) and accumulates
    three products."""
    u = U[prec]
    if prec == "bf16x3":
        return 3 * 2.0 ** -18 + (3 * n + 4) * u
    return (n + 4) * u


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_one_step_at_tile_edges(prec):
    import torch
    import paper_1507_02087_amd as sp2
    ctx = sp2.Context(0)
    try:
        for n in SIZES:
            rng = np.random.default_rng(n)
            A = rng.standard_normal((n, n))
            F = 0.5 * (A + A.T) / (2.0 * math.sqrt(n) + 2.0)   # spectrum inside [-1, 1]
            lo, hi = -max(1.0, np.abs(F).sum(1).max()), max(1.0, np.abs(F).sum(1).max())
            n_occ = max(0, min(n - 1, n // 2))
            # a view with an odd row stride
            buf = torch.zeros(n, n + 3, dtype=torch.float64, device="cuda")
            buf[:, :n] = torch.from_numpy(F).cuda()
            print_case(f"resident one step {prec} n={n}")
            r = sp2.run_dense(buf[:, :n], lo, hi, n_occ, precision=prec, max_iter=1,
                              as_fp64=True, ctx=ctx)
            X0 = (hi * np.eye(n) - F) / (hi - lo)
            if prec != "fp64":
                X0 = X0.astype(np.float32).astype(np.float64)
            if n_occ == 0:
                assert r.status == sp2.OK and r.n == 0 and float(r.D.abs().max()) == 0.0
                continue
            assert r.status_name == "NOT_CONVERGED" and r.n == 1
            S = X0 @ X0
            X1 = S if r.p[1] else 2 * X0 - S
            D = r.D.cpu().numpy()
            assert np.array_equal(D, D.T)
            # FP64: the reference product has the same bound of its own
            tol = _step_bound(prec, n) * (2.0 if prec == "fp64" else 1.0)
            assert np.max(np.abs(D - X1)) <= tol, (n, np.max(np.abs(D - X1)), tol)
            assert abs(r.v[0] - np.linalg.norm(X0 - S)) <= n * tol
            assert abs(r.t1[1] - np.trace(D)) <= 4 * n * U["fp64"] * max(1.0, n)
            assert abs(r.t2[1] - np.sum(D * D)) <= 4 * n * n * U["fp64"] * max(1.0, n)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("method", ["sp2", "acc", "mcweeny", "mcw_acc"])
def test_runs_reach_the_projector(prec, method):
    import torch
    import paper_1507_02087_amd as sp2
    for n, n_occ in ((40, 13), (170, 85), (431, 120), (1100, 550)):
        inst = dense_instance(n, n_occ, -1.0, 1.0, 0.1, seed=900 + n)
        F = torch.from_numpy(inst.F).cuda()
        homo, lumo = float(inst.lam[n_occ - 1]), float(inst.lam[n_occ])
        kw = {}
        if method == "acc":
            kw["homo_lumo"] = (homo, homo, lumo, lumo)
        elif method == "mcweeny":
            kw["mcweeny"] = (0.5 * (homo + lumo), None)
        elif method == "mcw_acc":
            kw["mcweeny"] = (0.5 * (homo + lumo), lumo - homo)
        print_case(f"resident {method} {prec} n={n}")
        r = sp2.run_dense(F, -1.0, 1.0, n_occ, precision=prec, **kw)
        again = sp2.run_dense(F, -1.0, 1.0, n_occ, precision=prec, **kw)
        assert r.status == sp2.OK
        assert again.n == r.n and again.v == r.v and torch.equal(again.D, r.D)
        De = oracle.density_from_eigenvectors(inst.Q, n_occ)
        err = float(np.linalg.norm(r.D.cpu().numpy() - De)) / math.sqrt(n_occ)
        assert err < D_TOL[prec], (n, err)
        assert torch.equal(r.D, r.D.t())


def test_truncation_and_cut_off_match_the_sequence():
    import torch
    import paper_1507_02087_amd as sp2
    inst = dense_instance(210, 100, -1.0, 1.0, 0.1, seed=12)
    F = torch.from_numpy(inst.F).cuda()
    for prec in ("fp64", "fp32"):
        a, b = [sp2.run_dense(F, -1.0, 1.0, 100, precision=prec, trunc_tau=1e-4, max_iter=4,
                              launch=launch) for launch in ("auto", "sequence")]
        assert a.status_name == b.status_name == "NOT_CONVERGED" and a.p == b.p
        # an entry within rounding of the threshold may fall on either side
        da, db = a.D.cpu().numpy(), b.D.cpu().numpy()
        off = np.abs(da - db) > 64 * 210 * U[prec]
        assert np.all((np.abs(da) < 1e-4 * 1.01) & (np.abs(db) < 1e-4 * 1.01) | ~off)
        assert np.mean(off) < 1e-3
    # a diverging run and one whose X_0 is exactly idempotent
    bad = [sp2.run_dense(F, -1.0, -0.99, 100, launch=launch) for launch in ("auto", "sequence")]
    assert bad[0].status == bad[1].status == sp2.DIVERGED and bad[0].n == bad[1].n
    E = torch.diag(torch.tensor([-1.0] * 3 + [1.0] * 5, dtype=torch.float64)).cuda()
    one = sp2.run_dense(E, -1.0, 1.0, 3)
    assert one.status == sp2.OK and one.n == 0 and one.v == [0.0]
    assert torch.equal(one.D, torch.diag((torch.diagonal(E) < 0).to(torch.float64)))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_batch_teams(prec):
    """Few large instances (teams over all XCDs), many small ones (teams of
    one) and trivial ones together; every result equals a second run's."""
    import torch
    import paper_1507_02087_amd as sp2
    rng = np.random.default_rng(3)
    # (600 instances: teams that take one after another from a list)
    for sizes in ([600, 33, 64], [int(x) for x in rng.integers(8, 140, 60)],
                  [int(x) for x in rng.integers(8, 160, 600)]):
        insts = [dense_instance(n, max(1, n // 3), -1.0, 1.0, 0.1, seed=40 + k)
                 for k, n in enumerate(sizes)]
        Fs = [torch.from_numpy(i.F).cuda() for i in insts] + [torch.eye(5, dtype=torch.float64).cuda()]
        lo, hi = [-1.0] * len(Fs), [1.0] * len(Fs)
        no = [i.n_occ for i in insts] + [5]
        print_case(f"resident batch {prec} of {len(Fs)}")
        a, _ = sp2.run_batch(Fs, lo, hi, no, precision=prec)
        b, _ = sp2.run_batch(Fs, lo, hi, no, precision=prec)
        for k, (inst, r, s) in enumerate(zip(insts, a, b)):
            assert r.status == sp2.OK and r.n == s.n and torch.equal(r.D, s.D)
            if k % max(1, len(insts) // 60):
                continue
            De = oracle.density_from_eigenvectors(inst.Q, inst.n_occ)
            err = float(np.linalg.norm(r.D.cpu().numpy() - De)) / math.sqrt(inst.n_occ)
            assert err < D_TOL[prec], (inst.n, err)
        assert a[-1].n == 0 and torch.equal(a[-1].D.cpu(), torch.eye(5, dtype=a[-1].D.dtype))


def test_wait_limit_reports_error(monkeypatch):
    """With a zero limit (forced from the host) a workgroup that has to wait
    for its team gives up at once: the kernel returns and the run reports it;
    a context made afterwards runs normally."""
    import torch
    import paper_1507_02087_amd as sp2
    inst = dense_instance(600, 300, -1.0, 1.0, 0.1, seed=5)
    F = torch.from_numpy(inst.F).cuda()
    monkeypatch.setenv("SP2_PERSIST_WAIT_MS", "0")
    ctx = sp2.Context(0)
    monkeypatch.delenv("SP2_PERSIST_WAIT_MS")
    try:
        ctx.init_dense(F, -1.0, 1.0, 300)
        with pytest.raises(sp2.SP2Error) as e:
            ctx.run()
        assert e.value.status == sp2.HIP_ERROR and "limit" in str(e.value)
    finally:
        ctx.close()
    assert sp2.run_dense(F, -1.0, 1.0, 300).status == sp2.OK


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("kw", [{}, {"launch": "sequence"}, {"homo_lumo": True}])
def test_all_densities_at_once(prec, kw):
    """sp2_batch_get_all equals sp2_batch_get of every instance: resident and
    row-major iterates, trivial and stretched instances, both output types."""
    import torch
    import paper_1507_02087_amd as sp2
    insts = [dense_instance(n, n // 2, -1.0, 1.0, 0.1, seed=70 + n) for n in (2, 31, 64, 97, 200)]
    Fs = [torch.from_numpy(i.F).cuda() for i in insts] + [torch.eye(9, dtype=torch.float64).cuda()]
    no = [i.n_occ for i in insts] + [9]
    m = len(Fs)
    ctx = sp2.BatchContext(0)
    try:
        kw = dict(kw)
        acc = kw.pop("homo_lumo", False)
        ctx.batch_init(Fs, [-1.0] * m, [1.0] * m, no, precision=prec, **kw)
        if acc:
            b = [(float(i.lam[i.n_occ - 1]),) * 2 + (float(i.lam[i.n_occ]),) * 2 for i in insts]
            b.append((-0.5, -0.5, 0.5, 0.5))
            ctx.set_homo_lumo(*[list(c) for c in zip(*b)])
        with pytest.raises(sp2.SP2Error) as e:
            ctx.batch_get_all()
        assert e.value.status == sp2.BAD_STATE
        ctx.batch_run()
        for as64 in (True, False):
            Ds, st, it, sq = ctx.batch_get_all(as_fp64=as64)
            for i in range(m):
                D, s, n, q = ctx.batch_get(i, as_fp64=as64)
                assert (st[i], it[i], sq[i]) == (s, n, q)
                assert Ds[i].dtype == D.dtype and torch.equal(Ds[i], D), i
    finally:
        ctx.close()
