"""Every kernel of the resident run, by precision, tile edge, single run or
batch, and short or long chains: one step against an FP64 product at the
remainders of its tiles, and runs of every method against the exact density.
That the sizes take these kernels is checked on the CPU (plan_edge.cpp)."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from workloads import dense_instance
from tests.gpu_helpers import print_case
from tests.test_gpu_resident import D_TOL, U, _step_bound

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# (precision, edge / 16): sizes of single runs. Whole tiles, one row more and
# one less, an odd K; the first of FP32's 32 and 48 rows are the short chains
# (N <= 1050), and so are FP64's of 32 rows up to there.
SINGLE = {
    ("fp64", 2): (351, 352, 353, 1089, 1120), ("fp64", 3): (767, 768, 769, 1250, 1441, 1450),
    ("fp64", 4): (1855, 1856, 1857, 1900),
    ("fp32", 2): (351, 352, 353, 1087, 1088, 1100), ("fp32", 3): (767, 768, 769, 1055, 1440, 1450),
    ("fp32", 4): (1279, 1280, 1281, 1300), ("fp32", 5): (1679, 1680, 1681, 1700),
    ("bf16x3", 2): (351, 352, 353, 975), ("bf16x3", 4): (1023, 1024, 1025, 1311),
}
# batches: (size, count); the odd member has a remainder of its own
BATCH = {
    ("fp64", 2): (353, 3), ("fp64", 3): (1000, 7), ("fp64", 4): (577, 63),
    ("fp32", 2): (1500, 3), ("fp32", 3): (1025, 4), ("fp32", 4): (1025, 31),
    ("bf16x3", 2): (193, 4), ("bf16x3", 4): (1025, 4),
}
PRECISIONS = {"fp64": 0, "fp32": 1, "bf16x3": 2}


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
def test_sizes_take_every_edge(tmp_path):
    exe = str(tmp_path / "plan_edge")
    csrc = os.path.join(ROOT, "paper_1507_02087_amd", "csrc")
    b = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950",
                        "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "plan_edge.cpp"),
                        "-x", "hip", os.path.join(csrc, "host_plan.hip"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-3000:]

    def edge(prec, *sizes):
        return int(subprocess.run([exe, str(PRECISIONS[prec]), *sizes], capture_output=True,
                                  text=True, check=True).stdout)
    for (prec, mb), sizes in SINGLE.items():
        assert [edge(prec, str(n)) for n in sizes] == [mb] * len(sizes), (prec, mb)
    for (prec, mb), (n, count) in BATCH.items():
        assert edge(prec, f"{n}x{count}", str(n - 13)) == mb, (prec, mb)


def _start(n, seed):
    """(F, bounds, X0): a dense F with spectrum inside [-1, 1]."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    F = (A + A.t()) / (4.0 * math.sqrt(n))
    hi = max(1.0, float(F.abs().sum(1).max()))
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    return F, hi, (hi * eye - F) / (2 * hi)


def _check_step(prec, n, X0, D, p1, t1):
    import torch
    if prec != "fp64":
        X0 = X0.to(torch.float32).to(torch.float64)
    S = X0 @ X0
    X1 = S if p1 else 2 * X0 - S
    assert torch.equal(D, D.t())
    tol = _step_bound(prec, n) * (2.0 if prec == "fp64" else 1.0)
    assert float((D - X1).abs().max()) <= tol, (n, float((D - X1).abs().max()), tol)
    assert abs(t1 - float(torch.trace(D))) <= 4 * n * U["fp64"] * max(1.0, n)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,mb", sorted(SINGLE))
def test_one_step_single(prec, mb):
    import paper_1507_02087_amd as sp2
    ctx = sp2.Context(0)
    try:
        for n in SINGLE[prec, mb]:
            F, hi, X0 = _start(n, n)
            print_case(f"edge {mb} one step {prec} n={n}")
            r = sp2.run_dense(F, -hi, hi, n // 2, precision=prec, max_iter=1, as_fp64=True, ctx=ctx)
            assert r.status_name == "NOT_CONVERGED" and r.n == 1
            _check_step(prec, n, X0, r.D, r.p[1], r.t1[1])
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec,mb", sorted(BATCH))
def test_one_step_batch(prec, mb):
    import paper_1507_02087_amd as sp2
    n, count = BATCH[prec, mb]
    two = [_start(n, 1), _start(n - 13, 2)]
    his = [two[0][1]] * count + [two[1][1]]
    print_case(f"edge {mb} one step {prec} batch {count} x {n}")
    rs, _ = sp2.run_batch([two[0][0]] * count + [two[1][0]], [-h for h in his], his,
                          [n // 2] * count + [n // 3], precision=prec, max_iter=1)
    for k in (0, count // 2, count - 1, count):
        r, (_, _, X0) = rs[k], two[k == count]
        assert r.status_name == "NOT_CONVERGED" and r.n == 1
        _check_step(prec, X0.shape[0], X0, r.D, r.p[1], r.t1[1])


def _methods(inst, n_occ):
    h, l = float(inst.lam[n_occ - 1]), float(inst.lam[n_occ])
    return {"sp2": {}, "acc": {"homo_lumo": (h, h, l, l)},
            "mcweeny": {"mcweeny": (0.5 * (h + l), None)},
            "mcw_acc": {"mcweeny": (0.5 * (h + l), l - h)}}


@pytest.mark.gpu
@pytest.mark.parametrize("prec,mb", sorted(SINGLE))
def test_methods_single(prec, mb):
    import torch
    import paper_1507_02087_amd as sp2
    n = SINGLE[prec, mb][-1]
    inst = dense_instance(n, n // 3, -1.0, 1.0, 0.1, seed=500 + n)
    F = torch.from_numpy(inst.F).cuda()
    De = oracle.density_from_eigenvectors(inst.Q, n // 3)
    for method, kw in _methods(inst, n // 3).items():
        print_case(f"edge {mb} {method} {prec} n={n}")
        r = sp2.run_dense(F, -1.0, 1.0, n // 3, precision=prec, **kw)
        assert r.status == sp2.OK
        err = float(np.linalg.norm(r.D.cpu().numpy() - De)) / math.sqrt(n // 3)
        assert err < D_TOL[prec], (method, err)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,mb", sorted(BATCH))
def test_methods_batch(prec, mb):
    """SP2 and McWeeny (the largest batches' goes to another driver)."""
    import torch
    import paper_1507_02087_amd as sp2
    n, count = BATCH[prec, mb]
    inst = dense_instance(n, n // 3, -1.0, 1.0, 0.1, seed=600 + n)
    F = torch.from_numpy(inst.F).cuda()
    De = oracle.density_from_eigenvectors(inst.Q, n // 3)
    m = count + 1
    for method in ("sp2", "mcweeny"):
        ctx = sp2.BatchContext(0)
        try:
            print_case(f"edge {mb} {method} {prec} batch {m} x {n}")
            ctx.batch_init([F] * m, [-1.0] * m, [1.0] * m, [n // 3] * m, precision=prec)
            if method == "mcweeny":
                ctx.set_mcweeny([0.5 * float(inst.lam[n // 3 - 1] + inst.lam[n // 3])] * m)
            ctx.batch_run()
            for k in (0, m // 2, m - 1):
                D, status, _, _ = ctx.batch_get(k)
                assert status == sp2.OK
                err = float(np.linalg.norm(D.cpu().numpy() - De)) / math.sqrt(n // 3)
                assert err < D_TOL[prec], (method, k, err)
        finally:
            ctx.close()
