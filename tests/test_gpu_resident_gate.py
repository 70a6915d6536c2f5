"""Small resident runs are ordinary launches behind a gate: runs of several
threads overlap, and one whose gate was shut is launched cooperatively, with
the same results bit for bit."""
import threading
import time

import pytest

from workloads import dense_instance
from tests.gpu_helpers import print_case

pytestmark = pytest.mark.gpu


def _threads(sp2, F, prec, launch, count, runs):
    """(densities, seconds) of `runs` runs on each of `count` threads."""
    import torch
    n = F.shape[0]
    ctxs = [sp2.Context(0, torch.cuda.Stream()) for _ in range(count)]
    Ds = [torch.empty(n, n, dtype=torch.float64, device="cuda") for _ in range(count)]
    torch.cuda.synchronize()
    bad = []

    def work(i, k):
        try:
            for _ in range(k):
                ctxs[i].init_dense(F, -1.0, 1.0, n // 2, prec, launch=launch)
                ctxs[i].run()
                ctxs[i].get_density(Ds[i])
        except Exception as e:   # reported below
            bad.append(e)

    def go(k):
        t = [threading.Thread(target=work, args=(i, k)) for i in range(count)]
        t0 = time.perf_counter()
        for x in t:
            x.start()
        for x in t:
            x.join()
        return time.perf_counter() - t0

    try:
        go(3)
        took = min(go(runs) for _ in range(3))
        assert not bad, bad
        return Ds, took
    finally:
        for c in ctxs:
            c.close()


@pytest.mark.parametrize("prec,n", [("fp64", 40), ("fp64", 64), ("fp32", 150), ("bf16x3", 480)])
def test_threads_overlap(prec, n):
    """Twelve threads' runs are not slower than as launch sequences (taking
    turns they were, by a tenth; overlapping they take a third)."""
    import torch
    import paper_1507_02087_amd as sp2
    inst = dense_instance(n, n // 2, -1.0, 1.0, 0.1, seed=33)
    F = torch.from_numpy(inst.F).cuda()
    print_case(f"gate threads {prec} n={n}")
    alone = sp2.run_dense(F, -1.0, 1.0, n // 2, precision=prec)
    Ds, took = _threads(sp2, F, prec, "auto", 12, 30)
    for D in Ds:
        assert torch.equal(D, alone.D)
    _, sequence = _threads(sp2, F, prec, "sequence", 12, 30)
    assert took < sequence, (took, sequence)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_a_shut_gate_changes_nothing(monkeypatch, prec):
    import torch
    import paper_1507_02087_amd as sp2
    # one workgroup, a few, the largest team behind a gate and one past it
    for n in (20, 33, 100, 480, 520):
        inst = dense_instance(n, n // 2, -1.0, 1.0, 0.1, seed=34)
        F = torch.from_numpy(inst.F).cuda()
        h, l = float(inst.lam[n // 2 - 1]), float(inst.lam[n // 2])
        for kw in ({}, {"mcweeny": (0.5 * (h + l), l - h)}):
            print_case(f"gate {prec} n={n} {kw}")
            want = sp2.run_dense(F, -1.0, 1.0, n // 2, precision=prec, **kw)
            assert want.status == sp2.OK
            monkeypatch.setenv("SP2_GATE_WAIT_MS", "0")
            ctx = sp2.Context(0)
            monkeypatch.delenv("SP2_GATE_WAIT_MS")
            try:
                for _ in range(3):
                    got = sp2.run_dense(F, -1.0, 1.0, n // 2, precision=prec, ctx=ctx, **kw)
                    assert got.v == want.v and got.p == want.p and torch.equal(got.D, want.D)
            finally:
                ctx.close()
