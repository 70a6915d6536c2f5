"""A resident run whose teams do not meet in time (other work holds the
device; here a limit of zero, set by the host) is done again by the other
driver: the same results as that driver's, bit for bit, and no error."""
import pytest

from workloads import dense_instance
from tests.gpu_helpers import print_case

pytestmark = pytest.mark.gpu


def _context(monkeypatch, cls):
    monkeypatch.setenv("SP2_RESIDENT_WAIT_MS", "0")
    ctx = cls(0)
    monkeypatch.delenv("SP2_RESIDENT_WAIT_MS")
    return ctx


def _equal(a, b):
    import torch
    assert a.status == b.status and a.n == b.n
    assert a.v == b.v and a.t1 == b.t1 and a.p == b.p and torch.equal(a.D, b.D)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_changes_over_to_the_other_driver(monkeypatch, prec):
    import torch
    import paper_1507_02087_amd as sp2
    insts = [dense_instance(n, n // 2, -1.0, 1.0, 0.1, seed=80 + n) for n in (300, 64, 129)]
    Fs = [torch.from_numpy(i.F).cuda() for i in insts]
    lam = insts[0].lam
    h, l = float(lam[149]), float(lam[150])
    for kw in ({}, {"homo_lumo": (h, h, l, l)}, {"mcweeny": (0.5 * (h + l), None)},
               {"mcweeny": (0.5 * (h + l), l - h)}):
        print_case(f"resident wait 0, {prec} {kw}")
        ctx = _context(monkeypatch, sp2.Context)
        try:
            want = sp2.run_dense(Fs[0], -1.0, 1.0, 150, precision=prec, launch="sequence", **kw)
            for _ in range(2):   # the run that changes over, and one after it
                _equal(sp2.run_dense(Fs[0], -1.0, 1.0, 150, precision=prec, ctx=ctx, **kw), want)
        finally:
            ctx.close()
    print_case(f"resident wait 0, batch {prec}")
    ctx = _context(monkeypatch, sp2.BatchContext)
    try:
        args = (Fs, [-1.0] * 3, [1.0] * 3, [i.n_occ for i in insts])
        want, _ = sp2.run_batch(*args, precision=prec, launch="persistent")
        for _ in range(2):
            got, _ = sp2.run_batch(*args, precision=prec, ctx=ctx)
            for a, b in zip(got, want):
                _equal(a, b)
    finally:
        ctx.close()


def test_spectral_norm_changes_over(monkeypatch):
    """To the chunked kernel, which a batch of two runs."""
    import torch
    import paper_1507_02087_amd as sp2
    inst = dense_instance(300, 150, -1.0, 1.0, 0.1, seed=77)
    F = torch.from_numpy(inst.F).cuda()
    two, _ = sp2.run_batch([F, F], [-1.0] * 2, [1.0] * 2, [150] * 2, precision="fp64",
                           norm="spectral", tail_split=1)
    print_case("spectral norm, wait 0")
    ctx = _context(monkeypatch, sp2.Context)
    try:
        for _ in range(2):
            one = sp2.run_dense(F, -1.0, 1.0, 150, precision="fp64", norm="spectral",
                                tail_split=1, ctx=ctx)
            _equal(one, two[0])
            assert one.m == two[0].m
    finally:
        ctx.close()
