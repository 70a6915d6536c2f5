"""The driver that a batch takes by default, told from its results bit by
bit: the queue's (McWeeny: the launch sequence's) where that is the faster
one, the resident run's, which add in another order, where it is not."""
import pytest

from tests.gpu_helpers import print_case

pytestmark = pytest.mark.gpu


def _matrix(n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    return (A + A.t()) / (4.0 * n ** 0.5)


def _run(sp2, Fs, prec, mcweeny):
    m = len(Fs)
    ctx = sp2.BatchContext(0)
    try:
        ctx.batch_init(Fs, [-1.0] * m, [1.0] * m, [F.shape[0] // 2 for F in Fs], precision=prec,
                       max_iter=3)
        if mcweeny:
            ctx.set_mcweeny([0.0] * m)
        ctx.batch_run()
        Ds, st, _, _ = ctx.batch_get_all()
        assert all(s == sp2.NOT_CONVERGED for s in st)
        return Ds
    finally:
        ctx.close()


@pytest.mark.parametrize("prec,sizes,mcweeny,resident", [
    ("bf16x3", [2000] * 5, False, False),
    ("bf16x3", [1300] * 2 + [301], False, True),
    ("bf16x3", [1250] * 8, True, False),
    ("bf16x3", [300] * 4, True, True),
    ("fp32", [2200] * 3, False, False),
    ("fp32", [900] * 3, False, True),
    ("fp32", [1600] * 3, True, False),
    ("fp32", [400, 700, 33], True, True),
    ("fp64", [1800] * 3, False, False),
    ("fp64", [700] * 3, False, True),
    ("fp64", [210] * 40, True, False),
    ("fp64", [410] * 3, True, True)])
def test_default_driver(monkeypatch, prec, sizes, mcweeny, resident):
    import torch
    import paper_1507_02087_amd as sp2
    mats = {n: _matrix(n) for n in set(sizes)}
    Fs = [mats[n] for n in sizes]
    print_case(f"default driver {prec} {len(sizes)} x {sizes[0]} mcweeny={mcweeny}")
    got = _run(sp2, Fs, prec, mcweeny)
    # a resident run that may not wait changes over to the other driver
    monkeypatch.setenv("SP2_RESIDENT_WAIT_MS", "0")
    other = _run(sp2, Fs, prec, mcweeny)
    same = all(torch.equal(a, b) for a, b in zip(got, other))
    assert same == (not resident)
    for a, b in zip(got, other):
        assert float((a - b).abs().max()) < 1e-3
