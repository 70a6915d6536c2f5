"""The spectral norm of a single instance from registers (spectral_run.hip)
against the chunked kernel, which a batch of two runs: the same Lanczos
process from the same start vector, so the same estimates after the same
number of steps, at the edges of every register layout, past the largest and
under a stretch."""
import numpy as np
import pytest

from tests.gpu_helpers import print_case
from tests.test_gpu_spectral import CLUSTER_REL

pytestmark = pytest.mark.gpu

# workgroups of 8 or 16 rows; 512, 1024, 2040 | 2816, 3072, 4080: the largest
# rows of a layout; 4081 / 2817 (FP64): the chunked kernel
SIZES = {"fp32": (1, 7, 8, 9, 33, 512, 513, 1024, 1030, 2040, 2041, 3072, 3073, 4080, 4081),
         "fp64": (2, 16, 100, 513, 1025, 2041, 2816, 2817)}


def _instance(n):
    """F with one eigenvalue of E_0 standing out (X_0 at 0.5), the rest within
    [0, 0.2] and [0.8, 1]: Lanczos converges in a few steps."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    lam = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 0.4 - 1.0
    lam[n // 2:] *= -1.0
    lam[0] = 0.0
    # Householder reflections keep the spectrum
    F = torch.diag(lam)
    for _ in range(3):
        u = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
        u /= u.norm()
        Fu = F @ u
        F = F - 2 * torch.outer(u, Fu) - 2 * torch.outer(Fu, u) + 4 * (u @ Fu) * torch.outer(u, u)
    return 0.5 * (F + F.t()), max(1, n // 2)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_matches_the_chunked_kernel(prec):
    import paper_1507_02087_amd as sp2
    for n in SIZES[prec]:
        F, n_occ = _instance(n)
        if n_occ == n:
            n_occ = 0
        print_case(f"spectral norm from registers {prec} n={n}")
        ctx, two = sp2.Context(0), sp2.BatchContext(0)
        try:
            kw = dict(precision=prec, norm="spectral", max_iter=3)
            ctx.init_dense(F, -1.0, 1.0, n_occ, **kw)
            ctx.run()
            e, k = ctx.get_norm_history(krylov=True)
            two.batch_init([F, F], [-1.0] * 2, [1.0] * 2, [n_occ] * 2, **kw)
            two.batch_run()
            e2, k2 = two.get_norm_history(0, krylov=True)
            assert len(e) == len(e2)
            for i, (a, b, ka, kb) in enumerate(zip(e, e2, k, k2)):
                if i > 0:
                    # E_1, E_2: a clustered top, where a process may stall on
                    # its way; each estimate is within CLUSTER_REL of the norm
                    # (test_gpu_spectral.py)
                    assert abs(a - b) <= CLUSTER_REL * b, (n, a, b)
                    continue
                # the isolated top of E_0: converged, the estimate is good to
                # the 1e-12 of its test; the sums are taken in another order,
                # so a step more or less
                assert abs(a - b) <= 1e-10 * b, (n, a, b)
                assert abs(ka - kb) <= 2, (n, ka, kb)
            if len(e) and n > 1:
                assert abs(e[0] - 0.25) < 1e-6
        finally:
            ctx.close()
            two.close()


def test_stretched_run_matches_the_chunked_kernel():
    """SP2-ACC: the buffer holds a X~ + c I."""
    import paper_1507_02087_amd as sp2
    from workloads import dense_instance
    import torch
    inst = dense_instance(300, 150, -1.0, 1.0, 0.1, seed=77)
    F = torch.from_numpy(inst.F).cuda()
    b = (float(inst.lam[149]),) * 2 + (float(inst.lam[150]),) * 2
    one = sp2.run_dense(F, -1.0, 1.0, 150, precision="fp64", norm="spectral", homo_lumo=b)
    out, _ = sp2.run_batch([F, F], [-1.0] * 2, [1.0] * 2, [150] * 2, precision="fp64",
                           norm="spectral", homo_lumo=[[x, x] for x in b])
    assert one.status == out[0].status == sp2.OK and one.n == out[0].n
    # clustered tops end at 64 steps, where the estimates agree less closely
    big = [i for i, x in enumerate(one.m) if x > 1e-10]
    assert np.allclose(np.array(one.m)[big], np.array(out[0].m)[big], rtol=1e-4)


def test_wait_limit_reports_error(monkeypatch):
    import paper_1507_02087_amd as sp2
    F, n_occ = _instance(300)
    monkeypatch.setenv("SP2_PERSIST_WAIT_MS", "0")
    ctx = sp2.Context(0)
    monkeypatch.delenv("SP2_PERSIST_WAIT_MS")
    try:
        ctx.init_dense(F, -1.0, 1.0, n_occ, norm="spectral", max_iter=3)
        with pytest.raises(sp2.SP2Error) as e:
            ctx.run()
        assert e.value.status == sp2.HIP_ERROR and "limit" in str(e.value)
    finally:
        ctx.close()
