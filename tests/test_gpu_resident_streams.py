"""Resident runs of several contexts at once: every run needs its whole grid
on the card, so runs on other streams and threads, and other work beside
them, may delay it but change neither its outcome nor its result."""
import threading

import pytest

from workloads import dense_instance
from tests.gpu_helpers import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [("fp64", 700), ("fp32", 1777), ("fp32", 3001)])
def test_threads_on_their_own_streams(prec, n):
    import torch
    import paper_1507_02087_amd as sp2
    # 231 to 512 workgroups a run: two runs together do not fit the card
    inst = dense_instance(n, n // 2, -1.0, 1.0, 0.1, seed=31)
    F = torch.from_numpy(inst.F).cuda()
    A = torch.ones(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    print_case(f"resident threads {prec} N={n}")
    alone = sp2.run_dense(F, -1.0, 1.0, n // 2, precision=prec)
    assert alone.status == sp2.OK
    out, bad = [], []

    def work():
        try:
            stream = torch.cuda.Stream()
            ctx = sp2.Context(0, stream)
            try:
                ctx.init_dense(F, -1.0, 1.0, n // 2, prec)
                for _ in range(5):
                    ctx.run()
                    D = torch.empty(n, n, dtype=alone.D.dtype, device="cuda")
                    stream.wait_stream(torch.cuda.current_stream())
                    ctx.get_density(D)
                    out.append((ctx.get_info()[1], D))
            finally:
                ctx.close()
        except Exception as e:   # reported by the main thread
            bad.append(e)

    threads = [threading.Thread(target=work) for _ in range(3)]
    for t in threads:
        t.start()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(40):
            A @ A
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad, bad
    assert len(out) == 15
    for squares, D in out:
        assert squares == out[0][0] and torch.equal(D, alone.D)
