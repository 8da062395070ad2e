"""Series by lists beside other work: threads with a context each run same
generation (a workgroup on every second and on every compute unit) and the
one-launch closure while products on another stream keep the chip busy.
Whether a launch finds its workgroups room together or gives up and the series
is run by products, every model, count and number of steps is right."""
from __future__ import annotations

import threading

import numpy as np
import pytest

import dlgen
import oracle
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu


def test_same_generation_on_a_busy_chip():
    import torch

    import paper_1608_00139_amd as dl

    cases = []
    for n in (1000, 4096, 8192):
        p = dlgen.to_dense(n, dlgen.forest_edges(n, n))
        pd = dev(p)
        s, iters = dl.dl_sg(pd)
        ref, _, it, _ = oracle.sg_seminaive(p)
        assert iters == it and np.array_equal(host(s), ref)
        cases.append((lambda out, ctx, pd=pd: dl.dl_sg(pd, out=out, ctx=ctx)[1], s, iters, n))
    a = dev(dlgen.to_dense(1500, dlgen.er_edges(1500, 2.0 / 1500, 3)))
    r, iters = dl.dl_tc(a)
    cases.append((lambda out, ctx: dl.dl_tc(a, out=out, ctx=ctx)[1], r, iters, 1500))
    wrong = []

    def work(call, want, iters, n):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = dl.Context()
            out = torch.empty_like(want)
            for k in range(15):
                announce("busy lists", n, k)
                try:
                    it = call(out, ctx)
                except dl.DLError as err:
                    wrong.append((n, k, str(err)))
                    continue
                if it != iters or not bool((out == want).all()):
                    wrong.append((n, k, it))
            ctx.close()

    torch.cuda.synchronize()
    busy = torch.cuda.Stream()
    threads = [threading.Thread(target=work, args=c) for c in cases]
    with torch.cuda.stream(busy):
        x = torch.rand((4096, 4096), device="cuda")
        y = torch.empty_like(x)
        for t in threads:
            t.start()
        while any(t.is_alive() for t in threads):
            for _ in range(4):
                torch.mm(x, x, out=y)
            busy.synchronize()
    for t in threads:
        t.join()
    assert not wrong, wrong[:5]


@pytest.mark.parametrize("n", [40, 300, 4096])
def test_beside_long_products(n):
    """Calls on a stream of their own while large products hold the chip: one
    that gives up is run by products, and the next launch clears its counters
    first."""
    import torch

    import paper_1608_00139_amd as dl
    from tests.gpu_routes import base, kernels

    lists = ["k_row_lists", "k_sg_lists"]
    x = torch.rand((8192, 8192), device="cuda")
    y = torch.empty_like(x)
    busy, side = torch.cuda.Stream(), torch.cuda.Stream()
    pd = dev(dlgen.to_dense(n, dlgen.forest_edges(n, n)))
    want, iters = dl.dl_sg(pd)
    got = []

    def beside():
        with torch.cuda.stream(busy):
            for _ in range(3):
                torch.mm(x, x, out=y)
        with torch.cuda.stream(side):
            got.append(dl.dl_sg(pd))

    for k in range(6):
        announce("beside products", n, k)
        first = base(kernels(beside))
        then = base(kernels(lambda: got.append(dl.dl_sg(pd))))
        gave_up = first[:2] == lists and "k_ingest" in first
        assert gave_up or first == lists, first
        assert then == (["k_lists_clear"] if gave_up else []) + lists, then
    for s, it in got:
        assert it == iters and bool((s == want).all())
