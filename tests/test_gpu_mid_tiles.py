"""The 128 x 128 and 64 x 64 product configurations where they can go wrong:
more tiles than resident workgroups (a workgroup takes several, the next one's
first slice fetched meanwhile), addends and identities (programs, same
generation), every precision, and the sizes around which the size rule
changes configuration.  Models and counts against the oracle, exactly."""
from __future__ import annotations

import numpy as np
import pytest

import dlgen
import oracle
from oracle import program as oprog
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu
PRECS = ["i8", "f32", "bf16", "fp8", "fp4"]


@pytest.fixture(scope="module")
def dl():
    import paper_1608_00139_amd as m

    m.load()
    return m


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,cfg", [(1500, 2), (1600, 1), (2900, 1), (3200, 1)])
def test_several_tiles_per_workgroup(dl, prec, n, cfg):
    ctx = dl.Context()
    a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, n))
    want = oracle.tc_seminaive(a)[0]
    ctx.set_tuning(prec, n, cfg)
    ad = dev(a)
    announce("mid tiles", prec, n, cfg)
    r, it = dl.dl_tc(ad, prec=prec, ctx=ctx)
    ones = dl.dl_tc_steps(ad, 64, prec=prec, ctx=ctx).ones
    ctx.set_tuning(prec, n, 0)
    r0, it0 = dl.dl_tc(ad, prec=prec, ctx=ctx)
    assert np.array_equal(host(r), want) and it == it0 and bool((r == r0).all())
    assert ones == dl.dl_tc_steps(ad, 64, prec=prec, ctx=ctx).ones
    ctx.close()


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [1024, 1025, 1537, 2817, 3073])
def test_sizes_around_the_rule(dl, prec, n):
    a = dlgen.to_dense(n, dlgen.er_edges(n, 1.5 / n, n))
    announce("size rule", prec, n)
    r, _ = dl.dl_tc(dev(a), prec=prec)
    assert np.array_equal(host(r), oracle.tc_seminaive(a)[0])


@pytest.mark.parametrize("n", [1100, 2900, 3100])
def test_same_generation(dl, n):
    p = dlgen.to_dense(n, dlgen.forest_edges(n, n))
    want, _, iters, _ = oracle.sg_seminaive(p)
    announce("mid tiles sg", n)
    s, it = dl.dl_sg(dev(p))
    assert np.array_equal(host(s), want) and it == iters


@pytest.mark.parametrize("cfg", [1, 2])
def test_program_addends(dl, cfg):
    """Two recursive terms a head: running sums as addends of the product."""
    text = ("p(X,Y) :- e(X,Y).\np(X,Y) :- e(X,Z), p(Z,Y).\np(X,Y) :- p(X,Z), f(Z,Y).\n"
            "q(X,Y) :- p(X,Z), not p(Z,Y).")
    n = 600
    ctx = dl.Context()
    ctx.set_tuning("i8", n, cfg)
    rels = {k: dlgen.to_dense(n, dlgen.er_edges(n, 1.0 / n, i)) for i, k in enumerate("ef")}
    keep = {k: dev(v) for k, v in rels.items()}
    prog = dl.Program(text, ctx=ctx)
    for k, t in keep.items():
        prog.bind(k, t)
    announce("mid tiles program", cfg)
    prog.run(dl.DL_EVAL_ITERATION)
    want, _ = oprog.evaluate(text, rels, n)
    for name in ("p", "q"):
        assert np.array_equal(host(prog.fetch(name, n=n)[0]), want[name]), name
    prog.close()
    ctx.close()
