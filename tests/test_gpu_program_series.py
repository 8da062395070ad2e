"""The Boolean series of program layers where its early exit can go wrong:
layers whose steps are element-wise kernels only, heads that mix products and
element-wise terms (partial sums in scratch), empty constant parts, and
series longer than one group of steps.  Models and iteration counts against
the oracle (exact)."""
from __future__ import annotations

import numpy as np
import pytest

import dlgen
from oracle import program as oprog
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu

UNIT = """
p(X,Y) :- e(X,Y).
p(X,Y) :- q(X,Y).
q(X,Y) :- p(X,Y).
q(X,Y) :- f(X,Y).
"""
MIXED = """
p(X,Y) :- q(X,Y).
p(X,Y) :- e(X,Z), p(Z,Y).
p(X,Y) :- f(X,Y).
q(X,Y) :- p(Y,X).
q(X,Y) :- e(X,Y).
q(X,Y) :- p(X,Z), f(Z,Y).
"""
NO_BASE = """
p(X,Y) :- e(X,Z), p(Z,Y).
q(X,Y) :- f(X,Y).
q(X,Y) :- p(X,Z), q(Z,Y).
"""
PATH = """
p(X,Y) :- e(X,Y).
p(X,Y) :- e(X,Z), p(Z,Y).
"""


@pytest.fixture(scope="module")
def dl():
    import paper_1608_00139_amd as m

    m.load()
    return m


def _check(dl, prog, text, rels, n):
    want, layers = oprog.evaluate(text, rels, n)
    iters = {tuple(h): it for h, it in layers}
    for name, m in want.items():
        got, ones = prog.fetch(name, n=n)
        assert np.array_equal(host(got), m), name
        assert ones == int(m.sum())
    for layer in prog.layers():
        assert layer["iters"] == iters[tuple(layer["heads"])], layer


@pytest.mark.parametrize("text", [UNIT, MIXED, NO_BASE], ids=["unit", "mixed", "no_base"])
@pytest.mark.parametrize("n", [2, 63, 256, 300])
def test_series_vs_oracle(dl, text, n):
    for seed in range(3):
        rels = {k: dlgen.to_dense(n, dlgen.er_edges(n, min(0.4, 1.5 / n), 10 * seed + i)) for i, k in enumerate("ef")}
        announce("program series", n, seed)
        prog = dl.Program(text)
        keep = {k: dev(v) for k, v in rels.items()}
        for k, t in keep.items():
            prog.bind(k, t)
        prog.run(dl.DL_EVAL_ITERATION)
        _check(dl, prog, text, rels, n)
        prog.close()


@pytest.mark.parametrize("m", [3, 4, 5, 6, 11, 20, 70])
def test_path_lengths_across_groups(dl, m):
    """A path of m edges: m + 1 applications, on both sides of every group end."""
    n = m + 1
    e = np.zeros((n, n), dtype=np.uint8)
    e[np.arange(m), np.arange(1, n)] = 1
    announce("program path", m)
    prog = dl.Program(PATH)
    ed = dev(e)
    prog.bind("e", ed)
    prog.run(dl.DL_EVAL_ITERATION)
    _check(dl, prog, PATH, {"e": e}, n)
    assert prog.layers()[0]["iters"] == m + 1
    prog.close()


def test_rerun_and_two_programs_share_a_context(dl):
    """Runs again at other sizes and beside other programs of the same
    context, some destroyed in between: results are each program's own."""
    ctx = dl.Context()
    b = dl.Program(PATH, ctx=ctx)
    old = []
    for k, n in enumerate((300, 40, 300, 700, 256)):
        rels = {e: dlgen.to_dense(n, dlgen.er_edges(n, 1.5 / n, 3 * n + i)) for i, e in enumerate("ef")}
        keep = {e: dev(v) for e, v in rels.items()}
        announce("program rerun", n)
        a = dl.Program(MIXED, ctx=ctx)
        for e in "ef":
            a.bind(e, keep[e])
        b.bind("e", keep["e"])
        for _ in range(2):
            a.run(dl.DL_EVAL_ITERATION)
            b.run(dl.DL_EVAL_ITERATION)
            _check(dl, a, MIXED, rels, n)
            _check(dl, b, PATH, {"e": rels["e"]}, n)
        b.run(dl.DL_EVAL_MATRIX)
        want, _ = oprog.evaluate(PATH, {"e": rels["e"]}, n)
        assert np.array_equal(host(b.fetch("p", n=n)[0]), want["p"])
        _check(dl, a, MIXED, rels, n)
        old.append((a, rels, n))
        if k % 2:
            old.pop(0)[0].close()
    for a, rels, n in old:  # results of earlier programs are still there
        _check(dl, a, MIXED, rels, n)
        a.close()
    b.close()
    ctx.close()


def test_budget_and_destroy_order(dl):
    """A context with a budget keeps nothing and still refuses past it; a
    program may outlive the runs of others that share its matrices."""
    n = 300  # Np = 512: 256 KB a matrix
    e = dlgen.to_dense(n, dlgen.er_edges(n, 1.5 / n, 1))
    ed = dev(e)
    want, _ = oprog.evaluate(PATH, {"e": e}, n)
    announce("program budget")
    small = dl.Context(workspace_budget=5 << 18)
    prog = dl.Program(PATH, ctx=small)
    prog.bind("e", ed)
    for _ in range(2):
        with pytest.raises(dl.DLError):
            prog.run(dl.DL_EVAL_ITERATION)
    prog.close()
    enough = dl.Context(workspace_budget=9 << 18)
    prog = dl.Program(PATH, ctx=enough)
    prog.bind("e", ed)
    for _ in range(3):
        prog.run(dl.DL_EVAL_ITERATION)
        assert np.array_equal(host(prog.fetch("p", n=n)[0]), want["p"])
    prog.close()
    one, two = dl.Program(PATH), dl.Program(PATH)
    for p in (one, two):
        p.bind("e", ed)
        p.run(dl.DL_EVAL_ITERATION)
    one.close()
    two.run(dl.DL_EVAL_ITERATION)
    assert np.array_equal(host(two.fetch("p", n=n)[0]), want["p"])
    two.close()
