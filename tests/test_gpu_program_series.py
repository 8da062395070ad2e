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


LEFT = """
p(X,Y) :- e(X,Y).
p(X,Y) :- p(X,Z), f(Z,Y).
"""
CHAINED = """
p(X,Y) :- e(X,Y).
p(X,Y) :- e(X,Z), f(Z,W), p(W,Y).
q(X,Y) :- f(X,Z), not p(Z,Y).
q(X,Y) :- e(X,Z), q(Z,Y).
"""
NEGATED = """
p(X,Y) :- e(X,Y).
q(X,Y) :- f(X,Y).
q(X,Y) :- not p(X,Z), q(Z,Y).
"""


@pytest.mark.parametrize("text", [PATH, LEFT, NO_BASE, CHAINED, NEGATED],
                         ids=["right", "left", "no_base", "chained", "negated"])
@pytest.mark.parametrize("n", [511, 512, 545, 1000])
def test_series_by_lists_vs_oracle(dl, text, n):
    """Layers with one recursive term, by lists of the relation's entries
    (at most 32 a row) and, for a longer row or a complement, by
    products: models and iteration counts."""
    rng = np.random.default_rng(n)
    for kind in ("sparse", "loops and longer lists", "long row", "empty base"):
        loops = kind == "loops and longer lists"
        rels = {k: dlgen.to_dense(n, dlgen.er_edges(n, (8 if loops else 1) * d / n, 5 * n + i, self_loops=loops))
                for i, (k, d) in enumerate((("e", 1.0), ("f", 2.0)))}
        if loops:  # lists on both sides of the entries kept at hand, each with its own row
            for m in rels.values():
                for row in range(0, n, 7):
                    m[row] = 0
                    m[row, rng.choice(n, row % 12, replace=False)] = 1
                    m[row, row] = 1
        if kind == "long row":
            for m in rels.values():
                m[n - 1] = 0
                m[n - 1, rng.choice(n, 33, replace=False)] = 1
                m[rng.choice(n, 33, replace=False), n - 2] = 1
        if kind == "empty base":
            rels["e"][:] = 0
        announce("program lists", n, kind)
        prog = dl.Program(text)
        keep = {k: dev(v) for k, v in rels.items()}
        for k, t in keep.items():
            if f"{k}(" in text:
                prog.bind(k, t)
        prog.run(dl.DL_EVAL_ITERATION)
        _check(dl, prog, text, {k: v for k, v in rels.items() if f"{k}(" in text}, n)
        prog.close()


@pytest.mark.parametrize("text", [PATH, LEFT], ids=["right", "left"])
@pytest.mark.parametrize("n", [1, 2, 31, 33, 64, 65, 200, 257])
def test_small_series_by_lists(dl, text, n):
    """The smallest sizes, where every row is short (n <= 32) or one in the
    middle, beyond the first eight, is too long for a list (n > 33)."""
    for long_row in (False, True):
        rels = {k: dlgen.to_dense(n, dlgen.er_edges(n, min(0.5, 1.5 / n), n + i, self_loops=True)) for i, k in enumerate("ef")}
        if long_row:
            for m in rels.values():
                m[n // 2] = 1
                m[:, n // 2] = 1
        announce("small program lists", n, long_row)
        prog = dl.Program(text)
        keep = {k: dev(v) for k, v in rels.items() if f"{k}(" in text}
        for k, t in keep.items():
            prog.bind(k, t)
        prog.run(dl.DL_EVAL_ITERATION)
        _check(dl, prog, text, {k: rels[k] for k in keep}, n)
        prog.close()


def test_long_path_by_lists(dl):
    """A path of 700 constants (the longest series), beside a run with the
    product configuration set, which keeps the products."""
    n = 700
    e = np.zeros((n, n), dtype=np.uint8)
    e[np.arange(n - 1), np.arange(1, n)] = 1
    ed = dev(e)
    announce("program long path")
    for tuned in (False, True):
        ctx = dl.Context()
        if tuned:
            ctx.set_tuning("i8", n, 1)
        prog = dl.Program(PATH, ctx=ctx)
        prog.bind("e", ed)
        prog.run(dl.DL_EVAL_ITERATION)
        _check(dl, prog, PATH, {"e": e}, n)
        assert prog.layers()[0]["iters"] == n
        prog.close()
        ctx.close()


def test_large_layer_by_lists_and_products(dl):
    """n = 5200, where fewer entries of a list are kept at hand: the layers by
    lists equal those by products (a configuration set by the caller)."""
    n = 5200
    e, f = (dev(dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 3 + i, self_loops=True))) for i in range(2))
    announce("program large layer")
    got = []
    for tuned in (False, True):
        ctx = dl.Context()
        if tuned:
            ctx.set_tuning("i8", n, 0)
        prog = dl.Program(CHAINED, ctx=ctx)
        prog.bind("e", e)
        prog.bind("f", f)
        prog.run(dl.DL_EVAL_ITERATION)
        got.append(([host(prog.fetch(k, n=n)[0]) for k in "pq"], [layer["iters"] for layer in prog.layers()]))
        prog.close()
        ctx.close()
    assert got[0][1] == got[1][1]
    assert all(np.array_equal(a, b) for a, b in zip(got[0][0], got[1][0]))
