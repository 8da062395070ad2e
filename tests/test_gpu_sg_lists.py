"""Same generation by lists (int8, at most 32 entries a row): models,
per-step sizes and iteration counts against the oracle, exactly, at the edges
of its 32-row slices and of its list length, and with the products' route
beside it (another precision takes it)."""
from __future__ import annotations

import numpy as np
import pytest

import dlgen
import oracle
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu


@pytest.fixture(scope="module")
def dl():
    import paper_1608_00139_amd as m

    m.load()
    return m


def _check(dl, p, tag, caps=()):
    n = p.shape[0]
    want, ones, iters, _ = oracle.sg_seminaive(p)
    announce("sg lists", tag, n)
    s, it = dl.dl_sg(dev(p))
    assert it == iters and np.array_equal(host(s), want), (tag, n)
    for cap in (*caps, n + 2):
        st = dl.dl_sg_steps(dev(p), cap)
        assert st.steps == min(cap, iters) and st.ones == list(ones[: st.steps + 1]), (tag, n, cap)
        assert st.converged == (cap >= iters)
        assert int(host(st.R).sum()) == ones[st.steps], (tag, n, cap)


@pytest.mark.parametrize("n", [511, 512, 513, 543, 544, 545, 1000, 1024, 1025, 2047, 3000])
def test_forests(dl, n):
    _check(dl, dlgen.to_dense(n, dlgen.forest_edges(n, n)), "forest", (0, 1, 2, 3))


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 65, 200, 257])
def test_small(dl, n):
    """One slice, two, an odd number of them; a row in the middle that is too
    long for a list from n = 33 on."""
    p = dlgen.to_dense(n, dlgen.forest_edges(n, n))
    _check(dl, p, "small forest", (0, 1, 2, 3))
    p[n // 2] = 1
    _check(dl, p, "small, long row", (2,))


@pytest.mark.parametrize("n", [600, 1100])
def test_several_parents(dl, n):
    for deg in (0.3, 2.0, 5.0):
        _check(dl, dlgen.to_dense(n, dlgen.er_edges(n, deg / n, 11 * n, self_loops=True)), f"er {deg}", (2,))


@pytest.mark.parametrize("extra", [0, 1])
def test_longest_list(dl, extra):
    """A row of 32 entries takes lists, one of 33 the products; same model."""
    n = 700
    rng = np.random.default_rng(5)
    p = dlgen.to_dense(n, dlgen.forest_edges(n, 3))
    for row in (0, 31, 64, 699):
        p[row] = 0
        p[row, rng.choice(n, 32 + (extra if row == 699 else 0), replace=False)] = 1
    _check(dl, p, f"row of {32 + extra}", (2, 4))


def test_special_relations(dl):
    n = 640
    _check(dl, np.zeros((n, n), dtype=np.uint8), "empty", (1, 2))
    _check(dl, np.eye(n, dtype=np.uint8), "identity")
    star = np.zeros((n, n), dtype=np.uint8)
    star[:, 7] = 1
    _check(dl, star, "one parent for all")
    full = np.ones((n, n), dtype=np.uint8)
    _check(dl, full, "full")
    chain = np.zeros((n, n), dtype=np.uint8)  # a parent each, and two children a parent: the longest series
    chain[np.arange(1, n), (np.arange(1, n) - 1) // 2] = 1
    _check(dl, chain, "binary tree", (5,))
    ladder = np.zeros((n, n), dtype=np.uint8)  # two chains from one root: a step per level
    ladder[np.arange(2, n), np.arange(0, n - 2)] = 1
    ladder[1, 0] = 1
    _check(dl, ladder, "two chains", (7, 100))


def test_strides_values_and_alignment(dl):
    import torch

    n, extra = 777, 13
    p = dlgen.to_dense(n, dlgen.forest_edges(n, 21))
    want = oracle.sg_seminaive(p)[0]
    flat = torch.zeros(n * (n + extra) + 8, dtype=torch.uint8, device="cuda")
    for off in range(4):
        announce("sg lists strides", off)
        a = flat[off : off + n * (n + extra)].view(n, n + extra)[:, :n]
        a.copy_(dev(p * (3 + 60 * off)))  # any nonzero byte is an entry
        buf = torch.full((n * (n + 5) + 8,), 9, dtype=torch.uint8, device="cuda")
        out = buf[off : off + n * (n + 5)].view(n, n + 5)[:, :n]
        dl.dl_sg(a, out=out)
        assert np.array_equal(host(out.contiguous()), want)
        h = host(buf)
        rows = h[off : off + n * (n + 5)].reshape(n, n + 5)
        assert (rows[:, n:] == 9).all() and (h[:off] == 9).all() and (h[off + n * (n + 5) :] == 9).all()


@pytest.mark.parametrize("n,cfg", [(600, 2), (900, 1), (1500, 2), (2500, 1), (4096, 0)])
def test_against_products(dl, n, cfg):
    """The route by products (a tile configuration set for the size keeps it,
    and so does another precision) and the one by lists, step by step."""
    p = dev(dlgen.to_dense(n, dlgen.forest_edges(n, n + cfg)))
    announce("sg lists against products", n, cfg)
    ctx = dl.Context(0)
    ctx.set_tuning("i8", n, cfg)
    a = dl.dl_sg_steps(p, 60, prec="i8")
    for b in (dl.dl_sg_steps(p, 60, prec="i8", ctx=ctx), dl.dl_sg_steps(p, 60, prec="fp8")):
        assert a.converged and b.converged
        assert a.ones == b.ones and a.steps == b.steps and np.array_equal(host(a.R), host(b.R))
    ctx.close()


@pytest.mark.parametrize("n", [513, 543, 545, 1000, 1024, 2047, 5200])
def test_plain_closure_by_lists(dl, n):
    """dl_tc's plain int8 series, which takes the same lists (a word of 32
    columns a row): models and iteration counts against the oracle, and against
    the squaring series' model; a row of 33 entries, a path and an empty
    relation too."""
    import torch

    rng = np.random.default_rng(n)
    rels = {"er": dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 3 * n, self_loops=True))}
    if n <= 2047:
        rels["sparse"] = dlgen.to_dense(n, dlgen.er_edges(n, 0.8 / n, 4 * n))
        rels["empty"] = np.zeros((n, n), dtype=np.uint8)
        long_row = rels["sparse"].copy()
        long_row[n - 1] = 0
        long_row[n - 1, rng.choice(n, 33, replace=False)] = 1
        rels["row of 33"] = long_row
        several = rels["sparse"].copy()
        for row in range(0, n, 5):
            several[row] = 0
            several[row, rng.choice(n, row % 33, replace=False)] = 1
        rels["lists of 0 to 32"] = several
    if n <= 600:
        path = np.zeros((n, n), dtype=np.uint8)
        path[np.arange(n - 1), np.arange(1, n)] = 1
        rels["path"] = path
    for tag, a in rels.items():
        announce("plain lists", n, tag)
        want, _, iters, _ = oracle.tc_seminaive(a)
        off = n % 4
        flat = torch.full((off + n * (n + off) + 8,), 9, dtype=torch.uint8, device="cuda")
        out = flat[off : off + n * (n + off)].view(n, n + off)[:, :n]
        _, it = dl.dl_tc(dev(a * np.uint8(5)), method=dl.DL_TC_PLAIN, prec="i8", out=out)
        assert it == iters, (tag, it, iters)
        h = host(flat)
        rows = h[off : off + n * (n + off)].reshape(n, n + off)
        assert np.array_equal(rows[:, :n], want), tag
        assert (rows[:, n:] == 9).all() and (h[:off] == 9).all() and (h[off + n * (n + off) :] == 9).all()
