"""Which kernels serve a call, from the profiler's trace: the models are the
same on every route, so only the trace tells whether a size or a relation took
the one meant for it."""
from __future__ import annotations

import numpy as np
import pytest

import dlgen
import oracle
from tests.gpu_routes import base, kernels
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu


@pytest.fixture(scope="module")
def dl():
    import paper_1608_00139_amd as m

    m.load()
    return m


def _sparse(n, seed, degree=2.0):
    return dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, degree / n), seed, self_loops=True))


@pytest.mark.parametrize("n,count,one", [(1920, 1, True), (1921, 1, False), (1728, 2, True), (1729, 2, False),
                                         (1, 3, True)])
def test_squaring_on_bits(dl, n, count, one):
    rels = [_sparse(n, n + k) for k in range(count)]
    devs = [dev(a) for a in rels]
    got = []
    announce("route squaring", n, count)
    if count == 1:
        names = base(kernels(lambda: got.append(dl.dl_tc(devs[0])[0])))
    else:
        names = base(kernels(lambda: got.extend(dl.dl_tc_batch(devs)[0])))
    assert names == ["k_fix_bits"] * count if one else "k_nt_dma" in names and "k_fix_bits" not in names, names
    for r, a in zip(got, rels):
        assert np.array_equal(host(r), oracle.tc_seminaive(a)[0])


LISTS = ["k_row_lists", "k_sg_lists"]


def _rows_of(n, entries, seed):
    """Exactly `entries` true entries in every row."""
    rng = np.random.default_rng(seed)
    a = np.zeros((n, n), dtype=np.uint8)
    for r in a:
        r[rng.permutation(n)[:entries]] = 1
    return a


@pytest.mark.parametrize("n,entries,prec,lists", [(1, 1, "i8", True), (64, 32, "i8", True), (300, 32, "i8", True),
                                                  (300, 33, "i8", False), (300, 2, "fp8", False)])
def test_same_generation(dl, n, entries, prec, lists):
    a = _rows_of(n, entries, n + entries)
    got = []
    announce("route sg", n, entries, prec)
    names = base(kernels(lambda: got.extend(dl.dl_sg(dev(a), prec=prec))))
    assert (names == LISTS) if lists else ("k_nt_dma" in names or "k_nt_small" in names), names
    ref, _, iters, _ = oracle.sg_seminaive(a)
    assert got[1] == iters and np.array_equal(host(got[0]), ref)


def test_same_generation_set_and_timed(dl):
    """A configuration set by the caller and kernel timing keep the products."""
    a = dev(_sparse(300, 5, 1.0))
    ctx = dl.Context()
    want, iters = dl.dl_sg(a, ctx=ctx)
    ctx.set_tuning("i8", 300, 2)
    announce("route sg set")
    got = []
    assert "k_nt_dma" in base(kernels(lambda: got.extend(dl.dl_sg(a, ctx=ctx))))
    ctx.set_tuning("i8", 300, -1)
    ctx.set_timing(True)
    assert "k_ingest" in base(kernels(lambda: got.extend(dl.dl_sg(a, ctx=ctx))))
    ctx.set_timing(False)
    assert base(kernels(lambda: got.extend(dl.dl_sg(a, ctx=ctx)))) == LISTS
    for k in (0, 2, 4):
        assert got[k + 1] == iters and bool((got[k] == want).all())
    ctx.close()


def _two_chains(depth):
    """A root with two chains of `depth` nodes: node 1 + k and node 1 + depth +
    k at depth k + 1, and no others, are of one generation."""
    n = 2 * depth + 1
    p = np.zeros((n, n), dtype=np.uint8)
    for first in (1, 1 + depth):
        p[first, 0] = 1
        k = np.arange(1, depth)
        p[first + k, first + k - 1] = 1
    return p


@pytest.mark.parametrize("depth,lists", [(4093, True), (4094, False)])
def test_same_generation_of_many_steps(dl, depth, lists):
    """Step t adds the pairs of depth t - 1, so the series repeats at depth + 2:
    the longest one that the ring of model sizes holds, and one step more,
    which runs out of it and is run again by products."""
    import torch

    p = _two_chains(depth)
    n = len(p)
    got = []
    announce("sg steps", depth)
    names = base(kernels(lambda: got.append(dl.dl_sg_steps(dev(p), 6000, prec="i8"))))
    assert (names == LISTS) if lists else (names[:2] == LISTS and "k_nt_dma_sk" in names), names[:5]
    r = got[0]
    assert r.converged and r.steps == depth + 2
    assert r.ones == [0] + [n + 2 * min(t - 1, depth) for t in range(1, depth + 3)]
    want = torch.eye(n, dtype=torch.uint8, device="cuda")
    i = torch.arange(1, 1 + depth, device="cuda")
    want[i, i + depth] = 1
    want[i + depth, i] = 1
    assert bool((r.R == want).all())


@pytest.mark.parametrize("n,prec,names", [(512, "i8", ["k_fix_small"]), (512, "f32", ["k_fix_small"]),
                                          (513, "i8", ["k_row_lists", "k_layer_lists"]),
                                          (5121, "i8", ["k_row_lists", "k_layer_lists"]), (513, "f32", None),
                                          (8193, "i8", None)])
def test_plain_closure(dl, n, prec, names):
    a = _sparse(n, n, 1.0 if n < 6000 else 0.3)
    got = []
    announce("route plain", n, prec)
    ran = base(kernels(lambda: got.extend(dl.dl_tc(dev(a), dl.DL_TC_PLAIN, prec))))
    assert ran == names if names else "k_nt_dma" in ran and "k_layer_lists" not in ran, ran
    ref, _, iters, _ = oracle.tc_seminaive(a)
    assert got[1] == iters and np.array_equal(host(got[0]), ref)


def test_plain_closure_with_sizes(dl):
    """Sizes per step are the products' alone."""
    a = _sparse(600, 8)
    got = []
    announce("route plain steps")
    ran = base(kernels(lambda: got.append(dl.dl_tc_steps(dev(a), 700, dl.DL_TC_PLAIN, "i8"))))
    assert "k_layer_lists" not in ran and "k_nt_dma" in ran
    ref, ones, iters, _ = oracle.tc_seminaive(a)
    assert got[0].steps == iters and got[0].ones == list(ones[: iters + 1]) and np.array_equal(host(got[0].R), ref)


@pytest.mark.parametrize("rule,lists", [("tc(X,Y) :- e(X,Z), tc(Z,Y).", True), ("tc(X,Y) :- tc(X,Z), e(Z,Y).", True),
                                        ("tc(X,Y) :- tc(X,Z), tc2(Z,Y).\ntc2(X,Y) :- e(X,Y).", True),
                                        ("tc(X,Y) :- e(X,Z), tc(W,Z), e(W,Y).", False)])
def test_program_layer(dl, rule, lists):
    from oracle import program as oprog

    n = 300
    a = _sparse(n, 11, 1.5)
    text = "tc(X,Y) :- e(X,Y).\n" + rule + "\n"
    p = dl.Program(text)
    p.bind("e", dev(a))
    announce("route program", rule)
    ran = base(kernels(lambda: p.run(dl.DL_EVAL_ITERATION)))
    assert ("k_layer_lists" in ran) == lists and (lists or "k_nt_dma" in ran), ran
    want, _ = oprog.evaluate(text, {"e": a}, n)
    assert np.array_equal(host(p.fetch("tc")[0]), want["tc"])
    p.close()


# ----------------------------------------------------------------- products that the lists pass by
def test_symmetric_stream_k_product_n8192(dl):
    """The stream-K S' product at N = 8192 (528 upper-triangle tiles, tiles
    split over two workgroups) by a configuration set for it."""
    n = 8192
    p = dlgen.to_dense(n, dlgen.forest_edges(n, 2))
    ctx = dl.Context()
    ctx.set_tuning("i8", n, 0)
    got = []
    announce("stream-k n8192")
    assert "k_nt_dma_sk" in base(kernels(lambda: got.extend(dl.dl_sg(dev(p), ctx=ctx))))
    ref, _, iters, _ = oracle.sg_seminaive(p)
    assert got[1] == iters and np.array_equal(host(got[0]), ref)
    ctx.close()


@pytest.mark.parametrize("cfg", [2, 4])
def test_iterate_in_the_output(dl, cfg):
    """n = 256 without padding: the caller's matrix is an iterate buffer of the
    product series, at every number of steps, and nothing is copied into it."""
    n = 256
    p = dlgen.to_dense(n, dlgen.forest_edges(n, 4))
    _, ones, iters, _ = oracle.sg_seminaive(p)
    ctx = dl.Context()
    ctx.set_tuning("i8", n, cfg)
    got = []
    for k in range(0, iters + 2):
        announce("sg in place", cfg, k)
        names = base(kernels(lambda: got.append(dl.dl_sg_steps(dev(p), k, prec="i8", ctx=ctx))))
        r = got[-1]
        assert np.array_equal(host(r.R), oracle.sg_seminaive(p, maxsteps=k)[0]), k
        assert r.steps == min(k, iters) and r.ones == list(ones[: r.steps + 1])
        if k >= iters or (k >= 2 and k % 2 == 0):
            assert "k_emit" not in names, k
    ctx.close()
