"""Relations with a row too long for lists: the launch that would have run the
series by lists writes the first operands of its products instead.  Sizes
around the tiles and units of that pass (32 rows or columns, units of 128
columns by a quarter of the padded rows), strides and offsets of the caller's
rows, bytes other than 1, and batches in which such a relation comes first or
later; models, iteration counts and sizes per step against the oracle."""
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


def _dense(n, p, seed, row):
    """Few entries a row, but for one of more than 32."""
    a = dlgen.to_dense(n, dlgen.er_edges(n, p / n, seed, self_loops=True))
    rng = np.random.default_rng(seed)
    a[row, rng.permutation(n)[: max(33, n // 5)]] = 1
    return a


def _placed(a, off):
    """`a` inside a larger device matrix, `off` bytes into its rows, true as 7."""
    import torch

    n = len(a)
    big = torch.full((n + 1, n + 21), 3, dtype=torch.uint8, device="cuda")
    big[:n, off : off + n] = dev(a * 7)
    return big[:n, off : off + n]


@pytest.mark.parametrize("n,off", [(33, 0), (64, 1), (255, 3), (256, 0), (257, 5), (300, 2), (513, 0), (1000, 7),
                                   (1024, 0), (1025, 1), (2049, 4)])
def test_same_generation(dl, n, off):
    for row in (0, n - 1):
        a = _dense(n, 1.0, n + row, row)
        ref, ones, iters, _ = oracle.sg_seminaive(a)
        p = _placed(a, off)
        announce("sg dense start", n, off, row)
        got = kernels(lambda: dl.dl_sg(p))
        assert "k_sg_lists" in got and not {"k_ingest", "k_identity"} & set(base(got))
        s, it = dl.dl_sg(p)
        assert it == iters and np.array_equal(host(s), ref)
        for k in (2, 3, iters + 1):
            r = dl.dl_sg_steps(p, k, prec="i8")
            assert r.steps == min(k, iters) and r.ones == list(ones[: r.steps + 1])
            assert np.array_equal(host(r.R), oracle.sg_seminaive(a, maxsteps=k)[0])


@pytest.mark.parametrize("n,off", [(513, 0), (600, 1), (767, 2), (768, 0), (769, 3), (1000, 5), (1023, 0), (1025, 7),
                                   (2049, 0), (4097, 2)])
def test_plain_closure(dl, n, off):
    for row in (0, n - 1):
        a = _dense(n, 1.0 if n < 3000 else 0.5, 3 * n + row, row)
        ref, _, iters, _ = oracle.tc_seminaive(a)
        p = _placed(a, off)
        announce("plain dense start", n, off, row)
        got = base(kernels(lambda: dl.dl_tc(p, dl.DL_TC_PLAIN, "i8")))
        assert "k_layer_lists" in got and not {"k_ingest", "k_ring_clear"} & set(got)
        r, it = dl.dl_tc(p, dl.DL_TC_PLAIN, "i8")
        assert it == iters and np.array_equal(host(r), ref)


@pytest.mark.parametrize("order", ["dsd", "sdd", "dd", "ssd"])
def test_batches(dl, order):
    """d: a row too long, s: none; the workspace of a context's first batch
    moves between the lists and the products, a second batch's does not."""
    n = 700
    rels = [_dense(n, 1.0, 10 + i, i) if c == "d" else dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 20 + i))
            for i, c in enumerate(order)]
    want = [oracle.tc_seminaive(a) for a in rels]
    ctx = dl.Context()
    for turn in range(2):
        announce("dense start batch", order, turn)
        rs, its = dl.dl_tc_batch([dev(a) for a in rels], method=dl.DL_TC_PLAIN, prec="i8", ctx=ctx)
        for r, it, w in zip(rs, its, want):
            assert it == w[2] and np.array_equal(host(r), w[0])
    ctx.close()


def test_large_same_generation(dl):
    """n = 4096: S' by the stream-K product, whose tile counters the list
    launch clears; twice, the second time in a workspace that holds others."""
    n = 4096
    ctx = dl.Context()
    for seed in (1, 2):
        a = _dense(n, 0.5, seed, 17 * seed)
        announce("sg dense start", n, seed)
        s, it = dl.dl_sg(dev(a), ctx=ctx)
        ref, _, iters, _ = oracle.sg_seminaive(a)
        assert it == iters and np.array_equal(host(s), ref)
        dl.dl_tc(dev(np.ones((2500, 2500), dtype=np.uint8)), prec="fp8", ctx=ctx)
    ctx.close()
