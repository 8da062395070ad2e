"""The one-launch squaring closure on bits (int8, n <= 2048): models, per-step
sizes and iteration counts against the oracle, exactly, at the edges of its
64 x 64 tiles and of its range, for the longest paths, cut-off step counts,
odd strides and alignments, and against the product kernels (a configuration
set by the caller keeps those)."""
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


def _square_iters(a):
    """Model, per-step sizes and iterations of the squaring series (numpy)."""
    r = np.zeros_like(a, dtype=bool)
    ab = a != 0
    ones = [0]
    while True:
        rf = r.astype(np.float32)
        nxt = ab | (rf @ rf > 0) if len(ones) > 1 else ab.copy()
        ones.append(int(nxt.sum()))
        r = nxt
        if ones[-1] == ones[-2]:
            return r.astype(np.uint8), ones, len(ones) - 1


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 300, 511, 512, 513, 960, 1024, 1025, 1500,
                               1984, 1985, 2047, 2048])
def test_sizes(dl, n):
    for seed, deg in ((0, 1.0), (1, 3.0)):
        a = dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, deg / n), 31 * n + seed, self_loops=True))
        want, ones, iters = _square_iters(a)
        announce("bits", n, seed)
        r, it = dl.dl_tc(dev(a))
        assert np.array_equal(host(r), want) and it == iters
        assert np.array_equal(want, oracle.tc_seminaive(a)[0])
        st = dl.dl_tc_steps(dev(a), 40)
        assert st.converged and st.ones == ones and np.array_equal(host(st.R), want)


@pytest.mark.parametrize("n", [64, 200, 1025, 2048])
def test_steps_cut_off(dl, n):
    """A path, whose series is the longest: every cut-off step count."""
    a = np.zeros((n, n), dtype=np.uint8)
    a[np.arange(n - 1), np.arange(1, n)] = 1
    ad = dev(a)
    want, ones, iters = _square_iters(a)
    for k in range(0, iters + 2):
        announce("bits path", n, k)
        st = dl.dl_tc_steps(ad, k)
        assert st.steps == min(k, iters) and st.converged == (k >= iters)
        assert st.ones == ones[:st.steps + 1]
        dist = 2 ** max(0, st.steps - 1) if st.steps else 0
        i, j = np.indices((n, n))
        assert np.array_equal(host(st.R), ((j > i) & (j - i <= dist)).astype(np.uint8))


@pytest.mark.parametrize("kind", ["empty", "complete", "identity", "cycle"])
@pytest.mark.parametrize("n", [1, 64, 130])
def test_special(dl, kind, n):
    a = np.zeros((n, n), dtype=np.uint8)
    if kind == "complete":
        a[:] = 200  # any nonzero byte is true
    elif kind == "identity":
        np.fill_diagonal(a, 1)
    elif kind == "cycle":
        a[np.arange(n), (np.arange(n) + 1) % n] = 128
    want, _, iters = _square_iters(a)
    announce("bits special", kind, n)
    r, it = dl.dl_tc(dev(a))
    assert np.array_equal(host(r), want) and it == iters


@pytest.mark.parametrize("off", [0, 1, 3, 16])
def test_strides_and_alignment(dl, off):
    import torch

    n = 333
    a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, off))
    big = torch.full((n, 400), 9, dtype=torch.uint8, device="cuda")
    big[:, off:off + n] = dev(a)
    out = torch.full((n, 421), 5, dtype=torch.uint8, device="cuda")
    announce("bits strides", off)
    r, _ = dl.dl_tc(big[:, off:off + n], out=out[:, off:off + n])
    got = host(out)
    assert np.array_equal(got[:, off:off + n], oracle.tc_seminaive(a)[0])
    assert np.all(got[:, :off] == 5) and np.all(got[:, off + n:] == 5)


def test_against_the_product_kernels(dl):
    """The same relations through the product kernels, chosen by the caller."""
    ctx = dl.Context()
    for n in (256, 700, 1024, 2048):
        a = dev(dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, n)))
        announce("bits and products", n)
        r, it = dl.dl_tc(a, ctx=ctx)
        ctx.set_tuning("i8", n, 2)
        r2, it2 = dl.dl_tc(a, ctx=ctx)
        ctx.set_tuning("i8", n, -1)
        rs, its = dl.dl_tc_batch([a, a.t().contiguous(), a], ctx=ctx)
        assert it == it2 == its[0] == its[1] == its[2]
        assert bool((r == r2).all()) and bool((rs[0] == r).all()) and bool((rs[1] == r.t()).all())
    ctx.close()


def test_many_calls_and_streams(dl):
    """Back-to-back calls on two streams and contexts: the counters of one
    launch are left clean for the next."""
    import torch

    n = 500
    rels = [dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, s)) for s in range(4)]
    want = [oracle.tc_seminaive(a)[0] for a in rels]
    ctxs = [dl.Context() for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    devs = [dev(a) for a in rels]
    torch.cuda.synchronize()
    announce("bits streams")
    for k in range(40):
        r, _ = dl.dl_tc(devs[k % 4], ctx=ctxs[k % 2], stream=streams[k % 2])
        streams[k % 2].synchronize()
        assert np.array_equal(host(r), want[k % 4])
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("off", [0, 1, 2, 7, 13])
@pytest.mark.parametrize("prec", ["i8", "f32", "bf16", "fp8", "fp4"])
def test_unaligned_rows_in_and_out(dl, off, prec):
    """Ingest, emit and the row norm at every alignment of the caller's rows,
    with sizes that end inside a 16-byte segment; bytes around are untouched."""
    import torch

    for n in (17, 250):
        a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, off)) * 255
        big = torch.full((n + 1, n + 37), 3, dtype=torch.uint8, device="cuda")
        big[:n, off:off + n] = dev(a)
        out = torch.full((n + 1, n + 29), 6, dtype=torch.uint8, device="cuda")
        view, want = big[:n, off:off + n], oracle.tc_seminaive(a)[0]
        ctx = dl.Context()
        ctx.set_tuning(prec, n, 2)  # the product kernels
        announce("unaligned", n, off, prec)
        r, _ = dl.dl_tc(view, prec=prec, out=out[:n, off:off + n], ctx=ctx)
        got = host(out)
        assert np.array_equal(got[:n, off:off + n], want)
        got[:n, off:off + n] = 6
        assert np.all(got == 6)
        bound = dl.dl_eps_bound(view, ctx=ctx)
        assert bound == 1.0 / (1.0 + int((a != 0).sum(axis=1).max()))
        ctx.close()


@pytest.mark.parametrize("n", [33, 300, 1001, 1024, 2047])
def test_result_is_seen_by_other_streams(dl, n):
    """The one-launch closures return once their result is stored: a copy on
    a stream of its own, made right after the call, sees it, at every offset
    of the rows within a word (squaring in int8; the plain series in fp32)."""
    import torch

    a = dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, 2.0 / n), 7 * n, self_loops=True))
    want = oracle.tc_seminaive(a)[0]
    ad = dev(a)
    side = torch.cuda.Stream()
    calls = [lambda out: dl.dl_tc(ad, out=out)]
    if n <= 512:
        calls.append(lambda out: dl.dl_tc(ad, dl.DL_TC_PLAIN, dl.DL_F32, out=out))
    for off in range(4):
        for call in calls:
            announce("streams", n, off)
            flat = torch.full((n * (n + off) + 4,), 9, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            out = flat[off : off + n * (n + off)].view(n, n + off)[:, :n]
            call(out)
            with torch.cuda.stream(side):
                got = out.clone()
            side.synchronize()
            assert np.array_equal(got.cpu().numpy(), want)
            flat = flat.cpu().numpy()
            pad = flat[off : off + n * (n + off)].reshape(n, n + off)[:, n:]
            assert (pad == 9).all() and (flat[:off] == 9).all() and (flat[off + n * (n + off) :] == 9).all()


def test_one_launch_closures_on_a_busy_chip(dl):
    """Four threads with a context and a stream each run the one-launch
    closures (both kinds) while products on a fifth stream keep the chip busy:
    whether a launch finds its workgroups room together or the series is run
    by product launches, every model and iteration count is right."""
    import threading

    import torch

    cases = []
    for n, method, prec in ((700, dl.DL_TC_SQUARE, dl.DL_I8), (400, dl.DL_TC_PLAIN, dl.DL_F32),
                            (2000, dl.DL_TC_SQUARE, dl.DL_I8), (512, dl.DL_TC_PLAIN, dl.DL_I8)):
        a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 9 * n))
        ad = dev(a)
        want, iters = dl.dl_tc(ad, method, prec)
        assert np.array_equal(host(want), oracle.tc_seminaive(a)[0])
        cases.append((ad, method, prec, host(want), iters))
    wrong = []

    def work(case):
        ad, method, prec, want, iters = case
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = dl.Context()
            out = torch.empty_like(ad)
            for k in range(25):
                announce("busy chip", ad.shape[0], k)
                try:
                    _, it = dl.dl_tc(ad, method, prec, out=out, ctx=ctx)
                except dl.DLError as err:
                    wrong.append((ad.shape[0], k, str(err)))
                    continue
                if it != iters or not np.array_equal(out.cpu().numpy(), want):
                    wrong.append((ad.shape[0], k, it))
            ctx.close()

    torch.cuda.synchronize()
    busy = torch.cuda.Stream()
    threads = [threading.Thread(target=work, args=(c,)) for c in cases]
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
