"""The doubling of the Stein equations at the sizes where its product kernels
change tiles (32 x 64, 64 x 64, 128 x 128 and, for the symmetric increment,
the upper triangle of each), for one doubling, many, and none needed.

Values: every term is non-negative, so X is computed with a relative error of
a few Np units of roundoff per doubling; the reference iterates the equation
in fp64.  Bound used: 8 Np d u for d doublings, u = 2^-53."""
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


def _fixpoint(q, b, c, eps):
    """x = eps (q + b x c) iterated on the device in fp64 (plain torch)."""
    import torch

    q, b, c = (torch.from_numpy(m.astype(np.float64)).cuda() for m in (q, b, c))
    x = eps * q
    for _ in range(4000):
        y = eps * (q + b @ x @ c)
        if bool(((y - x).abs() <= 1e-17 * y.abs()).all()):
            return y.cpu().numpy()
        x = y
    raise AssertionError("reference did not settle")


@pytest.mark.parametrize("n", [3, 128, 130, 1000, 1100, 1408, 2048, 2500, 3072])
def test_same_generation(dl, n):
    p = dlgen.to_dense(n, dlgen.forest_edges(n, n))
    d = int(p.sum(axis=1).max())
    eps = 1.0 / (1 + d * d)
    announce("stein sg", n)
    s, x, k = dl.dl_sg_eps(dev(p), eps, want_x=True)
    s2, _, k2 = dl.dl_sg_eps(dev(p), eps)
    xs = host(x)
    want = _fixpoint(np.eye(n), p, p.T, eps)
    np_ = (n + 127) // 128 * 128
    assert np.all(np.abs(xs - want) <= 8 * np_ * max(k, 1) * 2.0 ** -53 * want)
    assert np.array_equal(xs, xs.T)
    assert np.array_equal(host(s), (xs > 0).astype(np.uint8))
    assert np.array_equal(host(s), host(s2)) and 1 <= k2 <= k
    assert np.array_equal(host(s), oracle.sg_seminaive(p)[0])


@pytest.mark.parametrize("n", [2, 128, 300, 700, 1200, 2048])
def test_two_sided(dl, n):
    q, b, c = (dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, 2.0 / n), 7 * n + k)) for k in range(3))
    eps = 0.5 / (1 + int(b.sum(axis=1).max()) * int(c.sum(axis=0).max()))
    announce("stein two-sided", n)
    r, x, k = dl.dl_solve_two_sided(dev(q), dev(b), dev(c), eps, want_x=True)
    r2, _, k2 = dl.dl_solve_two_sided(dev(q), dev(b), dev(c), eps)
    want = _fixpoint(q, b, c, eps)
    np_ = (n + 127) // 128 * 128
    xs = host(x)
    assert np.all(np.abs(xs - want) <= 8 * np_ * max(k, 1) * 2.0 ** -53 * want)
    assert np.array_equal(host(r), (xs > 0).astype(np.uint8)) and np.array_equal(host(r), host(r2)) and k2 <= k


@pytest.mark.parametrize("n", [5, 200])
def test_nothing_to_add(dl, n):
    """Empty relations: the first doubling confirms X_0."""
    z = np.zeros((n, n), dtype=np.uint8)
    q = dlgen.to_dense(n, dlgen.er_edges(n, 0.3, 1))
    announce("stein empty", n)
    s, x, k = dl.dl_sg_eps(dev(z), 0.75, want_x=True)
    assert k == 1 and np.array_equal(host(x), 0.75 * np.eye(n)) and np.array_equal(host(s), np.eye(n, dtype=np.uint8))
    r, x, k = dl.dl_solve_two_sided(dev(q), dev(z), dev(z), 0.5, want_x=True)
    assert k == 1 and np.array_equal(host(x), 0.5 * q) and np.array_equal(host(r), q)
    r, _, k = dl.dl_solve_two_sided(dev(z), dev(q), dev(q), 0.5 / (1 + n * n))
    assert k == 1 and not host(r).any()


def test_long_walks_take_several_groups(dl):
    """A path of 200 constants: the pattern needs 2^k > 200 walks, more
    doublings than one group of launches holds."""
    n = 200
    p = np.zeros((n, n), dtype=np.uint8)
    p[np.arange(1, n), np.arange(n - 1)] = 1
    q = np.zeros((n, n), dtype=np.uint8)
    q[0, 0] = 1
    announce("stein path")
    # X = eps (Q + P X P^T): X_kk = eps^(k+1)
    r, _, k = dl.dl_solve_two_sided(dev(q), dev(p), dev(np.ascontiguousarray(p.T)), 0.5)
    assert np.array_equal(host(r), np.eye(n, dtype=np.uint8)) and k == 9


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000])
def test_column_norm_bound(dl, n):
    """The two-sided eps bound 1 / (1 + ||C||_1 ||B||_inf) is exact at every
    width: eps at the bound is accepted, above it refused."""
    c = dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, 5.0 / n), 2, self_loops=True))
    c[:, n - 1] = 1  # the largest column is the last one
    c *= 255  # any nonzero byte is true
    b = np.eye(n, dtype=np.uint8)
    z = np.zeros((n, n), dtype=np.uint8)
    announce("col norm", n)
    dl.dl_solve_two_sided(dev(z), dev(b), dev(c), 1.0 / (1 + n))
    with pytest.raises(dl.DLError):
        dl.dl_solve_two_sided(dev(z), dev(b), dev(c), 1.0 / (1 + n) * 1.001)


@pytest.mark.parametrize("n", [1930, 2100, 2250, 2688, 3500])
def test_split_products_same_generation(dl, n):
    """Sizes whose last pass of tiles is shared between owners and helpers
    (about half and nearly all of the slots in use; 3500 after a full pass):
    the equation's solution, and bit for bit the same one every time."""
    p = dlgen.to_dense(n, dlgen.forest_edges(n, 3 * n))
    d = int(p.sum(axis=1).max())
    eps = 1.0 / (1 + d * d)
    announce("stein split sg", n)
    s, x, k = dl.dl_sg_eps(dev(p), eps, want_x=True)
    xs = host(x)
    want = _fixpoint(np.eye(n), p, p.T, eps)
    np_ = (n + 127) // 128 * 128
    assert np.all(np.abs(xs - want) <= 8 * np_ * max(k, 1) * 2.0 ** -53 * want)
    assert np.array_equal(xs, xs.T) and np.array_equal(host(s), (xs > 0).astype(np.uint8))
    for _ in range(3):
        assert np.array_equal(host(dl.dl_sg_eps(dev(p), eps, want_x=True)[1]), xs)


@pytest.mark.parametrize("n", [2100, 2560, 2688])
def test_split_products_two_sided(dl, n):
    q, b, c = (dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 5 * n + i)) for i in range(3))
    eps = 0.5 / (1 + int(b.sum(axis=1).max()) * int(c.sum(axis=0).max()))
    announce("stein split two-sided", n)
    r, x, k = dl.dl_solve_two_sided(dev(q), dev(b), dev(c), eps, want_x=True)
    xs = host(x)
    want = _fixpoint(q, b, c, eps)
    np_ = (n + 127) // 128 * 128
    assert np.all(np.abs(xs - want) <= 8 * np_ * max(k, 1) * 2.0 ** -53 * want)
    assert np.array_equal(host(r), (xs > 0).astype(np.uint8))
    assert np.array_equal(host(dl.dl_solve_two_sided(dev(q), dev(b), dev(c), eps, want_x=True)[1]), xs)
