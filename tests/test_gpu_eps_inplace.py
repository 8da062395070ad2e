"""The closure's epsilon form through the in-place inverse, at the sizes where
its pieces change: one pivot block, several, the last size inverted in blocks
of 128 directly, and the first one in panels of 512 with a shorter last panel.

Values: every operation of the elimination adds terms of one sign, so each
entry is computed with a relative error of a few Np units of roundoff; the
reference is the series sum_k (eps A)^k, whose terms are non-negative too.
Bound used: 8 Np u, u = 2^-53."""
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


def _series(a, eps):
    """sum_{k >= 1} (eps A)^k by doubling, in fp64 on the CPU."""
    import torch

    m = torch.from_numpy(a.astype(np.float64)) * eps
    x = m.clone()
    for _ in range(40):
        y = x + m @ x
        m = m @ m
        if bool((y == x).all()):
            break
        x = y
    return x.numpy()


@pytest.mark.parametrize("n", [2, 127, 128, 200, 513, 1100, 2048, 2049, 2600])
def test_values_and_model(dl, n):
    a = dlgen.to_dense(n, dlgen.er_edges(n, min(1.0, 3.0 / n), n, self_loops=True))
    eps = 0.5 * oracle.eps_bound(a)
    announce("eps in place", n)
    r, x, flag = dl.dl_solve_eps(dev(a), eps, want_x=True, underflow=True)
    want = _series(a, eps)
    xs = host(x)
    assert flag == 0
    np_ = (n + 127) // 128 * 128
    assert np.all(np.abs(xs - want) <= 8 * np_ * 2.0 ** -53 * want)  # zeros are exactly zero
    assert np.array_equal(host(r), (xs > 0).astype(np.uint8))
    assert np.array_equal(host(r), oracle.tc_seminaive(a)[0])


def test_strided_input_and_outputs(dl):
    """Row strides larger than n, and rows that start at odd addresses."""
    import torch

    n = 301
    a = dlgen.to_dense(n, dlgen.er_edges(n, 3.0 / n, 5, self_loops=True))
    big = torch.full((n, 333), 7, dtype=torch.uint8, device="cuda")
    big[:, 1:1 + n] = dev(a)
    out = torch.zeros((n, 400), dtype=torch.uint8, device="cuda")
    eps = oracle.eps_bound(a)
    announce("eps in place strided")
    r, x = dl.dl_solve_eps(big[:, 1:1 + n], eps, want_x=True, out=out[:, 3:3 + n])
    r0, x0 = dl.dl_solve_eps(dev(a), eps, want_x=True)
    assert np.array_equal(host(r), host(r0)) and np.array_equal(host(x), host(x0))
    assert int(out[:, :3].sum()) == 0 and int(out[:, 3 + n:].sum()) == 0


@pytest.mark.parametrize("n", [100, 700])
def test_shared_relation_in_the_linear_form(dl, n):
    """dl_solve_linear with B and C the same tensor is the closure's equation;
    with C a copy it takes the general elimination: the same model, values
    within the rounding of both."""
    a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 3))
    ad = dev(a)
    eps = 0.5 * oracle.eps_bound(a)
    announce("linear shared", n)
    r1, x1 = dl.dl_solve_linear(ad, ad, eps, want_x=True)
    r2, x2 = dl.dl_solve_linear(ad, ad.clone(), eps, want_x=True)
    assert np.array_equal(host(r1), host(r2))
    np_ = (n + 127) // 128 * 128
    assert np.all(np.abs(host(x1) - host(x2)) <= 16 * np_ * 2.0 ** -53 * host(x2))
