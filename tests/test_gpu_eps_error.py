"""How far the closure's epsilon form is from the exact values.

Every term of the elimination has one sign, so its errors are those of its
sums.  The reference is the equation X = eps (A + A X) itself, iterated in
80-bit arithmetic from the computed X until its own error (a factor below 0.8 an
iteration) is under that arithmetic's rounding.  The bounds are the errors, by
the same measure and on the same inputs, of the elimination on the augmented
matrix [I - eps A | eps A] with divisions and accumulators that start from the
subtrahend, which this one replaced: it has to be no further off."""
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


def _error(a, eps, x):
    """||x - X|| / ||X|| over all entries, X exact."""
    n = len(a)
    rows = [np.flatnonzero(r) for r in a]
    idx = np.full((n, max(1, max(map(len, rows)))), n)
    for i, r in enumerate(rows):
        idx[i, : len(r)] = r
    e = np.longdouble(eps)
    z = np.zeros((n + 1, n), dtype=np.longdouble)
    z[:n] = x
    b = (a != 0).astype(np.longdouble)
    for _ in range(40):
        s = b.copy()
        for k in range(idx.shape[1]):
            s += z[idx[:, k]]
        z[:n] = e * s
    d = (x - z[:n]).astype(np.float64)
    return float(np.sqrt((d * d).sum()) / np.sqrt((x * x).sum()))


# n, degree, fraction of the largest eps, bound
CASES = [
    (64, 2.0, 1.0, 1.746e-16),
    (128, 3.0, 1.0, 3.046e-16),
    (200, 60.0, 1.0, 4.761e-16),
    (300, 4.0, 0.5, 6.856e-16),
    (513, 3.0, 1.0, 6.632e-16),
    (1000, 10.0, 1.0, 1.319e-15),
    (1100, 20.0, 1.0, 1.351e-15),
    (2048, 4.0, 0.5, 3.370e-15),
    (2600, 4.0, 0.5, 2.902e-15),
]


@pytest.mark.parametrize("n,degree,part,bound", CASES)
def test_no_further_off(dl, n, degree, part, bound):
    a = dlgen.to_dense(n, dlgen.er_edges(n, degree / n, n + int(degree)))
    eps = part * oracle.eps_bound(a)
    announce("eps error", n, degree)
    _, x = dl.dl_solve_eps(dev(a), eps, want_x=True)[:2]
    got = _error(a, eps, host(x))
    print("error", n, degree, part, "%.3e" % got, "bound %.3e" % bound, flush=True)
    assert got <= bound
