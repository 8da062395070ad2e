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
