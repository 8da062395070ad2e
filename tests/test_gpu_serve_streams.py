"""dl_batch_fetch_n returns before the models are written: their memory must not
go to another tensor until the stream that writes them has done so, whichever
stream the tensors belong to."""
from __future__ import annotations

import numpy as np
import pytest

import dlgen
import oracle
from tests.gpu_util import announce, dev, gpu, host

pytestmark = gpu


@pytest.mark.parametrize("own", [False, True])
def test_outputs_are_held_for_the_writing_stream(monkeypatch, own):
    """A batch with a stream of its own, and one on the stream current at the
    call; the outputs belong to the default stream."""
    import torch

    import paper_1608_00139_amd as dl

    n = 200
    a = dlgen.to_dense(n, dlgen.er_edges(n, 2.0 / n, 1))
    side = torch.cuda.Stream()
    out = torch.empty((n, n), dtype=torch.uint8, device="cuda")
    ad = dev(a)
    torch.cuda.synchronize()
    seen = []
    real = torch.Tensor.record_stream
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: (seen.append((t, s)), real(t, s))[1])
    announce("fetch stream", own)
    with torch.cuda.stream(side):
        b = dl.Batch(1 << 24, max_active=4, stream=side if own else None)
        slot = b.dl_batch_submit(dl.Batch.TC, ad, 5)
        for _ in range(20):
            b.dl_batch_step()
        assert b.dl_batch_poll()[0][:2] == (5, slot)
        b.dl_batch_fetch_n([slot], [out])
    assert any(t is out and s.cuda_stream == side.cuda_stream for t, s in seen)
    side.synchronize()
    assert np.array_equal(host(out), oracle.tc_seminaive(a)[0])
    b.close()
