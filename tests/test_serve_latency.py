"""When run_stream says a request finished, on the CPU with a stand-in batch and
events: with look-ahead the models are written while the loop goes on, and a
completion is timed when its model has been written, not when the loop next
runs a round."""
from __future__ import annotations

import time
from dataclasses import dataclass
from types import SimpleNamespace

import pytest
import torch

from paper_1608_00139_amd import serve
from tests.test_serve_host import StandInBulkBatch

WRITE = 0.002  # seconds from the fetch to the written model


class _Event:
    def record(self, stream=None):
        self.at = time.perf_counter() + WRITE

    def query(self):
        return time.perf_counter() >= self.at

    def synchronize(self):
        while not self.query():
            pass


class _Batch(StandInBulkBatch):
    stream = None

    def __init__(self, lookahead):
        super().__init__(slots=8, pool_bytes=1 << 30)
        self.lookahead = lookahead

    def dl_batch_fetch_n(self, slots, outs):
        assert len(slots) == len(outs)
        return [self.dl_batch_fetch(s) for s in slots]


@dataclass
class _Request:
    rid: int
    n: int
    arrival: float
    kind: str = "tc"


@pytest.mark.parametrize("lookahead", [0, 1])
def test_finished_before_an_idle_gap(monkeypatch, lookahead):
    """The only request running finishes and the next arrives much later."""
    cuda = SimpleNamespace(Event=_Event, current_stream=lambda: None, is_available=lambda: False)
    monkeypatch.setattr(serve, "torch", SimpleNamespace(
        int32=torch.int32, uint8=torch.uint8, cuda=cuda,
        empty=lambda shape, dtype, device: torch.empty(shape, dtype=dtype)))
    edges = torch.zeros((0, 2), dtype=torch.int32)
    reqs = [_Request(0, 64, 0.0), _Request(1, 65, 0.3), _Request(2, 66, 0.6)]
    stats, results = serve.run_stream(reqs, lambda q: edges, 0, batch=_Batch(lookahead), keep_results=True)
    assert sorted(results) == [0, 1, 2]
    for c in stats.completions:
        assert WRITE <= c.finished - c.arrival < 0.1, (c.tag, c.finished - c.arrival)
