"""The binding's workspace: a buffer that the caller drops or replaces is given back,
and a replaced one has its streams recorded anew."""
import weakref

import pytest
import torch

import paper_2606_11660_amd as P

pytestmark = pytest.mark.gpu


def test_a_dropped_buffer_is_given_back():
    ws = P.Workspace("cuda")
    ws.get(1 << 20)
    held = weakref.ref(ws.buf)
    ws.buf = None
    assert held() is None
    ptr, size = ws.get(1 << 10)
    assert size == 1 << 10 and ptr == ws.buf.data_ptr()


def test_streams_are_recorded_once_per_buffer(monkeypatch):
    seen = []
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: seen.append((t.data_ptr(), s.cuda_stream)))
    ws, side = P.Workspace("cuda"), torch.cuda.Stream()
    main = torch.cuda.current_stream().cuda_stream
    for _ in range(2):
        ws.get(1 << 10)
        ws.get(1 << 10, side)
    first = ws.buf.data_ptr()
    assert seen == [(first, main), (first, side.cuda_stream)]
    mine = torch.empty(1 << 12, dtype=torch.uint8, device="cuda")
    ws.buf = mine
    ws.get(1 << 11, side)
    assert seen[2:] == [(mine.data_ptr(), side.cuda_stream)]
    ws.get(1 << 13, side)  # grown
    assert seen[3:] == [(ws.buf.data_ptr(), side.cuda_stream)]
