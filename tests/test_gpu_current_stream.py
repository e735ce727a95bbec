"""Calls go to the caller's current stream: its handle as the binding takes it, with torch's short way to it and without."""
import threading

import pytest
import torch

from paper_2509_17396_amd import binding as ep

pytestmark = pytest.mark.gpu


def both():
    return ep._stream().value or 0, torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("short", [True, False])
def test_the_handle_is_the_current_streams(short, monkeypatch):
    if short:
        assert ep._raw_stream is not None
    else:
        monkeypatch.setattr(ep, "_raw_stream", None)
    outside = both()
    assert outside[0] == outside[1]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    handles = []
    for s in (a, b):
        with torch.cuda.stream(s):
            handles.append(both())
            assert handles[-1] == (s.cuda_stream, s.cuda_stream)
    assert handles[0] != handles[1] and outside not in handles
    assert both() == outside
    with torch.cuda.stream(a):   # the current stream is the thread's own
        other = []
        t = threading.Thread(target=lambda: other.append(both()))
        t.start()
        t.join()
        assert other == [outside]
        assert both() == handles[0]
