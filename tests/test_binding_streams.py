"""The binding's way to the current stream, with stand-ins for torch's modules (no GPU)."""
from types import SimpleNamespace

import pytest

from paper_2506_03700_amd import binding


class Stream:
    device_index = 1

    def __init__(self, handle):
        self.cuda_stream, self.waited = handle, 0

    def synchronize(self):
        self.waited += 1


@pytest.mark.parametrize("names", [(), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice", "_cuda_getCurrentRawStream")])
def test_current_stream_with_and_without_the_short_ways(names):
    current = [Stream(0x70)]
    short = dict(_cuda_getDevice=lambda: 1, _cuda_getCurrentRawStream=lambda dev: current[0].cuda_stream)
    torch = SimpleNamespace(_C=SimpleNamespace(**{n: short[n] for n in names}), cuda=SimpleNamespace(current_stream=lambda: current[0]))
    assert binding._current_stream(torch) == (1, 0x70)
    assert binding._stream_ptr(torch).value == 0x70
    m = binding.Model.__new__(binding.Model)
    m.torch = torch
    a, b = current[0], Stream(0x90)
    m._synchronize()
    current[0] = b
    m._synchronize()
    m._synchronize()
    assert (a.waited, b.waited) == (1, 2)
