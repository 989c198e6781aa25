"""The packed structs the binding passes per call are the ctypes structs, byte
for byte, and follow the tensors they are made from."""
import numpy as np
import pytest
import torch

from paper_2412_08585_amd import binding as b


@pytest.mark.parametrize("bits", [[4], [4, 2, 4], [2, 4] * 32])
def test_packed_structs_are_the_ctypes_structs(bits):
    c = b.PagedKVCache(3, 5, bits, device="cpu")
    t = b.KVTail(4, len(bits), device="cpu")
    assert c._packed() == bytes(c.struct())
    assert t._packed() == bytes(t.struct())
    assert t.narrow(1, 2)._packed() == bytes(t.narrow(1, 2).struct())
    c.pages = torch.zeros(7, c.page_bytes, dtype=torch.uint8)  # other storage, other widths
    c.head_bits = np.array([6 - x for x in bits], np.uint8)
    assert c._packed() == bytes(c.struct())


def test_default_scale_and_cpu_tensors():
    assert b._scale(128, None) == float(1.0 / np.sqrt(128)) and b._scale(128, 0.25) == 0.25
    with pytest.raises(ValueError):
        b._stream(torch.device("cpu"))
    with pytest.raises(ValueError):
        b._ptr(torch.zeros(4, 4).t()[:2])
    assert b._ptr(None) is None
