"""The CPython function of the decode step's call: what it hands to the entry point, and what it refuses (no GPU needed)."""
import ctypes as C

import pytest
import torch

from paper_2510_13797_amd import bc


def test_native_call_hands_over_addresses_and_numbers():
    bc.load()
    seen = []
    vp = C.c_void_p
    entry = C.CFUNCTYPE(C.c_int32, *[vp] * 10, C.c_size_t, vp)(lambda *a: seen.append(a) or 5)
    at = C.cast(entry, vp).value
    shape, cache = bc.bc_shape(2, 4, 1, 64, bc.BC_BF16, 0.125), bc.bc_cache()
    t = [torch.zeros(3 + i) for i in range(7)]
    args = [at, shape, cache, *t[:4], None, t[4], t[5], t[6], 1 << 40, 7]
    assert bc._call(*args) == 5
    assert [x or 0 for x in seen[0]] == [C.addressof(shape), C.addressof(cache), *(x.data_ptr() for x in t[:4]), 0,
                                         *(x.data_ptr() for x in t[4:]), 1 << 40, 7]
    for i, bad in ((0, None), (0, 0), (1, 3), (2, None), (3, 4), (11, -1), (11, "8"), (12, None)):
        with pytest.raises((TypeError, ValueError, AttributeError, OverflowError, BufferError)):
            bc._call(*[bad if j == i else x for j, x in enumerate(args)])
    with pytest.raises(TypeError):
        bc._call(*args[:-1])
    assert len(seen) == 1
