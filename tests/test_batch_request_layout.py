"""A batch request packed in one call has the bytes of one filled field by
field through ctypes."""

import ctypes

from paper_2304_08159_amd import _lib


def test_packed_request_equals_the_structure():
    ints, ptrs = (3, 64, 32, 16, 1, 0, 1), (0x7f0000001000, 0xffff00000000, 256)
    a = _lib.BatchRequest(ints[0], ints[1:4], ints[4:7], *ptrs, 1e-9, 17, 1)
    raw = bytearray(ctypes.sizeof(_lib.BatchRequest))
    _lib.BATCH_REQUEST.pack_into(raw, 0, *ints, *ptrs, 1e-9, 17, 1)
    got = _lib.BatchRequest.from_buffer(raw)
    for name, _ in _lib.BatchRequest._fields_:
        v, w = getattr(a, name), getattr(got, name)
        assert (list(v) == list(w)) if hasattr(v, "__len__") else v == w, name
