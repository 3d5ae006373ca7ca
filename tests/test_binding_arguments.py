"""What the binding hands to the library, watched without a GPU: the library's entry points are replaced by recorders and the
tensors by objects with made-up addresses."""
import ctypes as C
import os
import struct

import numpy as np
import pytest


class Tensor:
    def __init__(self, at, n, size=2):
        self.at, self.n, self.size = at, n, size

    def data_ptr(self):
        return self.at

    def numel(self):
        return self.n

    def element_size(self):
        return self.size


@pytest.fixture
def enec(monkeypatch):
    from paper_2604_03298_amd import enec as E
    if not os.path.exists(E.LIB_PATH):
        from paper_2604_03298_amd import build
        build.build()
    monkeypatch.setattr(E, "_stream_handle", lambda stream: 0)
    return E


def _record(monkeypatch, enec, name):
    calls = []
    monkeypatch.setattr(_where(enec), name, lambda *a: calls.append(a) or 0)
    return calls


def _where(enec):
    return getattr(enec.lib(), "raw", enec.lib())


def _bytes(pointer, n):
    return pointer if isinstance(pointer, bytes) else C.string_at(pointer, n)


SRCS, OUTS, WS = [Tensor(1 << 20, 5000), Tensor(2 << 20, 70000)], [Tensor(3 << 20, 10000, 1), Tensor(4 << 20, 300000, 1)], Tensor(5 << 20, 1 << 20, 1)
SIZES = [2048, 32768]


@pytest.mark.parametrize("kind", [list, tuple, np.array, lambda v: np.array(v, np.int32), lambda v: np.array(v, np.uint16), lambda v: [np.uint16(x) for x in v]])
def test_block_sizes_may_be_integers_of_any_kind(enec, monkeypatch, kind):
    sizes = kind(SIZES)
    calls = _record(monkeypatch, enec, "enec_compress_per_block_batch")
    assert enec.compress_per_block_batch(SRCS, OUTS, WS, block_sizes=sizes, dtype=0) == 0
    packed = _bytes(calls[0][0], 96)
    assert [struct.unpack_from("<QQI4xQQQ", packed, 48 * i) for i in range(2)] == [(1 << 20, 5000, 2048, 3 << 20, 10000, 0), (2 << 20, 70000, 32768, 4 << 20, 300000, 0)]
    if isinstance(sizes, np.ndarray):
        sizes = list(sizes)                     # (this call asks for the truth of the list)
    calls = _record(monkeypatch, enec, "enec_compress_batch")
    assert enec.compress_batch(SRCS, [(122, 6, 3, 16), None], OUTS, WS, block_sizes=sizes, dtype=0) == 0
    packed = _bytes(calls[0][0], 112)
    items = [struct.unpack_from("<QQI4xQQQQ", packed, 56 * i) for i in range(2)]
    assert [it[:3] + it[4:] for it in items] == [(1 << 20, 5000, 2048, 3 << 20, 10000, 0), (2 << 20, 70000, 32768, 4 << 20, 300000, 0)]
    assert items[0][3] != 0 and items[1][3] == 0


def test_tuples_may_come_from_an_iterator(enec, monkeypatch):
    calls = _record(monkeypatch, enec, "enec_compress_batch")
    assert enec.compress_batch(SRCS, (p for p in [(122, 6, 3, 16), None]), OUTS, WS, dtype=0) == 0
    items = [struct.unpack_from("<QQI4xQQQQ", _bytes(calls[0][0], 112), 56 * i) for i in range(2)]
    assert items[0][3] != 0 and items[1][3] == 0
