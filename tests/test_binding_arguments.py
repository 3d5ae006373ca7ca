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
    monkeypatch.setattr(enec.lib().raw, name, lambda *a: calls.append(a) or 0)
    return calls


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


def test_the_prototypes_of_lib_tell_their_structures_apart(enec):
    """lib() hands out the entry points with the structures they take; the binding's own calls, which pass packed bytes, don't
    loosen them.  Every accepted call fails in the library's first check (dtype 7)."""
    from paper_2604_03298_amd.enec import CompressItem, DecompressItem, Params, PerBlockItem, TuneItem
    L, at = enec.lib(), 1 << 20
    prm = Params(122, 6, 3, 16)
    for given in (prm, C.byref(prm), C.pointer(prm), None):
        assert L.enec_compress(at, 10, 7, 0, given, at, 1 << 20, None, at, 1 << 20, None) == enec.E_DTYPE
    assert L.enec_compress_batch((CompressItem * 1)(), 1, 7, at, 1 << 20, None) == enec.E_DTYPE
    assert L.enec_compress_per_block_batch((PerBlockItem * 1)(), 1, 7, 16, at, 1 << 20, None) == enec.E_DTYPE
    hist = (C.c_uint64 * 256)()
    assert L.enec_tune_batch((TuneItem * 1)(), 1, 7, 1, C.byref(prm), hist, at, 1 << 20, None) == enec.E_DTYPE
    for name, before, after in (("enec_compress_batch", (), (1, 7, at, 1 << 20, None)), ("enec_compress_per_block_batch", (), (1, 7, 16, at, 1 << 20, None)),
                                ("enec_tune_batch", (), (1, 7, 1, prm, hist, at, 1 << 20, None)),
                                ("enec_compress", (at, 10, 7, 0), (at, 1 << 20, None, at, 1 << 20, None))):
        with pytest.raises(C.ArgumentError):
            getattr(L, name)(*before, (DecompressItem * 1)(), *after)
