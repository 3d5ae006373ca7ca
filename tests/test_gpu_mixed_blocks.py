"""A decompression launch that takes streams of several block sizes: those of few blocks join the launch of the largest size.  At
the edges of blocks, with one tuple and one per block, with a damaged stream among them, against the oracle's streams."""
import numpy as np
import pytest

from paper_2604_03298_amd import workloads as W
from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

GEN = {BF16: W.gaussian, FP16: W.gaussian_fp16, FP32: W.gaussian_fp32}
SIZES = {8: [2048, 4096, 8192, 16384], 16: [2048, 4096, 8192, 16384, 32768], 32: [4096, 8192, 16384, 32768]}


@pytest.mark.parametrize("order", ["up", "down", "wide first"])
@pytest.mark.parametrize("L", [8, 16, 32])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_streams_of_all_block_sizes_in_one_call(gpu, oracle, dtype, L, order):
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(100 * dtype + L)
    made = []
    for B in SIZES[L]:
        # one element, a ragged block, whole blocks, the most that join (16) and one block more
        for i, n in enumerate([1, B - 3, 2 * B, 16 * B - 5, 16 * B + 1][:5 if B < 16384 else 3]):
            w = GEN[dtype](n, 0.02 * 4.0 ** (i % 3 - 1), B + i)
            if i == 1:                                   # random bits: the widest tuple, the largest payload
                w = rng.integers(0, np.iinfo(WORD[dtype]).max, n, dtype=WORD[dtype], endpoint=True)
            if i == 2:
                rc, s = oracle.compress_per_block(w, B, dtype, L)
            else:
                rc, s = oracle.compress(w, oracle.tune(w, dtype)[:3] + (L,), B, dtype=dtype)
            assert rc == 0
            made.append((w, s, B, i))
    if order != "up":
        made.reverse()
    if order == "wide first":                            # a small stream of few bits sets the launch up, wide ones join
        made.sort(key=lambda x: x[3] != 0)
    bad = next(j for j, x in enumerate(made) if x[3] == 2 and x[2] == SIZES[L][0])
    wide, poison = (torch.int32, 0x5A5A5A5A) if dtype == FP32 else (torch.int16, 0x5A5A)
    streams = [s.copy() for _, s, _, _ in made]
    headers = [s[:64].tobytes() for s in streams]
    streams[bad][64 + 8:64 + 16].view(np.uint64)[0] += 16 * 4096              # block 1 begins behind block 2
    bufs = [torch.from_numpy(np.ascontiguousarray(s)).cuda() for s in streams]
    backs = [torch.full((w.size + 16,), poison, dtype=wide, device="cuda") for w, _, _, _ in made]
    status = [torch.zeros(1, dtype=torch.int32, device="cuda") for _ in made]
    items, keep = enec.make_decompress_items(bufs, headers, [b[:w.size] for b, (w, _, _, _) in zip(backs, made)], status)
    assert enec.decompress_batch(bufs, None, backs, items=items) == enec.OK
    torch.cuda.synchronize()
    for j, ((w, _, B, i), back, st) in enumerate(zip(made, backs, status)):
        got = back.cpu().numpy().view(WORD[dtype])
        assert (got[w.size:] == poison).all(), f"blocks of {B}, {w.size} elements: wrote past the tensor"
        if j == bad:
            assert int(st.item()) == enec.E_FORMAT and (got[:w.size] == poison).all()
        else:
            assert np.array_equal(got[:w.size], w), f"blocks of {B}, {w.size} elements"
            assert int(st.item()) == 0


@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_more_small_streams_than_places_ahead_of_a_large_one(gpu, oracle, dtype):
    """The large stream's launch is filled up with some of the small ones, the others follow in one of their own."""
    torch, enec = gpu.torch, gpu.enec
    words = [GEN[dtype](n, 0.02, 50 + i) for i, n in enumerate([4096 - i for i in range(9)] + [2048] * 10 + [20 * 16384 + 5])]
    made = [oracle.compress(w, oracle.tune(w, dtype), oracle.default_block(w.size), dtype=dtype) for w in words]
    assert all(rc == 0 for rc, _ in made)
    bufs = [torch.from_numpy(s).cuda() for _, s in made]
    wide = torch.int32 if dtype == FP32 else torch.int16
    backs = [torch.zeros(w.size, dtype=wide, device="cuda") for w in words]
    assert enec.decompress_batch(bufs, [s[:64].tobytes() for _, s in made], backs) == enec.OK
    torch.cuda.synchronize()
    for w, back in zip(words, backs):
        assert np.array_equal(back.cpu().numpy().view(WORD[dtype]), w), w.size
