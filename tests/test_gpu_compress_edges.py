"""Compression where a block ends inside a row: the elements behind the tensor's end lie in the same buffer and have
exponents that no window of the tensor holds, so one that is read as an element shows in the stream or as a range error.
Against the oracle, every format, group length and both kinds of block size, with windows clear of the ends of the exponent
range, touching them, and covering all of it."""
import numpy as np
import pytest

from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHIFT = {BF16: 7, FP16: 10, FP32: 23}
EXP = {BF16: 255, FP16: 31, FP32: 255}


def _tensor(rng, dtype, n, lo, hi, rare):
    """n elements with exponents in [lo, hi], mostly in the upper half of it; `rare` = share anywhere in the range."""
    x = rng.integers((lo + hi + 1) // 2, hi, n, endpoint=True)
    x = np.where(rng.random(n) < rare, rng.integers(lo, hi, n, endpoint=True), x)
    bits = rng.integers(0, np.iinfo(WORD[dtype]).max, n, dtype=WORD[dtype], endpoint=True)
    keep = WORD[dtype](~(EXP[dtype] << SHIFT[dtype]) & np.iinfo(WORD[dtype]).max)
    return (bits & keep) | (x.astype(WORD[dtype]) << WORD[dtype](SHIFT[dtype]))


@pytest.mark.parametrize("L,B", [(16, 16384), (16, 2048), (8, 16384), (8, 4096), (32, 16384), (32, 32768)])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_blocks_that_end_inside_a_row(gpu, oracle, dtype, L, B):
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(100 * dtype + L + B)
    C = B // 8
    # every remainder of a vector, in the first, a middle and the last row, the last lane of a row and of a block
    ends = [1, 7, 9, C - 1, C, C + 2, 3 * C + 8 * 5 + 3, 4 * C - 4, 7 * C + 6, B - 8, B - 5, B - 1]
    full = 5 if dtype == FP16 else 8
    windows = ([(3, 10), (0, 6), (24, 31), (0, 31)] if dtype == FP16 else [(100, 118), (0, 11), (240, 255), (0, 255)])
    ws = enec.new_workspace(3 * B, B)
    for i, end in enumerate(ends):
        lo, hi = windows[i % 4]
        n = (0, B, 2 * B)[i % 3] + end
        w = _tensor(rng, dtype, n, lo, hi, (0.0, 0.02, 0.5, 1.0)[(i // 4) % 4])
        b, nw, m, _ = oracle.tune(w, dtype)
        prm = (b, full if i % 4 == 3 else nw, m, L)
        rc, want = oracle.compress(w, prm, B, dtype=dtype)
        assert rc == 0
        outside = 0 if lo > 0 else EXP[dtype]                      # an exponent that the tensor doesn't have
        buf = np.full(n + 64, outside << SHIFT[dtype], dtype=WORD[dtype])
        buf[:n] = w
        wide = np.int32 if dtype == FP32 else np.int16
        src = torch.from_numpy(buf.view(wide)).cuda()[:n]
        out = torch.full((enec.compress_bound(n, dtype, B),), 0xA5, dtype=torch.uint8, device="cuda")
        assert enec.compress(src, prm, out, ws, block_size=B, dtype=dtype) == enec.OK
        torch.cuda.synchronize()
        got = out.cpu().numpy()[:want.size]
        assert np.array_equal(got, want), f"{n} elements, exponents {lo}..{hi}, tuple {prm}"
