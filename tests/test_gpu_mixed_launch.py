"""One decompression launch takes streams of one element format, group length and block size whatever their tuples, with one
tuple or one per data block: batches that mix all of them, at the edges of blocks and vectors, against the oracle's streams."""
import numpy as np
import pytest

from paper_2604_03298_amd import workloads as W
from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

GEN = {BF16: W.gaussian, FP16: W.gaussian_fp16, FP32: W.gaussian_fp32}


def _streams(oracle, dtype, L, B, sizes):
    """(tensor, stream, one tuple per block?) per size: standard deviations far apart, so that the tuples differ; every
    third tensor with one tuple per block, every fifth of random bits (the widest tuple)."""
    rng = np.random.default_rng(1000 * dtype + L)
    out = []
    for i, n in enumerate(sizes):
        w = GEN[dtype](n, 0.02 * 4.0 ** (i % 5 - 2), 50 + i)
        if i % 5 == 4:
            w = rng.integers(0, np.iinfo(WORD[dtype]).max, n, dtype=WORD[dtype], endpoint=True)
        per_block = i % 3 == 2
        if per_block:
            rc, s = oracle.compress_per_block(w, B, dtype, L)
        else:
            b, n_, m, _ = oracle.tune(w, dtype)
            rc, s = oracle.compress(w, (b, n_, m, L), B, dtype=dtype)
        assert rc == 0
        out.append((w, s, per_block))
    return out


@pytest.mark.parametrize("L,B", [(8, 2048), (16, 2048), (16, 16384), (32, 4096), (8, 16384), (32, 32768)])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_one_launch_for_streams_with_different_tuples(gpu, oracle, dtype, L, B):
    torch, enec = gpu.torch, gpu.enec
    # one element, vector edges (4 and 8 elements, 256 and 512 of a wave), block edges, more tensors than a launch takes
    sizes = [1, 3, 4, 5, 8, 9, 255, 257, 511, 513, B - 1, B, B + 1, 2 * B, 2 * B + 7, 3 * B - 4, 5 * B + 3, B + 260]
    made = _streams(oracle, dtype, L, B, sizes)
    assert len({tuple(s[24:27]) for _, s, per_block in made if not per_block}) > 2
    bufs = [torch.from_numpy(np.ascontiguousarray(s)).cuda() for _, s, _ in made]
    wide = torch.int32 if dtype == FP32 else torch.int16
    poison = 0x5A5A5A5A if dtype == FP32 else 0x5A5A
    backs = [torch.full((w.size + 16,), poison, dtype=wide, device="cuda") for w, _, _ in made]
    status = [torch.zeros(1, dtype=torch.int32, device="cuda") for _ in made]
    items, keep = enec.make_decompress_items(bufs, [s[:64].tobytes() for _, s, _ in made], [b[:w.size] for b, (w, _, _) in zip(backs, made)], status)
    assert enec.decompress_batch(bufs, None, backs, items=items) == enec.OK
    torch.cuda.synchronize()
    for (w, _, per_block), back, st in zip(made, backs, status):
        got = back.cpu().numpy().view(WORD[dtype])
        assert np.array_equal(got[:w.size], w), f"{w.size} elements, one tuple per block: {per_block}"
        assert (got[w.size:] == poison).all(), f"{w.size} elements: wrote past the tensor"
        assert int(st.item()) == 0


@pytest.mark.parametrize("L,B", [(8, 2048), (16, 2048), (16, 16384), (32, 4096), (8, 16384), (32, 32768)])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_launches_of_one_two_and_three_streams(gpu, oracle, dtype, L, B):
    """A stream alone has an instance of its own; the second and the third stream of a launch are found by their fields, which come
    with the first one's."""
    torch, enec = gpu.torch, gpu.enec
    made = _streams(oracle, dtype, L, B, [1, 9, 257, B - 1, B, B + 1, 2 * B, 3 * B - 4, 5 * B + 3])
    wide = torch.int32 if dtype == FP32 else torch.int16
    poison = 0x5A5A5A5A if dtype == FP32 else 0x5A5A
    bufs = [torch.from_numpy(np.ascontiguousarray(s)).cuda() for _, s, _ in made]
    for count in (1, 2, 3):
        for i in range(0, len(made), count):
            part = made[i:i + count]
            backs = [torch.full((w.size + 16,), poison, dtype=wide, device="cuda") for w, _, _ in part]
            status = [torch.zeros(1, dtype=torch.int32, device="cuda") for _ in part]
            items, keep = enec.make_decompress_items(bufs[i:i + count], [s[:64].tobytes() for _, s, _ in part],
                                                     [b[:w.size] for b, (w, _, _) in zip(backs, part)], status)
            assert enec.decompress_batch(bufs[i:i + count], None, backs, items=items) == enec.OK
            torch.cuda.synchronize()
            for (w, _, per_block), back, st in zip(part, backs, status):
                got = back.cpu().numpy().view(WORD[dtype])
                assert np.array_equal(got[:w.size], w) and (got[w.size:] == poison).all(), (w.size, per_block, count)
                assert int(st.item()) == 0


@pytest.mark.parametrize("per_block", [False, True])
def test_a_misaligned_offset_is_skipped_and_reported(gpu, oracle, per_block):
    """Both ends of block 1 moved by 8 bytes: its size still fits, its start is no multiple of 16."""
    torch, enec = gpu.torch, gpu.enec
    B = 2048
    w = W.gaussian(4 * B, 0.02, 9)
    rc, s = oracle.compress_per_block(w, B, BF16, 16) if per_block else oracle.compress(w, oracle.tune(w), B)
    assert rc == 0
    bad = s.copy()
    table = bad[64:64 + 8 * 5].view(np.uint64)
    table[1] += 8
    table[2] += 8
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full((w.size,), 0x5A5A, dtype=torch.int16, device="cuda")
    assert enec.decompress_with_header(torch.from_numpy(bad).cuda(), bad[:64].tobytes(), out, status=status) == enec.OK
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint16)
    assert int(status.item()) == enec.E_FORMAT
    assert (got[B:2 * B] == 0x5A5A).all() and np.array_equal(got[3 * B:], w[3 * B:])
