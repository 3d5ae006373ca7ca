"""Tensors of one data block: a launch takes them whatever their tuples and block sizes.  Edges of vectors, rows and blocks, windows
at the ends of the exponent range, range errors of one tensor among others, more tensors than a launch takes, and tensors of one
block beside larger ones that they share a kernel with; against the oracle, byte for byte."""
import numpy as np
import pytest

from test_gpu_compress_edges import EXP, SHIFT, _tensor
from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _run(gpu, oracle, dtype, jobs):
    """jobs: (tensor, params, block size); every stream against the oracle's."""
    torch, enec = gpu.torch, gpu.enec
    wide = np.int32 if dtype == FP32 else np.int16
    srcs = [torch.from_numpy(np.ascontiguousarray(w).view(wide)).cuda() for w, _, _ in jobs]
    caps = [enec.compress_bound(w.size, dtype, B) for w, _, B in jobs]
    outs = [torch.full((c + 64,), 0xA5, dtype=torch.uint8, device="cuda") for c in caps]
    sizes = torch.full((len(jobs),), -1, dtype=torch.int64, device="cuda")
    ws = enec.new_workspace(sum(w.size for w, _, _ in jobs) + 32768 * len(jobs), 2048)
    for _ in range(2):
        assert enec.compress_batch(srcs, [p for _, p, _ in jobs], outs, ws, block_sizes=[B for _, _, B in jobs],
                                   out_bytes=[sizes[i:i + 1] for i in range(len(jobs))], dtype=dtype) == enec.OK
    torch.cuda.synchronize()
    for (w, p, B), out, size, cap in zip(jobs, outs, sizes.tolist(), caps):
        rc, want = oracle.compress(w, p, B, dtype=dtype)
        got = out.cpu().numpy()
        assert (got[cap:] == 0xA5).all()
        if rc == enec.E_RANGE:
            info = enec.stream_info(got[:64])
            assert info["status"] == enec.E_RANGE and info["total_bytes"] == 0 and size == 0, (w.size, p, B)
        else:
            assert rc == 0 and size == want.size and np.array_equal(got[:size], want), (w.size, p, B)


@pytest.mark.parametrize("L", [8, 16, 32])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_tensors_of_one_block(gpu, oracle, dtype, L):
    rng = np.random.default_rng(10 * dtype + L)
    full = 5 if dtype == FP16 else 8
    windows = [(3, 10), (0, 6), (24, 31), (0, 31)] if dtype == FP16 else [(100, 118), (0, 11), (240, 255), (0, 255)]
    jobs, i = [], 0
    for B in (2048, 4096, 8192, 16384, 32768):
        if not (128 * L <= B <= 2048 * L):
            continue
        for n in (1, 7, 8, B // 8 - 1, B // 8 + 3, 5 * (B // 8) + 17, B - 1, B):
            lo, hi = windows[i % 4]
            w = _tensor(rng, dtype, n, lo, hi, (0.0, 0.03, 0.5, 1.0)[(i // 4) % 4])
            b, nw, m, _ = oracle.tune(w, dtype)
            jobs.append((w, (b, full if i % 4 == 3 else nw, m, L), B))
            if i % 4 == 1:                               # an exponent outside a window that is clear of the ends, or touches them
                bad = w.copy()
                keep = WORD[dtype](~(EXP[dtype] << SHIFT[dtype]) & np.iinfo(WORD[dtype]).max)
                bad[n // 2] = (bad[n // 2] & keep) | (WORD[dtype](EXP[dtype]) << WORD[dtype](SHIFT[dtype]))
                jobs.append((bad, (b, nw, m, L), B))
            i += 1
    assert len(jobs) > 32
    _run(gpu, oracle, dtype, jobs)
    for j in jobs[:6]:
        _run(gpu, oracle, dtype, [j])


@pytest.mark.parametrize("n", range(1, 9))
def test_every_width_pair(gpu, oracle, n):
    rng = np.random.default_rng(n)
    for dtype in (BF16, FP16, FP32):
        if n > (5 if dtype == FP16 else 8):
            continue
        b = 1 << (n - 1) if dtype == FP16 else 120
        lo, hi = (0, EXP[dtype]) if n == (5 if dtype == FP16 else 8) else (max(0, b - (1 << (n - 1)) + 1), min(EXP[dtype], b + (1 << (n - 1))))
        jobs = [(_tensor(rng, dtype, 3000 + 64 * m, lo, hi, 0.3), (b, n, m, L), 4096) for m in range(n + 1) for L in (8, 16, 32)]
        _run(gpu, oracle, dtype, jobs)


@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_whole_exponents_as_records(gpu, oracle, dtype):
    """m = 0: no low plane (fp16: three bits), records as long as they get; blocks of 32768 take more than 64 KB of LDS."""
    rng = np.random.default_rng(dtype)
    full = 5 if dtype == FP16 else 8
    jobs = [(_tensor(rng, dtype, B - 3, 0, EXP[dtype], 1.0), (7, full, 0, L), B)
            for B in (2048, 4096, 16384, 32768) for L in (8, 16, 32) if 128 * L <= B <= 2048 * L]
    for j in jobs:
        _run(gpu, oracle, dtype, [j])


@pytest.mark.parametrize("dtype", [BF16, FP32])
@pytest.mark.parametrize("L", [16, 32])
def test_whole_exponents_as_records_of_many_tensors(gpu, oracle, dtype, L):
    """The same where a launch has more than four tensors: more than 64 KB of LDS for the kernel with the long arguments, smaller
    blocks among its workgroups."""
    rng = np.random.default_rng(40 + dtype + L)
    jobs = [(_tensor(rng, dtype, B - i, 0, EXP[dtype], 1.0), (7, 8, 0, L), B)
            for i, B in enumerate((32768, 4096, 32768, 16384, 8192, 32768, 4096))]
    _run(gpu, oracle, dtype, jobs)


def test_beside_larger_tensors(gpu, oracle):
    """One-block tensors that share (m, n, L, block size) with a tensor of more blocks go through its launch, the others don't."""
    rng = np.random.default_rng(3)
    jobs = []
    for i in range(40):
        B = (16384, 4096)[i % 2]
        w = _tensor(rng, BF16, (B - 5, 3 * B + 1, 77, B, 9 * B)[i % 5], 100 + i % 3, 118, 0.02)
        jobs.append((w, (115, 5, 2 + i % 3, 16), B))
    _run(gpu, oracle, BF16, jobs)


@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
@pytest.mark.parametrize("L", [8, 16, 32])
def test_in_the_launch_of_a_larger_tensor(gpu, oracle, dtype, L):
    """One-block tensors with tuples and block sizes of their own beside tensors of the default block size: the first sixteen of the
    same group length ride along, unless their records need more LDS than the larger tensors' kernel has (the second call: a tuple of
    one bit beside whole exponents as records), one of them with an exponent outside its window."""
    rng = np.random.default_rng(30 + 3 * dtype + L)
    full = 5 if dtype == FP16 else 8
    lo, hi = (10, 17) if dtype == FP16 else (100, 118)
    small = []
    for i in range(19):
        B = max((2048, 4096, 8192, 16384)[i % 4], 128 * L)
        w = _tensor(rng, dtype, (1, 700, B - 1, B)[i // 4 % 4] if B < 16384 else B - 9 * i, lo, hi, 0.1)
        b, n, m, _ = oracle.tune(w, dtype)
        small.append((w, (b, n, m, L), B))
    w = small[5][0].copy()
    keep = WORD[dtype](~(EXP[dtype] << SHIFT[dtype]) & np.iinfo(WORD[dtype]).max)
    w[w.size // 2] = (w[w.size // 2] & keep) | (WORD[dtype](EXP[dtype]) << WORD[dtype](SHIFT[dtype]))
    small[5] = (w, small[5][1], small[5][2])
    big = _tensor(rng, dtype, 5 * 16384 + 77, lo, hi, 0.05)
    _run(gpu, oracle, dtype, small[:7] + [(big, oracle.tune(big, dtype)[:3] + (L,), 16384)] + small[7:] + [(small[0][0], small[0][1][:3] + (16,), 4096)])
    flat = np.full(3 * 16384 - 5, WORD[dtype](lo) << WORD[dtype](SHIFT[dtype]), dtype=WORD[dtype])
    wide = [(_tensor(rng, dtype, 16384 - i, 0, EXP[dtype], 1.0), (7, full, 0, L), 16384) for i in range(2)]
    _run(gpu, oracle, dtype, wide + [(flat, (lo, 1, 1, L), 16384)] + small[:2])


@pytest.mark.parametrize("larges", [11, 16, 17])
def test_in_launches_with_little_room(gpu, oracle, larges):
    """The more tensors a launch has, the fewer of one block it takes along: six, none, and sixteen with the seventeenth."""
    rng = np.random.default_rng(larges)
    jobs = [(_tensor(rng, BF16, 16384 + 999 * i + 1, 100, 118, 0.02), (115, 5, 3, 16), 16384) for i in range(larges)]
    for i in range(18):
        w = _tensor(rng, BF16, 4096 - 13 * i, 100, 118, 0.1)
        jobs.insert(2 * i, (w, oracle.tune(w, BF16), 4096))
    _run(gpu, oracle, BF16, jobs)


@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
@pytest.mark.parametrize("L", [8, 16, 32])
def test_in_the_launches_that_take_them(gpu, oracle, dtype, L):
    """Beside each tuple whose instance takes tensors of one block along, from the lengths at which a vector, a thread's turn and a
    block end; records of whole exponents, which the kernel's LDS may be too small for."""
    rng = np.random.default_rng(60 + 3 * dtype + L)
    full = 5 if dtype == FP16 else 8
    lo, hi = (10, 17) if dtype == FP16 else (100, 118)
    for a in (1, 2, 3):
        for m in range(2, full - a + 1):
            big = _tensor(rng, dtype, 2 * 16384 + 5, lo, lo + 1, 0.0)
            jobs = [(big, (lo, m + a, m, L), 16384), (_tensor(rng, dtype, 16384 - a, 0, EXP[dtype], 1.0), (7, full, 0, L), 16384)]
            for n in (1, 2047, 2049, 4096 - m):
                w = _tensor(rng, dtype, n, lo, hi, 0.1)
                jobs.append((w, oracle.tune(w, dtype)[:3] + (L,), 4096 if n > 2048 or L == 32 else 2048))
            _run(gpu, oracle, dtype, jobs)
