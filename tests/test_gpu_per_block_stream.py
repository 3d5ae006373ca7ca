"""The per-block kernel with deferred stores (default block size) where it can go wrong: grids of one block, fewer blocks than
workgroup slots, exactly as many, two rounds (tickets drawn ahead) and a ragged end; launches that mix tensors, block sizes and
both kinds of call on one workspace; a workspace with room for the other kernel's words only; waits that are given up."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2604_03298_amd import workloads as W
from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)
from test_gpu_per_block import _batch, _check, _mixed16

pytestmark = pytest.mark.gpu
B = 16384


def _tensor(n, dtype, seed):
    """Blocks of several kinds: a pool of 23 mixed blocks, repeated with another rotation each time."""
    if dtype == FP32:
        up = _mixed16(23, B, seed).astype(np.uint32) << 16
        pool = up | np.random.default_rng(seed).integers(0, 1 << 16, up.size).astype(np.uint32)
    else:
        pool = _mixed16(23, B, seed, dtype)
    out = np.empty(n, WORD[dtype])
    for i, s in enumerate(range(0, n, pool.size)):
        out[s:s + pool.size] = np.roll(pool, 977 * i)[:min(pool.size, n - s)]
    return out


@pytest.mark.parametrize("L", [8, 16, 32])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_numbers_of_blocks(gpu, oracle, dtype, L):
    # 512 or 768 workgroups fit the device
    for blocks, more in [(1, 0), (1, 1), (7, 5), (8, 0), (9, B - 1)] + ([(511, 0), (512, 3), (768, 0), (768, 1), (1537, 777)] if L == 16 else [(771, 9)]):
        _check(gpu, oracle, _tensor(blocks * B + more, dtype, blocks), dtype, B, f"{blocks} blocks and {more}", L)


def test_both_kinds_of_call_and_all_block_sizes_on_one_workspace(gpu, oracle):
    torch, enec = gpu.torch, gpu.enec
    ws = enec.new_workspace(64 * B, 2048)
    one = W.gaussian(30 * B + 5, 0.02, 3)
    prm = oracle.tune(one)
    want_one = oracle.compress(one, prm, B)[1]
    out = torch.empty(enec.compress_bound(one.size), dtype=torch.uint8, device="cuda")
    src = gpu.to_dev(one, BF16)
    for turn in range(3):
        tensors = [_tensor(n, BF16, turn + i) for i, n in enumerate([5 * B, 4097, B + 1, 2 * B - 1, 0, 30000, 9 * B + 8])]
        Bs = [B, 2048, B, 4096, B, 32768, B]
        rc, res = _batch(gpu, tensors, BF16, Bs, 16, ws)
        assert rc == 0
        for w, block, (got, nbytes, cap) in zip(tensors, Bs, res):
            s_o = oracle.compress_per_block(w, block, BF16, 16)[1]
            assert nbytes == s_o.size and np.array_equal(got[:nbytes], s_o), (turn, w.size, block)
            assert (got[cap:] == 0xA5).all()
        assert enec.compress(src[:one.size], prm, out, ws) == 0
        torch.cuda.synchronize()
        assert np.array_equal(out[:want_one.size].cpu().numpy(), want_one)


def test_a_workspace_with_room_for_the_look_back_words_only(gpu, oracle):
    """Smaller than enec_workspace_bytes says, but it was always enough for this call, and stays so."""
    torch, enec = gpu.torch, gpu.enec
    blocks = 900
    w = _tensor(blocks * B, BF16, 77)
    state = 1024 + 16 * 2048
    words = next(n for n in range(blocks, 4 * blocks) if n >= n // 9 + (n // 9) % 2 + 64 + blocks)
    ws = torch.zeros((state + 8 * words + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
    assert ws.numel() < enec.workspace_bytes(w.size)
    rc, [(got, nbytes, _)] = _batch(gpu, [w], BF16, [B], 16, ws)
    s_o = oracle.compress_per_block(w, B, BF16, 16)[1]
    assert rc == 0 and nbytes == s_o.size and np.array_equal(got[:nbytes], s_o)
    rc, _ = _batch(gpu, [w], BF16, [B], 16, ws[:-1024])
    assert rc == enec.E_CAPACITY


def _test_library(enec):
    """libenec_test.so, which reads ENEC_SPIN_LIMIT."""
    L = C.CDLL(os.path.join(os.path.dirname(enec.LIB_PATH), "libenec_test.so"))
    L.enec_compress_per_block.restype = C.c_int
    L.enec_compress_per_block.argtypes = [C.c_void_p, C.c_size_t, C.c_int, C.c_uint32, C.c_uint32, C.c_void_p, C.c_size_t, C.c_void_p,
                                          C.c_void_p, C.c_size_t, C.c_void_p]
    return L


def test_a_wait_given_up_shows_in_the_header(gpu, oracle, monkeypatch):
    """With a bound of one poll every run ends with status 0 and the oracle's stream, or with ENEC_E_HIP and size 0."""
    torch, enec = gpu.torch, gpu.enec
    L = _test_library(enec)
    w = _tensor(1900 * B + 77, BF16, 5)
    s_o = oracle.compress_per_block(w, B, BF16, 16)[1]
    ref = torch.from_numpy(s_o).cuda()
    src = gpu.to_dev(w, BF16)
    ws = enec.new_workspace(w.size)
    out = torch.zeros(enec.compress_bound_per_block(w.size), dtype=torch.uint8, device="cuda")
    size = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    monkeypatch.setenv("ENEC_SPIN_LIMIT", "1")
    for _ in range(6):
        out.zero_()
        assert L.enec_compress_per_block(src.data_ptr(), w.size, 0, B, 16, out.data_ptr(), out.numel(), size.data_ptr(), ws.data_ptr(), ws.numel(), None) == 0
        torch.cuda.synchronize()
        info = enec.stream_info(out[:64].cpu().numpy())
        if info["status"] == 0:
            assert int(size.item()) == s_o.size and torch.equal(out[:s_o.size], ref)
        else:
            assert info["status"] == enec.E_HIP and info["total_bytes"] == 0 and int(size.item()) == 0
            enec.workspace_init(ws)
            torch.cuda.synchronize()
    monkeypatch.delenv("ENEC_SPIN_LIMIT")
    enec.workspace_init(ws)
    assert enec.compress_per_block(src[:w.size], out, ws, block_size=B, out_bytes=size) == 0
    torch.cuda.synchronize()
    assert int(size.item()) == s_o.size and torch.equal(out[:s_o.size], ref)


def test_a_dirty_workspace_ends_in_a_status_not_in_a_hang(gpu, oracle, monkeypatch):
    """Accumulators that claim 100 blocks too many, as a call that died may leave them: no group of blocks ever completes, so every
    block behind the first group gives up after 200 polls.  Each is then stored at a start that misses sizes, below its own."""
    torch, enec = gpu.torch, gpu.enec
    L = _test_library(enec)
    w = _tensor(400 * B + 9, BF16, 6)
    src = gpu.to_dev(w, BF16)
    ws = enec.new_workspace(w.size)
    state = 1024 + 16 * 2048                             # control records and histograms, then the state words
    words = ws[state:state + (ws.numel() - state) // 8 * 8].view(torch.int64)
    words[:words.numel() // 9] = 100 << 48
    out = torch.zeros(enec.compress_bound_per_block(w.size), dtype=torch.uint8, device="cuda")
    size = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    monkeypatch.setenv("ENEC_SPIN_LIMIT", "200")
    assert L.enec_compress_per_block(src.data_ptr(), w.size, 0, B, 16, out.data_ptr(), out.numel(), size.data_ptr(), ws.data_ptr(), ws.numel(), None) == 0
    torch.cuda.synchronize()
    monkeypatch.delenv("ENEC_SPIN_LIMIT")
    info = enec.stream_info(out[:64].cpu().numpy())
    assert info["status"] == enec.E_HIP and info["total_bytes"] == 0 and int(size.item()) == 0
    enec.workspace_init(ws)
    assert enec.compress_per_block(src[:w.size], out, ws, block_size=B, out_bytes=size) == 0
    torch.cuda.synchronize()
    s_o = oracle.compress_per_block(w, B, BF16, 16)[1]
    assert int(size.item()) == s_o.size and np.array_equal(out[:s_o.size].cpu().numpy(), s_o)
