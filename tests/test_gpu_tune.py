"""The counting kernel at the edges of its loop (a workgroup's vectors in flight, whole chunks of a sample, elements behind the
last vector), and calls that tune from several threads at once, more of them than pinned slots are kept."""
import threading

import numpy as np
import pytest

from test_gpu_dtypes import gpu, BF16, FP16, FP32, WORD  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

STEP = 512 * 8          # elements that one round of a workgroup's loads covers (16-bit formats)


@pytest.mark.parametrize("every", [1, 2, 16])
@pytest.mark.parametrize("dtype", [BF16, FP16, FP32])
def test_counts_at_the_edges_of_the_loop(gpu, oracle, dtype, every):
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(10 * dtype + every)
    sizes = [1, 3, 8, 9, STEP - 1, STEP, STEP + 1, 4 * STEP + 5, 5 * STEP, 256 * STEP - 3, 256 * STEP * 4 + 4097, 256 * STEP * 5 + 2]
    ws_tensors = [rng.integers(0, np.iinfo(WORD[dtype]).max, n, dtype=WORD[dtype], endpoint=True) for n in sizes]
    dev = [torch.from_numpy(w.view(np.int32 if dtype == FP32 else np.int16)).cuda() for w in ws_tensors]
    ws = enec.new_workspace(sum(sizes))
    alone = [enec.tune_batch([d], ws, every=every, dtype=dtype, want_histograms=True) for d in dev]
    together = enec.tune_batch(dev, ws, every=every, dtype=dtype, want_histograms=True)
    for i, w in enumerate(ws_tensors):
        part = w if every == 1 else oracle.sample(w, every, dtype)
        want = oracle.histogram(part, dtype)
        assert np.array_equal(alone[i][1][0], want), sizes[i]
        assert np.array_equal(together[1][i], want), sizes[i]
        E = 5 if dtype == FP16 else 8
        assert tuple(alone[i][0][0])[:3] == tuple(oracle.tune_hist(want, E)[0])[:3] == tuple(together[0][i])[:3]


def test_calls_from_many_threads(gpu, oracle):
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(5)
    jobs = []
    for i in range(7):
        ws = [rng.integers(i << 10, (i << 10) + 3000, 50001 + 777 * i + j, dtype=np.uint16) for j in range(17 if i == 3 else 3)]
        dev = [torch.from_numpy(w.view(np.int16)).cuda() for w in ws]
        jobs.append((ws, dev, enec.new_workspace(sum(w.size for w in ws)), torch.cuda.Stream()))
    torch.cuda.synchronize()
    got = [[] for _ in jobs]

    def work(i):
        for _ in range(5):
            got[i].append(enec.tune_batch(jobs[i][1], jobs[i][2], stream=jobs[i][3], want_histograms=True))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, (ws, _, _, _) in enumerate(jobs):
        want = np.stack([oracle.histogram(w) for w in ws])
        assert len(got[i]) == 5
        for _, hist in got[i]:
            assert np.array_equal(hist, want), i


@pytest.mark.parametrize("every", [1, 3])
@pytest.mark.parametrize("dirt", ["counts", "done", "both", "after an early last"])
def test_a_workspace_whose_counters_are_not_zero(gpu, oracle, dirt, every):
    """Every call leaves its counters zero for the next one.  Where something else lies there the counts are right all the same."""
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(3)
    sizes = [5 * STEP + 3, 1, 4096, 40 * STEP + 4099]
    data = [rng.integers(15000, 17000, n, dtype=np.uint16) for n in sizes]
    dev = [torch.from_numpy(w.view(np.int16)).cuda() for w in data]
    ws = enec.new_workspace(sum(sizes))
    want = [oracle.histogram(w if every == 1 else oracle.sample(w, every, BF16), BF16) for w in data]
    wgs = sum(max(1, -(-(n // 8 // every) // 512)) for n in sizes)     # of the launch: one for every 512 vectors of a tensor's sample
    for _ in range(2):
        if dirt in ("counts", "both"):
            ws[1024:1024 + 4 * 2048] = 7
        if dirt in ("done", "both"):
            ws[1008:1012] = 255
        if dirt == "after an early last":
            ws[1008] = wgs - 6                                    # (the sixth workgroup takes itself for the last)
        for _ in range(2):
            _, hist = enec.tune_batch(dev, ws, every=every, dtype=BF16, want_histograms=True)
            for h, w in zip(hist, want):
                assert np.array_equal(h, w)
    assert int(ws[1008:1012].sum()) == 0 and int(ws[1024:1024 + 4 * 2048].to(torch.int64).sum()) == 0


@pytest.mark.parametrize("count", [1, 2, 15, 16, 17])
def test_as_many_histograms_as_a_launch_hands_over(gpu, oracle, count):
    """Two counters at a time for every thread of the last workgroup, up to sixteen tensors' of them; empty tensors among these."""
    torch, enec = gpu.torch, gpu.enec
    rng = np.random.default_rng(count)
    data = [rng.integers(0, 65536, (0 if i % 5 == 3 else 700 * i + 1), dtype=np.uint16) for i in range(count)]
    dev = [torch.from_numpy(w.view(np.int16)).cuda() for w in data]
    ws = enec.new_workspace(sum(w.size for w in data) + 1)
    for _ in range(2):
        prm, hist = enec.tune_batch(dev, ws, dtype=BF16, want_histograms=True)
        for w, p, h in zip(data, prm, hist):
            want = oracle.histogram(w, BF16)
            assert np.array_equal(h, want) and tuple(p) == oracle.tune_hist(want)[0], w.size
