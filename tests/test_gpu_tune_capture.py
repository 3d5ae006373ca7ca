"""The parameter search waits for its stream, which a capture cannot: refused, and the capture goes on as if it had not been asked."""
import numpy as np
import pytest

from paper_2604_03298_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_a_search_inside_a_capture_is_refused_and_leaves_the_graph_alone(oracle):
    import torch
    from paper_2604_03298_amd import enec
    t = W.gaussian(9 * 16384 + 77, 0.02, 61)
    prm = oracle.tune(t)
    want = oracle.compress(t, prm, 16384)[1]
    src = torch.from_numpy(t.view(np.int16)).cuda()
    out = torch.zeros(enec.compress_bound(t.size), dtype=torch.uint8, device="cuda")
    ws = enec.new_workspace(t.size)
    assert enec.compress(src, prm, out, ws) == 0          # (the occupancy figure is looked up)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(torch.cuda.Stream()):
        graph.capture_begin()
        with pytest.raises(enec.EnecError) as e:
            enec.tune(src, ws)
        assert e.value.status == enec.E_HIP
        assert enec.compress(src, None, out, ws) == enec.E_HIP       # tunes first
        assert enec.compress(src, prm, out, ws) == 0
        graph.capture_end()
    torch.cuda.synchronize()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out[:want.size].cpu().numpy(), want)
        assert enec.tune(src, ws) == prm
