"""The selection entry point that allocates nothing, against the allocating one (and the oracle)."""
import numpy as np
import pytest

from paper_2110_10548_amd import workloads


@pytest.fixture(scope="module")
def B():
    from paper_2110_10548_amd import binding
    binding.lib()
    return binding


def _inputs(seed, n, torch):
    rng = workloads.SplitMix64(seed)
    cost = np.array([rng.below(997) / 8.0 for _ in range(n)], dtype=np.float64)          # many ties
    index = np.array([rng.next_u64() >> 16 for _ in range(n)], dtype=np.uint64)
    return cost, index, torch.from_numpy(cost).cuda(), torch.from_numpy(index.view(np.int64)).cuda()


@pytest.mark.gpu
def test_topk_without_allocation_matches_the_allocating_call(B, oracle):
    import torch
    nan = torch.zeros(1, dtype=torch.int32, device="cuda")
    # two calls in a row on the same fixed scratch, the second smaller (fewer stage-1 lists, shorter lists)
    for seed, n, k in ((11, 300_007, 64), (12, 4_099, 10), (13, 50, 64)):
        cost, index, dc, di = _inputs(seed, n, torch)
        kk = min(k, n)
        ref = torch.full((kk,), -7, dtype=torch.int64, device="cuda")
        got = torch.full((kk,), -7, dtype=torch.int64, device="cuda")
        B.p2_topk_device(dc.data_ptr(), 1, di.data_ptr(), n, k, ref.data_ptr())
        free_before = torch.cuda.mem_get_info()[0]
        B.p2_topk_device_noalloc(dc.data_ptr(), 1, di.data_ptr(), n, k, got.data_ptr(), nan.data_ptr())
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free_before
        assert got.cpu().tolist() == ref.cpu().tolist() == oracle.topk(cost, index, k).tolist()
        assert int(nan.item()) == 0
    # a NaN is flagged on the device and left out of the list
    cost, index, dc, di = _inputs(14, 1000, torch)
    dc[17] = float("nan")
    got = torch.full((5,), -7, dtype=torch.int64, device="cuda")
    B.p2_topk_device_noalloc(dc.data_ptr(), 1, di.data_ptr(), 1000, 5, got.data_ptr(), nan.data_ptr())
    torch.cuda.synchronize()
    cost[17] = np.inf
    assert int(nan.item()) == 1 and got.cpu().tolist() == oracle.topk(cost, index, 5).tolist()
    # strided costs, no flag word
    cost, index, dc, di = _inputs(15, 2048, torch)
    wide = torch.zeros((2048, 3), dtype=torch.float64, device="cuda")
    wide[:, 1] = dc
    got = torch.full((8,), -7, dtype=torch.int64, device="cuda")
    B.p2_topk_device_noalloc(wide.data_ptr() + 8, 3, di.data_ptr(), 2048, 8, got.data_ptr())
    torch.cuda.synchronize()
    assert got.cpu().tolist() == oracle.topk(cost, index, 8).tolist()
    with pytest.raises(B.P2Error) as e:
        B.p2_topk_device_noalloc(dc.data_ptr(), 1, di.data_ptr(), 2048, 65, got.data_ptr())
    assert e.value.code == B.P2_EUNSUPPORTED


@pytest.mark.gpu
def test_calls_that_overlap_stay_inside_their_buffers(B, oracle):
    """Calls on several streams share one scratch and race, which the header rules out; what they write all the same are
    positions of their own columns or -1, and the next call alone is right."""
    import torch
    n, k = 1_000_003, 64                        # (123 blocks, up to 320 entries each: three calls' entries exceed the lists)
    _, _, dc, di = _inputs(16, n, torch)
    # columns that fall: every block keeps more than it may leave uncut
    falls = torch.arange(n, 0, -1, dtype=torch.float64, device="cuda")
    sizes = (n, 300_007, 700_001, n)
    outs = [torch.full((k,), 1 << 40, dtype=torch.int64, device="cuda") for _ in sizes]
    streams = [torch.cuda.Stream() for _ in sizes]
    torch.cuda.synchronize()
    for i, (m, st) in enumerate(zip(sizes, streams)):
        B.p2_topk_device_noalloc((dc if i == 1 else falls).data_ptr(), 1, di.data_ptr(), m, k, outs[i].data_ptr(), stream=st.cuda_stream)
    torch.cuda.synchronize()
    for m, out in zip(sizes, outs):
        got = out.cpu().numpy()
        assert ((got >= -1) & (got < m)).all()
    cost, index, dc, di = _inputs(17, 4_099, torch)
    out = torch.full((10,), -7, dtype=torch.int64, device="cuda")
    B.p2_topk_device_noalloc(dc.data_ptr(), 1, di.data_ptr(), 4_099, 10, out.data_ptr())
    torch.cuda.synchronize()
    assert out.cpu().tolist() == oracle.topk(cost, index, 10).tolist()


@pytest.mark.gpu
@pytest.mark.parametrize("n,k", [(3_000, 4), (300_007, 3), (20_011, 64), (4_300_003, 64)])
def test_recorded_into_a_graph(B, oracle, n, k):
    """One block and several, a few entries and more, with a bound from a sample: every replay, on other inputs and with eager
    calls in between, gives what the eager call gives."""
    import torch
    rng = np.random.default_rng(n)

    def inputs():
        return torch.from_numpy(rng.integers(0, 997, n) / 8.0).cuda(), torch.from_numpy(rng.integers(0, 1 << 40, n)).cuda()

    dc, di = inputs()
    out, nan = torch.full((k,), -7, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    eager = torch.full((k,), -7, dtype=torch.int64, device="cuda")

    def call(into, flag):
        B.p2_topk_device_noalloc(dc.data_ptr(), 1, di.data_ptr(), n, k, into.data_ptr(), flag, stream=torch.cuda.current_stream().cuda_stream)

    call(eager, None)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out, nan.data_ptr())
    for replay in range(4):
        c, i = inputs()
        dc.copy_(c)
        di.copy_(i)
        if replay == 2:
            dc[n // 2] = float("nan")
        out.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert int(nan.item()) == int(replay == 2)
        call(eager, None)
        torch.cuda.synchronize()
        cost = dc.cpu().numpy()
        cost[cost != cost] = np.inf
        assert out.cpu().tolist() == eager.cpu().tolist() == oracle.topk(cost, di.cpu().numpy().view(np.uint64), k).tolist()
