"""The selection kernels at the sizes where their walk changes: edges of tiles, one block or many, a sampled bound or none,
buffers that overflow, costs that a histogram does not tell apart."""
import numpy as np
import pytest


@pytest.fixture(scope="module")
def B():
    from paper_2110_10548_amd import binding
    binding.lib()
    return binding


def _costs(kind, n, rng):
    if kind == "random":
        c = rng.normal(size=n)
        if n > 2:
            c[n // 2], c[n - 1] = -np.inf, np.inf
        return c
    if kind == "ties":
        return np.round(rng.random(n), 2)
    if kind == "falling":
        return np.arange(n, 0, -1).astype(np.float64)
    c = np.zeros(n)                      # nothing but zeros of both signs: the candidate indices decide
    c[::3] = -0.0
    return c


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,kind", [(1, 1, "random"), (65, 64, "ties"), (1023, 1024, "random"), (8192, 7, "random"), (8193, 300, "zeros"),
                                      (16384, 1024, "random"), (16385, 1024, "falling"), (100003, 513, "ties"), (262144, 1024, "random"),
                                      (300001, 128, "zeros"), (4194304, 33, "random"), (4200001, 1000, "falling")])
def test_selection_at_the_edges_of_its_walk(B, n, k, kind):
    import torch
    rng = np.random.default_rng(n + k)
    cost, index = _costs(kind, n, rng), rng.permutation(n).astype(np.int64)
    want = np.lexsort((np.arange(n), index, cost))[:k]
    wide = np.zeros((n, 3))
    wide[:, 2] = cost
    di = torch.from_numpy(index).cuda()
    out = torch.full((min(k, n),), -5, dtype=torch.int64, device="cuda")
    for data, stride, shift in ((cost, 1, 0), (wide, 3, 16)):
        dc = torch.from_numpy(data).cuda()
        for _ in range(2):               # (the second call finds the words that the blocks share as the first one left them)
            B.p2_topk_device(dc.data_ptr() + shift, stride, di.data_ptr(), n, k, out.data_ptr())
            assert np.array_equal(out.cpu().numpy(), want)
        if k <= 64:
            out.fill_(-5)
            B.p2_topk_device_noalloc(dc.data_ptr() + shift, stride, di.data_ptr(), n, k, out.data_ptr())
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.gpu
@pytest.mark.parametrize("topk", [1, 300])
def test_shortlists_are_the_heads_of_the_sorted_lists(B, topk):
    """Both block widths of the per-query selections (few short lists, long lists), several message sizes."""
    links = dict(bw=[25e9, 100e9, 300e9], alpha=[20e-6, 10e-6, 5e-6])
    for card, max_len in (([4, 2, 4], 4), ([2, 4, 8], 5)):
        n = int(np.prod(card))
        q = dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, **links)
        msg = [1e6, 3e7, 5e8]
        full, short = B.p2_synthesize_batch([q], msg)[0], B.p2_synthesize_batch([dict(q, topk=topk)], msg)[0]
        kk = min(topk, len(full["programs"]))
        for m in range(len(msg)):
            want = np.lexsort((full["programs"]["index"], full["cost"][:, m]))[:kk]
            assert np.array_equal(short["programs"]["index"][m * kk:(m + 1) * kk], full["programs"]["index"][want])


@pytest.mark.gpu
def test_shortlists_of_long_lists_in_a_batch(B):
    """Queries with more than 2^18 valid programs: all blocks for one selection after the other, several of them (two
    queries of different length, two message sizes) on one set of lists and shared words."""
    def query(card, max_len, **more):
        n, levels = int(np.prod(card)), len(card)
        return dict(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len,
                         bw=[12.7e9, 30e9, 50.3e9, 151e9, 307e9][-levels:], alpha=[2.3e-5, 1.5e-5, 1.1e-5, 5.7e-6, 1.9e-6][-levels:]), **more)
    msg = [1e6, 5e8]
    asked = [([2, 2, 2, 2], 7, 700), ([2, 2, 2, 2, 2], 6, 9), ([2, 2, 2], 4, 20)]
    full = B.p2_synthesize_batch([query(card, max_len) for card, max_len, _ in asked], msg)
    assert [len(f["programs"]) > 1 << 18 for f in full] == [True, True, False]
    for _ in range(2):                       # (the second call finds the shared words as the first one left them)
        short = B.p2_synthesize_batch([query(card, max_len, topk=k) for card, max_len, k in asked], msg)
        for f, s, (_, _, k) in zip(full, short, asked):
            for m in range(2):
                want = np.lexsort((f["programs"]["index"], f["cost"][:, m]))[:k]
                assert np.array_equal(s["programs"][m * k:(m + 1) * k], f["programs"][want])
                assert np.array_equal(s["cost"][m * k:(m + 1) * k], f["cost"][want])


@pytest.mark.gpu
@pytest.mark.parametrize("topk", [1, 10, 64, 65])
@pytest.mark.parametrize("engine", [0, 3])
def test_shortlists_of_short_lists(B, topk, engine):
    """Lists of at most 512 programs all over the batch: a wavefront each up to 64 kept (a list within a wavefront, of two,
    and one entry alone), wider blocks above.  Equal links and no latency make many costs equal: indices decide."""
    queries = []
    for card, max_len in (([4], 1), ([4], 2), ([2, 4], 3), ([2, 4], 5), ([2, 2, 2, 2], 3)):
        n, levels = int(np.prod(card)), len(card)
        for bw, alpha in (([25e9] * levels, [0.0] * levels), ([25e9, 100e9, 200e9, 300e9][:levels], [20e-6, 10e-6, 5e-6, 2e-6][:levels])):
            queries.append(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, bw=bw, alpha=alpha, engine=engine))
    msg = [1e6, 5e8]
    full, short = B.p2_synthesize_batch(queries, msg), B.p2_synthesize_batch([dict(q, topk=topk) for q in queries], msg)
    assert [len(f["programs"]) for f in full][::2] == [1, 3, 35, 110, 138]
    for f, s in zip(full, short):
        kk = min(topk, len(f["programs"]))
        for m in range(len(msg)):
            want = np.lexsort((f["programs"]["index"], f["cost"][:, m]))[:kk]
            assert np.array_equal(s["programs"][m * kk:(m + 1) * kk], f["programs"][want])
            assert np.array_equal(s["cost"][m * kk:(m + 1) * kk], f["cost"][want])


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,where", [(4_194_304, 33, "skipped"), (4_200_001, 64, "all but k - 1"), (300_001, 64, "all but k - 1"), (20_000, 7, "all but k - 1"),
                                       (5_000, 64, "everywhere"), (4_194_304, 10, "everywhere"), (3_000, 4, "all but k - 1"), (500_000, 3, "all but k - 1"),
                                       (200_000, 10, "skipped"), (40_000, 1, "everywhere")])
def test_nan_costs(B, n, k, where):
    """Columns with a bound from a sample (of every 4 096 entries the first 64), without, and of one block: a NaN is flagged
    wherever it stands and never selected, and the words that the blocks share are left clean."""
    import torch
    rng = np.random.default_rng(n + k)
    clean, index = rng.normal(size=n), rng.permutation(n).astype(np.int64)
    cost = clean.copy()
    if where == "skipped":
        cost[[100, 4_096 + 64, n - 1]] = np.nan
        cost[[64, n - 2]] = -np.inf                       # (and the cheapest ones beside them)
    else:
        keep = rng.choice(n, k - 1 if where == "all but k - 1" else 0, replace=False)
        cost[:] = np.nan
        cost[keep] = clean[keep]
    def head(c):
        ok = np.flatnonzero(c == c)
        want = ok[np.lexsort((ok, index[ok], c[ok]))[:k]]
        return np.concatenate([want, np.full(k - len(want), -1)]).tolist()
    di, dc, good = (torch.from_numpy(a).cuda() for a in (index, cost, clean))
    bad_head, good_head = head(cost), head(clean)
    out, flag = torch.full((k,), -5, dtype=torch.int64, device="cuda"), torch.full((1,), 9, dtype=torch.int32, device="cuda")
    for data, want, nan in ((dc, bad_head, True), (good, good_head, False), (dc, bad_head, True), (good, good_head, False)):
        if nan:
            with pytest.raises(B.P2Error) as e:
                B.p2_topk_device(data.data_ptr(), 1, di.data_ptr(), n, k, out.data_ptr())
            assert e.value.code == B.P2_EINVAL
        else:
            B.p2_topk_device(data.data_ptr(), 1, di.data_ptr(), n, k, out.data_ptr())
            assert out.cpu().tolist() == want
        out.fill_(-5)
        B.p2_topk_device_noalloc(data.data_ptr(), 1, di.data_ptr(), n, k, out.data_ptr(), flag.data_ptr())
        torch.cuda.synchronize()
        assert out.cpu().tolist() == want and int(flag.item()) == int(nan)
        out.fill_(-5)


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,topk", [([2, 2, 2, 2], 3, 1), ([2, 2, 2, 2], 3, 64), ([2, 2, 2, 2], 4, 1), ([2, 2, 2, 2], 4, 256),
                                               ([2, 2, 2, 2], 6, 10), ([2, 2, 2, 2], 6, 1024)])
def test_shortlists_of_equal_costs(B, card, max_len, topk):
    """Every program costs nothing: more ties than the buffers of the three block widths hold (138, 1 646 and 83 920
    programs), in one tile and in several; the candidate indices decide."""
    n = int(np.prod(card))
    q = dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, bw=[25e9] * len(card), alpha=[0.0] * len(card))
    full, short = B.p2_synthesize_batch([q], [0.0, 0.0])[0], B.p2_synthesize_batch([dict(q, topk=topk)], [0.0, 0.0])[0]
    assert len(full["programs"]) == {3: 138, 4: 1646, 6: 83920}[max_len] and not full["cost"].any()
    for m in range(2):
        assert np.array_equal(short["programs"][m * topk:(m + 1) * topk], full["programs"][:topk])


def _few_costs(kind, n, rng):
    if kind == "one lane":               # the smallest ones 64 apart: a lane has all of them
        c = 10.0 + rng.random(n)
        at = np.arange(5, n, 64)
        c[at] = rng.permutation(len(at)) / len(at)
        return c
    return {"rising": np.arange(n, dtype=np.float64), "ties": np.floor(4.0 * rng.random(n)), "equal": np.zeros(n)}.get(kind, rng.normal(size=n))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["random", "rising", "ties", "equal", "one lane"])
@pytest.mark.parametrize("n,k", [(1, 4), (64, 1), (511, 10), (512, 1), (513, 2), (1024, 10), (8193, 4), (32_768, 10), (32_769, 1), (32_769, 10), (40_000, 3),
                                 (262_144, 10), (262_145, 10), (2_100_001, 1), (2_100_001, 4)])
def test_shortlists_of_few_entries(B, n, k, kind):
    """Up to ten entries kept in the lanes of a wavefront: a wavefront, a block and several blocks; columns whose order or
    ties leave nearly every entry below the bounds, with indices that rise, fall and are mixed."""
    import torch
    rng = np.random.default_rng(n + k)
    cost = _few_costs(kind, n, rng)
    dc, out = torch.from_numpy(cost).cuda(), torch.full((min(k, n),), -5, dtype=torch.int64, device="cuda")
    for index in (np.arange(n), np.arange(n, 0, -1), rng.permutation(n) // 2):
        index = index.astype(np.int64)
        want = np.lexsort((np.arange(n), index, cost))[:k].tolist()
        di = torch.from_numpy(index).cuda()
        for call in (B.p2_topk_device, B.p2_topk_device_noalloc, B.p2_topk_device):
            call(dc.data_ptr(), 1, di.data_ptr(), n, k, out.data_ptr())
            torch.cuda.synchronize()
            assert out.cpu().tolist() == want
            out.fill_(-5)
