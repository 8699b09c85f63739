"""The final merge of the streaming reduction at the edges of its selection: fewer segments than
wavefronts, fewer than K, more than one batch of segments, full and partial lists, and values with
many ties (ordered by the lower index).  The lists are an exact selection, so no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def lists(v, K):
    """(values, indices) of the K largest and K smallest, ties by the lower index."""
    i = np.arange(len(v))
    top, bot = np.lexsort((i, -v))[:K], np.lexsort((i, v))[:K]
    return (v[top], top), (v[bot], bot)


# 256 values per segment up to 4096 segments, more beyond
@pytest.mark.parametrize("B", [1, 40, 3 * 256, 9 * 256 + 1, 130 * 256 + 7, 2050 * 256, 4096 * 256 + 300])
@pytest.mark.parametrize("K", [1, 7, 100, 256])
@pytest.mark.parametrize("ties", [False, True])
def test_final_merge_is_an_exact_selection(B, K, ties):
    import torch
    from paper_2501_03381_amd import api
    print(f"[gpu-case] final merge B={B} K={K} ties={ties}", flush=True)
    rng = np.random.default_rng(B + K)
    v = np.round(rng.standard_normal(B), 1) if ties else np.sort(rng.standard_normal(B))
    if B > 100:
        v[rng.integers(0, B, 5)] = np.nan                   # not counted
    st = None
    for part in np.array_split(np.arange(B), 2):            # the second call merges into the first's lists
        x = np.full(B, np.nan)
        x[part] = v[part]
        _, st = api.objective(torch.from_numpy(x[None]).cuda(), "mean", write=False, topk=K, state=st)
    tv, tg, _ = st.result()
    ref = np.where(np.isnan(v), np.nan, v)
    keep = np.nonzero(~np.isnan(ref))[0]
    for l, (val, idx) in enumerate(lists(ref[keep], K)):
        n = len(val)
        assert np.array_equal(tg[0, 0, l, :n], keep[idx]) and np.array_equal(tv[0, 0, l, :n], val)
        assert np.all(tg[0, 0, l, n:] == -1)


def test_equal_values_cost_about_what_distinct_ones_do():
    """Of equal values the lowest indices are kept: the merge must not collect the rest of them (it sorted every
    segment's K entries: 25 times as long as with distinct values)."""
    import torch
    from paper_2501_03381_amd import api
    B, t = 4096 * 256, {}
    for name, v in (("distinct", torch.randn(1, B, dtype=torch.float64, device="cuda")),
                    ("equal", torch.zeros(1, B, dtype=torch.float64, device="cuda"))):
        print(f"[gpu-case] final merge of {name} values", flush=True)
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            api.objective(v, "mean", write=False, topk=100)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        t[name] = best
    assert t["equal"] < 4 * t["distinct"], t


def _time(run):
    import torch
    best = float("inf")
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_many_lists_cost_what_their_evaluation_does():
    """Thousands of datasets, a segment or two per list: a workgroup of 512 threads and 67 KB of LDS for each of 48,000
    lists took 12 times the evaluation (a reduction without lists), one of 256 threads and 21 KB for both lists of a
    pair 5.7 times; the line is halfway."""
    import torch
    from paper_2501_03381_amd import api
    D, N = 4000, 10
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((D, 200, N), dtype=torch.float64, device="cuda", generator=g)
    S = torch.stack([x.t().contiguous() @ x / 199 for x in X])
    kw = dict(orders=(3, 5), hist_bins=64, precision="fp64", check=False)
    print("[gpu-case] many lists", flush=True)
    without = _time(lambda: api.nplets_reduce(S, topk=0, **kw))
    with_lists = _time(lambda: api.nplets_reduce(S, topk=100, **kw))
    assert with_lists < 9 * without, (with_lists, without)


# lists on both sides of the choice between the two forms of the merge, against one dataset at a time
@pytest.mark.parametrize("N,kmin,kmax,D,K", [(12, 3, 12, 3, 100), (13, 4, 6, 230, 7), (16, 5, 9, 160, 64), (9, 3, 9, 1, 256)])
def test_many_lists_are_each_datasets_own(N, kmin, kmax, D, K):
    import torch
    from paper_2501_03381_amd import api
    g = torch.Generator(device="cuda").manual_seed(N)
    X = torch.randn((D, 300, N), dtype=torch.float64, device="cuda", generator=g)
    X[:, :, 2] += X[:, :, 0] + X[:, :, 1]
    S = torch.stack([x.t().contiguous() @ x / 299 for x in X])
    kw = dict(orders=(kmin, kmax), topk=K, hist_bins=0, precision="fp64", engine="factor")
    print(f"[gpu-case] many lists N={N} orders {kmin}..{kmax} D={D} K={K}", flush=True)
    st = api.nplets_reduce(S, **kw)
    for d in {0, 1, D // 2, D - 1} & set(range(D)):
        one = api.nplets_reduce(S[d], **kw)
        assert torch.equal(st.top_g[d], one.top_g[0])
        assert torch.equal(st.top_val[d].nan_to_num(nan=7.0), one.top_val[0].nan_to_num(nan=7.0))
