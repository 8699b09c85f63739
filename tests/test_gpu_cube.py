"""Subset-table engine of whole-order reductions (FP64: 21..30 variables, FP32 with refinement: 26..30) against
one factorisation per n-plet (engine="factor"): the table only decides where the factorisation cannot differ,
so values, indices, counts and flags are the same bit for bit."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2501_03381_amd import api, binding, synth
    return torch, api, binding, synth


def sigma(torch, synth, N, D, seed=0):
    rng = np.random.default_rng(1000 * N + seed)
    return torch.from_numpy(np.stack([np.cov(synth.factor_model(rng, 3000, N, 5).T) for _ in range(D)])).cuda()


def both(api, S, kmin, kmax, **kw):
    r = [api.nplets_reduce(S, orders=(kmin, kmax), precision="fp64", engine=e, **kw).result() for e in ("factor", "auto")]
    return r


def same(a, b):
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
    assert np.array_equal(a[0], b[0], equal_nan=True)


# orders that start or end inside a row, a single order, every order, several datasets
@pytest.mark.parametrize("N,kmin,kmax,D,K,bins", [
    (21, 3, 21, 1, 100, 256), (21, 3, 14, 2, 1, 16), (25, 12, 12, 1, 256, 8), (22, 3, 22, 3, 64, 64),
    (22, 12, 22, 1, 65, 0), (23, 3, 11, 1, 0, 4096), (24, 3, 24, 1, 7, 32)])
def test_cube_matches_factorisation(env, N, kmin, kmax, D, K, bins):
    torch, api, B, synth = env
    print(f"[gpu-case] cube N={N} orders {kmin}..{kmax} D={D} K={K} bins={bins}", flush=True)
    S = sigma(torch, synth, N, D)
    kw = dict(topk=K, hist_bins=bins, hist_range=(-7.3, 5.1))
    a, b = both(api, S, kmin, kmax, **kw)
    if K == 0:
        a, b = [(np.zeros(1), np.zeros(1), x[2]) for x in (a, b)]
    if bins == 0:
        a, b = [(x[0], x[1], np.zeros(1)) for x in (a, b)]
    same(a, b)


def test_cube_bias_flags_and_not_positive_definite(env):
    torch, api, B, synth = env
    N = 21
    S = sigma(torch, synth, N, 1)
    S[0, 3, 18] = S[0, 18, 3] = 2.0 * torch.sqrt(S[0, 3, 3] * S[0, 18, 18])   # every superset of {3, 18} fails
    n = B.thoi_count(N, 3, N)
    fl = [torch.zeros((1, n), dtype=torch.uint8, device="cuda") for _ in range(2)]
    r = []
    for e, f in zip(("factor", "auto"), fl):
        print(f"[gpu-case] cube not positive definite, bias, {e}", flush=True)
        r.append(api.nplets_reduce(S, orders=(3, N), precision="fp64", engine=e, topk=20, hist_bins=32,
                                   hist_range=(-7.3, 5.1), bias_correct=True, T=500, flags=f).result())
    same(*r)
    assert torch.equal(fl[0], fl[1]) and int((fl[1] == B.THOI_NPLET_NOT_PD).sum()) == 2 ** (N - 2) - 1


def test_cube_accumulates_and_takes_the_least_workspace(env):
    torch, api, B, synth = env
    N = 21
    S = sigma(torch, synth, N, 2, 1)
    sel = api.range_selection(N, 3, N)
    res = []
    for full in (False, True):
        print(f"[gpu-case] cube workspace full={full}", flush=True)
        st = api.ReduceState(1, N, 30, 64, (-7.3, 5.1), S.device)
        o = api.make_opts("fp64", torch.float32)
        o.reduce = ctypes.pointer(st.struct)
        least = B.thoi_workspace_bytes(B.THOI_WS_EVAL, 1, 0, N, sel, o)
        most = B.thoi_eval_workspace_bytes_full(1, N, sel, o)
        assert most > least + (8 << N) // 2
        ws = torch.empty(most if full else least, dtype=torch.uint8, device="cuda")
        for d in range(2):                       # the second call merges into the lists of the first
            B.thoi_nplets_eval(api._ptr(S[d].contiguous()), 1, N, sel, o, None, None, api._ptr(ws), ws.numel(),
                               api._stream(S.device))
        torch.cuda.synchronize()
        assert api.device_status(ws) == B.THOI_OK
        res.append(st.result())
    same(*res)


# FP32 with refinement: FP64 decides only where FP32 cannot differ, so everything is the lane engine's bit for bit
@pytest.mark.parametrize("kmin,kmax,K,bins,near,sym", [
    (3, 13, 100, 256, False, False), (3, 14, 256, 4096, True, False), (5, 26, 7, 0, False, False),
    (3, 26, 0, 64, False, False), (4, 12, 20, 16, False, True)])
def test_filtered_fp32_is_the_lane_engine_bit_for_bit(env, kmin, kmax, K, bins, near, sym):
    torch, api, B, synth = env
    N = 26
    rng = np.random.default_rng(kmax)
    X = synth.factor_model(rng, 2000, N, 6)
    if near:
        X[:, 20] = X[:, 3] + 0.03 * rng.standard_normal(2000)     # VIFs on both sides of the threshold
    S = torch.from_numpy(np.cov(X.T)).cuda()
    if sym:                                                       # every n-plet of an order ties
        S = torch.full((N, N), 0.25, dtype=torch.float64, device="cuda") + 0.75 * torch.eye(N, dtype=torch.float64, device="cuda")
    n = B.thoi_count(N, kmin, kmax)
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] fp32 cube orders {kmin}..{kmax} K={K} bins={bins} near={near} sym={sym} {e}", flush=True)
        f = torch.full((1, n), 9, dtype=torch.uint8, device="cuda")
        st = api.nplets_reduce(S, orders=(kmin, kmax), topk=K, hist_bins=bins, hist_range=(-7.3, 5.1), engine=e, flags=f,
                               bias_correct=near, T=400 if near else 0, check=not near)
        res.append(([st.top_val, st.top_g] if K else []) + ([st.hist] if bins else []) + [f])
    for x, y in zip(*res):
        assert torch.equal(torch.nan_to_num(x.double(), nan=77.0), torch.nan_to_num(y.double(), nan=77.0))
    if near:
        assert 0 < int((res[0][-1] == B.THOI_NPLET_REFINED).sum()) < n


# from 29 variables on the rows go in several blocks, each evaluated beside the next one's filter
@pytest.mark.parametrize("prec,kmin,kmax", [("fp64", 4, 13), ("fp32_refine", 3, 14)])
def test_blocks_of_rows(env, prec, kmin, kmax):
    torch, api, B, synth = env
    S = torch.from_numpy(np.cov(synth.factor_model(np.random.default_rng(29), 2000, 29, 6).T)).cuda()
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] blocks {prec} orders {kmin}..{kmax} {e}", flush=True)
        st = api.nplets_reduce(S, orders=(kmin, kmax), topk=50, hist_bins=100, hist_range=(-6, 6), engine=e, precision=prec)
        res.append((st.top_val, st.top_g, st.hist))
    for x, y in zip(*res):
        assert torch.equal(torch.nan_to_num(x.double(), nan=77.0), torch.nan_to_num(y.double(), nan=77.0))


def test_exchangeable_variables_tie_by_index(env):
    """Equal sub-matrices give equal values: of a compound-symmetric matrix every n-plet of an order ties, so
    the lists are the first indices of the order."""
    torch, api, B, synth = env
    N = 21
    S = torch.full((1, N, N), 0.25, dtype=torch.float64, device="cuda") + 0.75 * torch.eye(N, dtype=torch.float64, device="cuda")
    print("[gpu-case] cube ties", flush=True)
    tv, tg, h = api.nplets_reduce(S, orders=(3, N), precision="fp64", topk=10, hist_bins=16, hist_range=(-7.3, 5.1)).result()
    g = 0
    for k in range(3, N + 1):
        n = B.thoi_count(N, k, k)
        m = min(n, 10)
        for l in range(2):
            assert np.array_equal(tg[0, k, l, :m], np.arange(g, g + m)) and len(set(tv[0, k, l, :m])) == 1
        assert h[0, k].max() == n == h[0, k].sum()
        g += n


def timed(torch, run, n=5):
    run()
    best = float("inf")
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def ar1(torch, N, rho):
    i = torch.arange(N, dtype=torch.float64, device="cuda")
    return rho ** (i[:, None] - i[None]).abs()


def bits(st, *more):
    return [torch_nan(st.top_val), st.top_g, st.hist, *more]


def torch_nan(x):
    return x.nan_to_num(nan=77.0)


# strong autocorrelation, or bins as narrow as FP32's error: most n-plets stay open beside the table, which
# then costs its own time (a quarter of the call) and that of the separate evaluation; the margin of a third
# is for a box's noise
@pytest.mark.parametrize("rho,bins,width", [(0.99, 4096, 4.0), (0.9, 4096, 1.0), (0.999, 0, 1.0)])
def test_open_nplets_do_not_make_the_call_slower(env, rho, bins, width):
    torch, api, B, synth = env
    N = 26
    S = ar1(torch, N, rho)
    t, res = {}, {}
    for e in ("factor", "auto"):
        print(f"[gpu-case] cube open share rho={rho} bins={bins} {e}", flush=True)
        kw = dict(orders=(3, N), topk=100, hist_bins=bins, hist_range=(-width, width), engine=e)
        res[e] = api.nplets_reduce(S, **kw)
        t[e] = timed(torch, lambda: api.nplets_reduce(S, check=False, **kw))
    for x, y in zip(bits(res["factor"])[:3 if bins else 2], bits(res["auto"])):
        assert torch.equal(x, y)
    assert t["auto"] < 1.33 * t["factor"], t


def test_datasets_choose_for_themselves(env):
    """FP32, several datasets in one call: an easy one, one for the factorisation and one with VIFs around the
    refinement threshold; every order, flags and device status."""
    torch, api, B, synth = env
    N, D = 26, 4
    rng = np.random.default_rng(5)
    X = synth.factor_model(rng, 2000, N, 6)
    Y = X.copy()
    Y[:, 20] = Y[:, 3] + 0.03 * rng.standard_normal(2000)
    S = torch.stack([torch.from_numpy(np.cov(X.T)).cuda(), ar1(torch, N, 0.99), torch.from_numpy(np.cov(Y.T)).cuda(),
                     torch.from_numpy(np.cov(X[:900].T)).cuda()]).contiguous()
    n = B.thoi_count(N, 3, N)
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] cube FP32 D={D} {e}", flush=True)
        f = torch.full((D, n), 9, dtype=torch.uint8, device="cuda")
        st = api.nplets_reduce(S, orders=(3, N), topk=33, hist_bins=1024, hist_range=(-7.3, 5.1), engine=e, flags=f)
        res.append(bits(st, f))
    for x, y in zip(*res):
        assert torch.equal(x, y)
    refined = (res[1][-1] == B.THOI_NPLET_REFINED).sum(1).tolist()
    assert refined[0] == refined[1] == refined[3] == 0 and 0 < refined[2] < n


def near_singular(torch, synth, N, noise):
    """A channel recorded twice up to `noise`: half of its n-plets are singular to working precision."""
    rng = np.random.default_rng(77)
    X = synth.factor_model(rng, 3000, N, 5)
    X[:, N - 1] = X[:, 2] + noise * rng.standard_normal(3000)
    X[:, 12] = X[:, 5] + noise * rng.standard_normal(3000)
    return torch.from_numpy(np.cov(X.T)).cuda()


# whether a pivot near the rounding of 1 is positive is the factorisation's to say, also where the bins are so wide
# that Omega's place among them is certain
@pytest.mark.parametrize("noise", [1e-7, 2e-8, 1e-9])
@pytest.mark.parametrize("bins,topk", [(4, 0), (16, 20)])
def test_singular_to_working_precision_fp64(env, noise, bins, topk):
    torch, api, B, synth = env
    N = 21
    S = near_singular(torch, synth, N, noise)
    n = B.thoi_count(N, 3, N)
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] cube near singular noise={noise} bins={bins} topk={topk} {e}", flush=True)
        f = torch.full((1, n), 9, dtype=torch.uint8, device="cuda")
        st = api.nplets_reduce(S, orders=(3, N), precision="fp64", topk=topk, hist_bins=bins, hist_range=(-1e9, 1.6e9),
                               engine=e, flags=f)
        res.append([f] + ([st.hist] if bins else []) + ([torch_nan(st.top_val), st.top_g] if topk else []))
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.parametrize("tau,noise", [(1e5, 3e-3), (1e6, 1e-3), (1e8, 1e-6), (1e8, 1e-5)])
def test_thresholds_at_the_precision_of_fp32(env, tau, noise):
    """A refinement threshold where FP32 cannot resolve the VIF: what the table holds above it the FP32
    factorisation may hold below, so that n-plet is evaluated, not queued on the table's word."""
    torch, api, B, synth = env
    N, kmin, kmax = 26, 3, 12
    rng = np.random.default_rng(8)
    X = synth.factor_model(rng, 4000, N, 6)
    X[:, 20] = X[:, 3] + noise * rng.standard_normal(4000)
    S = torch.from_numpy(np.cov(X.T)).cuda()
    n = B.thoi_count(N, kmin, kmax)
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] cube tau={tau} noise={noise} {e}", flush=True)
        f = torch.full((1, n), 9, dtype=torch.uint8, device="cuda")
        st = api.nplets_reduce(S, orders=(kmin, kmax), topk=100, hist_bins=64, hist_range=(-30, 30), engine=e, flags=f,
                               vif_tau=tau)
        res.append((f, st.top_g, st.hist, torch.nan_to_num(st.top_val, nan=77.0)))
    for x, y in zip(*res):
        assert torch.equal(x, y)


# more datasets than tables at a time, and every order of the largest system in several blocks of rows
@pytest.mark.parametrize("prec,N,kmin,kmax,D,K", [("fp64", 25, 3, 25, 2, 100), ("fp32_refine", 29, 3, 14, 2, 40),
                                                  ("fp64", 29, 4, 15, 2, 256), ("fp64", 30, 3, 30, 1, 100)])
def test_groups_of_tables_and_blocks_of_rows(env, prec, N, kmin, kmax, D, K):
    torch, api, B, synth = env
    S = sigma(torch, synth, N, D, 2)
    res = []
    for e in ("factor", "auto"):
        print(f"[gpu-case] cube groups {prec} N={N} orders {kmin}..{kmax} D={D} {e}", flush=True)
        res.append(bits(api.nplets_reduce(S, orders=(kmin, kmax), topk=K, hist_bins=100, hist_range=(-6, 6), engine=e,
                                          precision=prec)))
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.parametrize("prec,N", [("fp64", 22), ("fp32_refine", 26)])
def test_table_in_a_graph(env, prec, N):
    torch, api, B, synth = env
    S = sigma(torch, synth, N, 1, 3)
    if prec == "fp32_refine":
        S = torch.stack([S[0], ar1(torch, N, 0.99)]).contiguous()
    D = S.shape[0]
    sel = api.range_selection(N, 3, N)
    st = api.ReduceState(D, N, 50, 128, (-7.3, 5.1), S.device)
    o = api.make_opts(prec, torch.float32)
    o.reduce = ctypes.pointer(st.struct)
    ws = torch.empty(B.thoi_eval_workspace_bytes_full(D, N, sel, o), dtype=torch.uint8, device="cuda")

    def call():
        B.thoi_reduce_init(st.struct, D, N, api._stream(S.device))
        B.thoi_nplets_eval(api._ptr(S), D, N, sel, o, None, None, api._ptr(ws), ws.numel(), api._stream(S.device))

    print(f"[gpu-case] cube graph {prec} N={N}", flush=True)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for i in range(4):
        S.copy_(S.flip(1).flip(2).contiguous() if i % 2 else S * (1.0 + 0.5 * i))
        ref = api.nplets_reduce(S, orders=(3, N), topk=50, hist_bins=128, hist_range=(-7.3, 5.1), precision=prec,
                                engine="factor")
        g.replay()
        torch.cuda.synchronize()
        assert api.device_status(ws) == B.THOI_OK
        for x, y in zip(bits(ref), bits(st)):
            assert torch.equal(x, y)


def test_table_on_streams_of_several_threads(env):
    import threading
    torch, api, B, synth = env
    N = 22
    S = [sigma(torch, synth, N, 1, 10 + i) for i in range(3)]
    kw = dict(orders=(3, N), topk=50, hist_bins=64, hist_range=(-7.3, 5.1), precision="fp64")
    ref = [bits(api.nplets_reduce(s, engine="factor", **kw)) for s in S]
    torch.cuda.synchronize()
    got, err = [[] for _ in S], []
    print("[gpu-case] cube threads", flush=True)

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    got[i].append(bits(api.nplets_reduce(S[i], **kw)))
                torch.cuda.current_stream().synchronize()
        except Exception as e:                   # reported by the test's own thread
            err.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(len(S))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not err, err
    for r, runs in zip(ref, got):
        assert len(runs) == 4
        for run in runs:
            for x, y in zip(r, run):
                assert torch.equal(x, y)


def test_no_memory_for_the_table(env, monkeypatch):
    """A device without the memory for the table: the call takes its least workspace, same results."""
    torch, api, B, synth = env
    N = 21
    S = sigma(torch, synth, N, 1, 4)
    kw = dict(orders=(3, N), topk=30, hist_bins=64, hist_range=(-7.3, 5.1), precision="fp64")
    a = bits(api.nplets_reduce(S, **kw))
    asked, plain = [], api._workspace

    def small(nbytes, device):
        asked.append(int(nbytes))
        if len(asked) == 1:
            raise torch.OutOfMemoryError("no room")
        return plain(nbytes, device)

    monkeypatch.setattr(api, "_workspace", small)
    print("[gpu-case] cube without memory", flush=True)
    b = bits(api.nplets_reduce(S, **kw))
    assert len(asked) == 2 and asked[1] < asked[0]
    for x, y in zip(a, b):
        assert torch.equal(x, y)
