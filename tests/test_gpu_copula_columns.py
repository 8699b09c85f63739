"""The copula with one workgroup per column (enough columns, T up to the column limit) at the edges of
its sizes and on the values that decide between its two comparisons: continuous values (32-bit codes),
and ties, outliers, infinities and constant columns (full keys).  Ranks are exact, so the scores agree
with the oracle to the rounding of the inverse normal CDF (1e-12 relative to the largest score, as for the
other copula tests)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KINDS = ("normal", "rounded", "constant", "outlier", "infinite", "tiny", "heavy", "zeros", "sorted")


def column(rng, kind, T):
    x = rng.standard_normal(T)
    if kind == "rounded":
        x = np.round(x, 1)
    elif kind == "constant":
        x[:] = 2.5
    elif kind == "outlier":
        x[T // 2] = 1e30
    elif kind == "infinite":
        x[1], x[T - 1] = np.inf, -np.inf
    elif kind == "tiny":
        x *= 1e-310
    elif kind == "heavy":
        x = x / rng.standard_normal(T)
    elif kind == "zeros":
        x[x > 0] = 0.0
        x[::3] = -0.0
    elif kind == "sorted":
        x.sort()
    return x


@pytest.mark.parametrize("T", [1025, 1026, 2048, 2049, 5000, 12287, 12288, 12289])
def test_column_path_matches_oracle(orc, T):
    import torch
    from paper_2501_03381_amd import api
    print(f"[gpu-case] copula columns T={T}", flush=True)
    rng = np.random.default_rng(T)
    D, N = 9, 11                                        # 99 columns
    X = np.stack([np.stack([column(rng, KINDS[(d * N + c) % len(KINDS)], T) for c in range(N)], 1) for d in range(D)])
    Z = api.copulize(torch.from_numpy(X).cuda()).cpu().numpy()
    Z32 = api.copulize(torch.from_numpy(X).cuda(), z_dtype=torch.float32).cpu().numpy()
    for d in range(D):
        ref = orc.copula(X[d])
        tol = 1e-12 * np.abs(ref).max()
        assert np.abs(Z[d] - ref).max() <= tol
        assert np.array_equal(Z32[d], Z[d].astype(np.float32))


def test_column_path_reports_nan(orc):
    import torch
    from paper_2501_03381_amd import api, binding
    print("[gpu-case] copula columns with NaN", flush=True)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((10, 3000, 12))
    X[4, 2999, 7] = np.nan
    with pytest.raises(binding.ThoiError) as e:
        api.copulize(torch.from_numpy(X).cuda())
    assert e.value.status == binding.THOI_EINVAL_DATA
    Z = api.copulize(torch.from_numpy(X).cuda(), check=False).cpu().numpy()
    assert np.all(np.isnan(Z[4, :, 7]))
    ref = orc.copula(X[4][:, :7])
    assert np.abs(Z[4][:, :7] - ref).max() <= 1e-12 * np.abs(ref).max()
    assert np.isfinite(np.delete(Z, 4, 0)).all()


MORE = ("one", "two", "three", "few ties", "integers", "tied and squeezed", "hidden", "two values", "signed zeros", "ramp",
        "plateau")


def more(rng, kind, T):
    """Ties of every share, and equal codes (2^-32 of the range) that are not equal values."""
    x = rng.standard_normal(T)
    if kind in ("one", "two", "three"):
        x = np.round(x, 1 + ("one", "two", "three").index(kind))
    elif kind == "few ties":
        x[rng.random(T) < 0.004] = 0.25
    elif kind == "integers":
        x = np.round(1000 * x) * 3.0
    elif kind == "tied and squeezed":           # half the values tie, the others differ in less than a code
        x = np.where(rng.random(T) < 0.5, 0.0, 1e-11 * x)
        x[3] = 1.0
    elif kind == "hidden":                      # two values beside a heavy tie, which the samples hardly ever meet
        x = np.where(rng.random(T) < 0.3, 0.5, x)
        x[[5, T - 2]] = 0.5 + 1e-12, 0.5 - 1e-12
    elif kind == "two values":
        x = np.where(x > 0, 1e300, -1e300)
    elif kind == "signed zeros":
        x = np.where(rng.random(T) < 0.4, np.where(x > 0, 0.0, -0.0), np.round(x, 2))
    elif kind == "ramp":
        x = np.arange(T) // 7 * 1.0
    elif kind == "plateau":
        x = np.where(np.arange(T) % 5 == 0, x, 3.0)
    return x


@pytest.mark.parametrize("T", [1025, 2048, 2049, 6000, 10000, 12288])
def test_ties_and_shared_codes_match_oracle(orc, T):
    import torch
    from paper_2501_03381_amd import api
    print(f"[gpu-case] copula ties T={T}", flush=True)
    rng = np.random.default_rng(T + 1)
    D, N = 14, 11                                       # 154 columns, every kind in every dataset
    X = np.stack([np.stack([more(rng, k, T) for k in MORE], 1) for _ in range(D)])
    Z = api.copulize(torch.from_numpy(X).cuda()).cpu().numpy()
    for d in range(0, D, 3):
        ref = orc.copula(X[d])
        assert np.abs(Z[d] - ref).max() <= 1e-12 * np.abs(ref).max()
    # against the other path, for all of them: one dataset at a time is too few columns for this one
    for d in range(D):
        assert np.array_equal(Z[d], api.copulize(torch.from_numpy(X[d]).cuda()).cpu().numpy())


def test_more_columns_nan():
    import torch
    from paper_2501_03381_amd import api
    rng = np.random.default_rng(8)
    X = np.round(rng.standard_normal((16, 3000, 9)), 1)
    assert torch.isfinite(api.copulize(torch.from_numpy(X).cuda())).all()
    X[15, 2999, 8] = np.nan
    with pytest.raises(api.B.ThoiError):
        api.copulize(torch.from_numpy(X).cuda())


def test_ties_cost_about_what_distinct_values_do():
    """Rounded columns take 1.1 times the time of continuous ones, and took 2.05 times it with full
    keys for every tied column: the line lies halfway."""
    import torch
    from paper_2501_03381_amd import api
    X = torch.randn((64, 10000, 20), device="cuda", dtype=torch.float64, generator=torch.Generator("cuda").manual_seed(1))
    times = []
    for x in (X, (10 * X).round() / 10):
        best = float("inf")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            api.copulize(x)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"[gpu-case] copula continuous / tied ms: {times}", flush=True)
    assert times[1] < 1.55 * times[0]
