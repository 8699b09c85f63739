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
