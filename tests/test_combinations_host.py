"""The device form of the first order's combinations against the host's (CPU tensors here)."""
import numpy as np
import pytest


@pytest.mark.parametrize("N", [1, 2, 5, 9, 13])
def test_combinations_on_matches_host(N):
    from paper_2501_03381_amd import search
    for k in range(N + 1):
        a, b = search.combinations(N, k), search.combinations_on("cpu", N, k).numpy()
        assert a.dtype == b.dtype and a.shape == b.shape and np.array_equal(a, b), k
