"""The device form of the first order's combinations against the host's (CPU tensors here)."""
import numpy as np
import pytest


@pytest.mark.parametrize("N", [1, 2, 5, 9, 13])
def test_combinations_on_matches_host(N):
    from paper_2501_03381_amd import search
    for k in range(N + 1):
        a, b = search.combinations(N, k), search.combinations_on("cpu", N, k).numpy()
        assert a.dtype == b.dtype and a.shape == b.shape and np.array_equal(a, b), k


@pytest.mark.parametrize("N,k", [(0, 1), (2, 3), (3, 9)])
def test_combinations_on_of_more_than_there_are(N, k):
    from paper_2501_03381_amd import search
    a, b = search.combinations(N, k), search.combinations_on("cpu", N, k).numpy()
    assert a.dtype == b.dtype and a.shape == b.shape == (0, k)


@pytest.mark.parametrize("N,k", [(10, 3), (42, 3), (43, 3), (4, 6)])      # 11,480 and 12,341 rows: either form
def test_first_rows_are_the_combinations(N, k):
    from paper_2501_03381_amd import search
    a, b = search.combinations(N, k), search.first_rows("cpu", N, k).numpy()
    assert a.dtype == b.dtype and np.array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("N,k", [(100, 3), (100, 4)])
def test_combinations_on_the_device(N, k):
    """Realistic sizes, and what is held beside the int32 rows: no more than twice those and 256 MB."""
    import torch
    from paper_2501_03381_amd import search
    print(f"[gpu-case] combinations N={N} k={k}", flush=True)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    b = search.combinations_on("cuda", N, k)
    held = torch.cuda.max_memory_allocated() - before
    assert np.array_equal(search.combinations(N, k), b.cpu().numpy())
    assert held < 2 * 4 * b.numel() + (256 << 20), held
