"""The device annealer across the edges of its launches (many iterations per launch, 256 at most; chains two
per wavefront, one to four wavefronts per workgroup, an odd last chain) and of the factorisation's order
classes (8, 16, 24, 32, and one wavefront per chain above), against the host-driven loop: the same states,
acceptance counts and, to 1e-9 (the FP64 tolerance of the other search tests), values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kappa,iters,k_lo,k_hi,mode", [
    (12, 1, 1, 3, 3, "within"), (20, 3, 257, 8, 9, "across"), (40, 7, 60, 15, 17, "within"),
    (50, 6, 60, 24, 25, "within"), (90, 5, 40, 31, 32, "across"), (80, 4, 30, 33, 40, "within"),
    (24, 1027, 20, 3, 6, "within"), (24, 2051, 5, 3, 6, "across"), (128, 9, 20, 5, 12, "across")])
def test_device_annealer_matches_host_loop(N, kappa, iters, k_lo, k_hi, mode):
    import torch
    from paper_2501_03381_amd import search, synth
    print(f"[gpu-case] anneal N={N} kappa={kappa} iters={iters} orders {k_lo}..{k_hi} {mode}", flush=True)
    X = synth.factor_model(np.random.default_rng(N), 3000, N, 5)
    S = torch.from_numpy(np.cov(X.T)).cuda()
    m0 = synth.sa_initial(1, kappa, N, k_lo, k_hi)
    dr = synth.sa_draws(2, iters, kappa)
    kw = dict(T0=0.3, alpha=0.99, mode=mode, k_min=min(3, k_lo), k_max=None if mode == "within" else min(k_hi, N - 1))
    for maximize in (True, False):
        a = search.anneal(S, m0, dr, maximize=maximize, on_device=True, **kw)
        b = search.anneal(S, m0, dr, maximize=maximize, on_device=False, **kw)
        for i in (0, 2, 4):
            assert np.array_equal(a[i], b[i]), i
        for i in (1, 3):
            assert np.abs(a[i] - b[i]).max() <= 1e-9
