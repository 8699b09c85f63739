"""FP32 output of several datasets' low orders goes through a wavefront's buffer and its n-plets are unranked by
bisection; FP64 output of the same FP32 evaluation is stored by each lane, unranked step by step.  One arithmetic,
so the two agree bit for bit (the entropy after its one rounding to FP32)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# datasets smaller than the order, one n-plet, partial and full rows of 64 x 12, unranking above and below 33
# variables, the largest dataset; orders of this class alone and together with larger ones; every option
@pytest.mark.parametrize("Ns,kmin,kmax,prec,entropy,bias", [
    ([3, 2, 8, 9, 10, 25, 1, 12, 17, 25], 1, 8, "fp32_refine", True, True),
    ([5, 40, 33, 34, 32, 31, 10, 5, 5, 40, 39, 40, 40, 40], 3, 5, "fp32_refine", False, False),
    ([62, 61, 3, 33, 62, 62, 60, 62, 62], 2, 4, "fp32", True, False),
    ([14, 15, 16, 20, 27, 20, 20], 7, 9, "fp32_refine", False, True),
    ([20, 24, 8, 25, 25, 25], 8, 8, "fp32", False, False),
    ([7, 31], 0, 7, "fp32_refine", True, False),
    ([7, 12, 20], 0, 7, "fp32_refine", True, False)])          # too few for the buffer
def test_staged_output_is_the_lane_output(Ns, kmin, kmax, prec, entropy, bias):
    import torch
    from paper_2501_03381_amd import api, synth
    rng = np.random.default_rng(kmax)
    Ss = []
    for N in Ns:
        X = synth.factor_model(rng, 400, N, min(N, 3))
        if N > 4:
            X[:, 4] = X[:, 0] + 0.02 * rng.standard_normal(400)    # some VIFs above the threshold
        if N > 9:
            X[:, 9] = X[:, 1]                                      # some n-plets not positive definite
        Ss.append(torch.from_numpy(np.atleast_2d(np.cov(X.T))).cuda())
    T_d = np.full(len(Ns), 400, dtype=np.int32) if bias else None
    print(f"[gpu-case] staged {Ns} orders {kmin}..{kmax} {prec} entropy={entropy} bias={bias}", flush=True)
    flat, n = api.pack_covariances(Ss)
    res = []
    for odt in (torch.float32, torch.float64):
        ev = api.MultiEvaluator(n, kmin, kmax, flat.device, prec, odt, T_d, bias, entropy)
        ev.out.fill_(-3.0)
        ev.flags.fill_(9)
        out, flags = ev(flat)
        api.raise_on_device_status(ev.ws, "multi")
        res.append((out.float().clone(), flags.clone()))
    (a, fa), (b, fb) = res
    refined = ((fa & 1) != 0) if prec == "fp32_refine" else torch.zeros_like(fa, dtype=torch.bool)
    assert torch.equal(fa, fb)
    assert torch.equal(torch.isnan(a), torch.isnan(b))
    assert torch.equal(torch.nan_to_num(a), torch.nan_to_num(b))
    assert len(fa) == 0 or bool(refined.any()) or prec == "fp32" or max(Ns) < 5
