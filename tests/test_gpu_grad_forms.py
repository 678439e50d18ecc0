"""FP64 gradients at the edges of their dispatch: 1024 blocks of 16 particles, from which each wave
of a workgroup takes its own block (every row width), and 2049 particles, from which the pass that
combines the ranges takes four coefficients per lane (16, 32 and 64 lanes per row); first and last
rows against the oracle (1e-10 of sum_k |X_kj| per element and of the log posterior), and the whole
against the same particles in two halves, which take the other form.  And products of prior factors
that overflow (a tiny scale with ordinary coefficients), whose logs are then added one by one."""
import numpy as np
import pytest

from oracle import gt_prior, likelihood
from tests.gpu_util import dataset, particles

pytestmark = pytest.mark.gpu


def _handle(n, p, prec="fp64"):
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    cfg, X, y, Xs = dataset("n2000_p50_rwm_fp32", n, p)
    return SpaSMC(SamplerConfig(n=n, p=p, N=64, a=1.0, lambdas=np.geomspace(10, 1, 2), move="rwm", sweeps=0,
                                init_sweeps=0, prec=prec, seed=0), X, y), X, y, Xs


@pytest.mark.parametrize("n,p,M", [(40, 10, 16368), (40, 10, 16369), (66, 30, 16385), (50, 60, 16447), (80, 120, 16369),
                                   (34, 200, 16385), (48, 250, 16447), (200, 250, 16368),
                                   (300, 10, 2049), (300, 64, 2049), (300, 65, 2050), (300, 129, 2049), (300, 255, 2048)])
def test_fp64_gradient_forms(n, p, M):
    import torch
    s, X, y, Xs = _handle(n, p)
    b = particles(M, p, seed=n + p)
    bt = torch.from_numpy(b).cuda()
    lam = 0.3
    print(f"FP64 gradient n={n} p={p} M={M}", flush=True)
    g, lp = (v.cpu().numpy() for v in s.grad(bt, lam, "fp64"))
    rows = np.unique(np.r_[0:40, M // 2 - 20:M // 2 + 20, M - 70:M])
    ll, gl = likelihood.loglik_and_grad(b[rows], Xs, y)
    tol = 1e-10 * np.abs(Xs).sum(axis=0)
    assert np.all(np.abs(g[rows] - gl - gt_prior.gt_grad(b[rows], 1.0, lam)) <= tol)
    lref = ll + gt_prior.log_prior(b[rows], 1.0, lam)
    assert np.all(np.abs(lp[rows] - lref) <= 1e-10 * (np.abs(ll) + np.abs(lref)))
    h = M // 2
    for part in (slice(0, h), slice(h, M)):
        g2, lp2 = (v.cpu().numpy() for v in s.grad(bt[part].contiguous(), lam, "fp64"))
        assert np.all(np.abs(g2 - g[part]) <= tol)
        assert np.all(np.abs(lp2 - lp[part]) <= 1e-10 * (np.abs(lp2) + n))
    s.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x2"])
@pytest.mark.parametrize("p,M", [(40, 2049), (100, 2100), (200, 2049), (17, 30)])
def test_prior_factors_beyond_the_double_range(p, M, prec):
    import torch
    n = 600
    s, X, y, Xs = _handle(n, p)
    lam = 1e-100                                  # 1 + |b| / (a lam) near 1e99: four of them overflow
    b = particles(M, p, seed=p)
    b[0] = 0.0
    b[1, ::2] = 0.0
    b[2] = 0.0
    b[2, 3:5] = 0.1
    bt = torch.from_numpy(b).to("cuda", torch.float64)
    print(f"prior overflow {prec} p={p} M={M}", flush=True)
    lp = s.grad(bt, lam, prec)[1].cpu().numpy()
    rows = np.r_[0:20, M - 10:M]
    ll = likelihood.loglik(b[rows], Xs, y)
    prior = gt_prior.log_prior(b[rows], 1.0, lam)
    assert np.all(np.isfinite(prior))
    size = np.abs(prior).max()                    # of the terms, which cancel in a row that is half zeros
    tol = 1e-10 * size + (1e-10 if prec == "fp64" else 1e-4) * np.abs(ll)
    assert np.all(np.abs(lp[rows] - (ll + prior)) <= tol)
    s.close()
