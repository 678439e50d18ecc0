"""GPU parity of the streamed FP32/FP64 contraction (the FP32 gradient is the tiled one) and of the one-launch random-walk sweeps
at the sizes where they can go wrong: every instantiated row width and both its ends, a
partial last k-step, one individual more or less than a block of 16, one particle more or
less than a workgroup's 16, one and several ranges of individuals.  Tolerances are those of
the other precision tests (1e-10 FP64, 1e-4 FP32 relative log-likelihood; gradients 1e-10 and
1e-5 times the column's absolute sum)."""
import numpy as np
import pytest

from oracle import gt_prior, likelihood, smc
from tests.gpu_util import dataset, particles, rel_err

pytestmark = pytest.mark.gpu


def _sampler(n, p, prec):
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    cfg, X, y, Xs = dataset("n2000_p50_rwm_fp32", n, p)
    sc = SamplerConfig(n=X.shape[0], p=X.shape[1], N=64, a=cfg.a, lambdas=np.geomspace(10, 1, 2), move="rwm",
                       sweeps=0, init_sweeps=0, prec=prec, seed=0)
    return SpaSMC(sc, X, y), cfg, X, y, Xs


# (n, p, M): widths of 1, 2, 3-4, 5-8, 9-13, 14-16 groups of 16 markers (FP32: 17-24, 25-32)
SHAPES = [(30, 1, 1), (32, 16, 15), (34, 17, 17), (64, 32, 16), (66, 33, 40), (200, 61, 33), (1000, 64, 5),
          (130, 65, 16), (3000, 128, 31), (80, 129, 18), (1200, 207, 64), (70, 208, 3), (4000, 209, 100), (96, 255, 20)]
WIDE = [(100, 256, 17), (2000, 383, 16), (48, 385, 5), (600, 511, 33)]


@pytest.mark.parametrize("prec,n,p,M", [(q, *s) for q in ("fp64", "fp32") for s in SHAPES] + [("fp32", *s) for s in WIDE])
def test_streamed_loglik_and_gradient(prec, n, p, M):
    import torch
    s, cfg, X, y, Xs = _sampler(n, p, prec)
    lam = 0.3
    b = particles(M, p, seed=n + p)
    print(f"streamed {prec} n={n} p={p} M={M}", flush=True)
    for dt in (torch.float64, torch.float32):
        bt = torch.from_numpy(b).to("cuda", dt)
        bs = bt.double().cpu().numpy()
        ll = s.loglik(bt, prec).cpu().numpy()
        g, lp = s.grad(bt, lam, prec)
        assert g.dtype == dt
        ll_ref, gl_ref = likelihood.loglik_and_grad(bs, Xs, y)
        g_ref = gl_ref + gt_prior.gt_grad(bs, cfg.a, lam)
        lp_ref = ll_ref + gt_prior.log_prior(bs, cfg.a, lam)
        rel = 1e-10 if prec == "fp64" else 1e-4
        assert rel_err(ll, ll_ref).max() <= rel
        assert rel_err(lp.cpu().numpy(), lp_ref).max() <= rel
        tol = (1e-10 if prec == "fp64" else 1e-5) * np.abs(Xs).sum(axis=0)
        if dt == torch.float32:
            tol = tol + 2.0 ** -24 * np.abs(g_ref)
        assert np.all(np.abs(g.double().cpu().numpy() - g_ref) <= tol)
    s.close()


def test_overflowing_prior_factors():
    """A product of prior factors beyond the FP64 range falls back to the sum of logs."""
    import torch
    s, cfg, X, y, Xs = _sampler(64, 40, "fp64")
    b = np.zeros((3, 40))
    b[1] = 1e200 * np.sign(np.random.default_rng(0).normal(size=40))
    g, lp = s.grad(torch.from_numpy(b).cuda(), 0.3, "fp64")
    ll = s.loglik(torch.from_numpy(b).cuda(), "fp64").cpu().numpy()
    prior = gt_prior.log_prior(b, cfg.a, 0.3)
    assert np.allclose(lp.cpu().numpy()[1] - ll[1], prior[1], rtol=1e-9, atol=1e-12 * abs(ll[1]))
    assert np.allclose(lp.cpu().numpy()[[0, 2]], (ll + prior)[[0, 2]], rtol=1e-12)


# sizes of the one-launch sweeps (every row width, ragged rows, blocks and workgroups), and
# one that takes the separate launches (few particles, many individuals)
@pytest.mark.parametrize("n,p,N", [(48, 1, 17), (66, 16, 40), (100, 30, 33), (130, 63, 20), (200, 65, 49), (90, 130, 31),
                                   (64, 255, 16), (500, 10, 4100), (4000, 10, 17)])
@pytest.mark.parametrize("a", [1.0, float("inf")], ids=["a1", "a_inf"])
def test_fp64_random_walk_tracks_oracle(n, p, N, a):
    cfg, X, y, Xs = dataset("n500_p10_rwm_fp64", n=n, p=p)
    cfg = cfg.replace(n=n, p=p, N=N, T=4, sweeps=3, init_sweeps=5, a=a, lambdas=tuple(np.geomspace(2.0, 0.2, 4)))
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    print(f"random walk n={n} p={p} N={N} a={a}", flush=True)
    r = smc.run_config(cfg, X, y)
    g = SpaSMC(SamplerConfig.from_workload(cfg), X, y)
    stats = g.run()
    mean, _, logz = g.paths()
    beta, _ = g.particles()
    assert np.abs(mean - r.mean).max() <= 1e-8
    assert np.abs(beta.cpu().numpy() - r.state.beta).max() <= 1e-8
    assert np.allclose(logz, r.log_z, rtol=1e-10, atol=1e-9)
    assert np.allclose([s["accept_rate"] for s in stats[1:]], r.accept[1:], rtol=0, atol=1e-12)
    ll = g.state_loglik().cpu().numpy()
    assert rel_err(ll, likelihood.loglik(beta.cpu().numpy(), Xs, y)).max() <= 1e-10
    g.close()


def test_fp32_one_launch_keeps_its_likelihoods():
    """The log-likelihoods kept by the FP32 sweeps are those of the particles they leave."""
    cfg, X, y, Xs = dataset("n2000_p50_rwm_fp32", n=300, p=45)
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    cfg = cfg.replace(n=300, p=45, N=1000, T=4, sweeps=4, init_sweeps=6, lambdas=tuple(np.geomspace(2.0, 0.2, 4)))
    g = SpaSMC(SamplerConfig.from_workload(cfg), X, y)
    g.run()
    beta, _ = g.particles()
    kept, fresh = g.state_loglik().cpu().numpy(), g.loglik(beta).cpu().numpy()
    assert rel_err(kept, fresh).max() <= 1e-13      # same FP32 terms, FP64 sums in another order
    assert 0.0 < g.stats(2)["accept_rate"] < 1.0
    g.close()


@pytest.mark.parametrize("prec,n,p,M", [("fp64", 90, 129, 4097), ("fp64", 130, 208, 4096), ("fp64", 50, 255, 4113),
                                        ("fp32", 90, 257, 4097), ("fp32", 40, 400, 4128), ("fp32", 60, 511, 4096)])
def test_wide_rows_beyond_one_block_per_cu(prec, n, p, M):
    """Wide rows on both sides of 256 blocks of particles (8 and 4 waves per workgroup)."""
    import torch
    s, cfg, X, y, Xs = _sampler(n, p, prec)
    b = particles(M, p, seed=n + p, scale=0.05)
    bt = torch.from_numpy(b).to("cuda", torch.float64 if prec == "fp64" else torch.float32)
    print(f"wide rows {prec} n={n} p={p} M={M}", flush=True)
    rows = np.r_[0:40, M - 40:M]
    ref = likelihood.loglik(bt.double().cpu().numpy()[rows], Xs, y)
    ll = s.loglik(bt, prec).cpu().numpy()
    assert rel_err(ll[rows], ref).max() <= (1e-10 if prec == "fp64" else 1e-4)
    s.close()


@pytest.mark.parametrize("prec,n,p,N", [("fp64", 2000, 200, 100), ("fp64", 100, 150, 4200), ("fp64", 3000, 100, 600),
                                        ("fp32", 300, 129, 200), ("fp32", 120, 200, 4200), ("fp32", 6400, 100, 300)])
def test_random_walk_apart_keeps_its_likelihoods(prec, n, p, N):
    """Random walks on the side of separate launches: the kept log-likelihoods are those of the
    particles (the same terms, FP64 sums in another order)."""
    cfg, X, y, Xs = dataset("n2000_p50_rwm_fp32", n=n, p=p)
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    cfg = cfg.replace(n=n, p=p, N=N, T=3, sweeps=3, init_sweeps=4, lambdas=tuple(np.geomspace(2.0, 0.2, 3)))
    print(f"random walk {prec} n={n} p={p} N={N}", flush=True)
    g = SpaSMC(SamplerConfig.from_workload(cfg, prec=prec), X, y)
    g.run()
    beta, _ = g.particles()
    kept, fresh = g.state_loglik().cpu().numpy(), g.loglik(beta, prec).cpu().numpy()
    assert rel_err(kept, fresh).max() <= 1e-13
    assert 0.0 < g.stats(2)["accept_rate"] < 1.0
    g.close()
