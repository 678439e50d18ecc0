"""Rounding of the EM kernel's coordinate sweep with rare markers and unbalanced labels, against the
same sweep in extended precision.  In one sweep from zero, coordinate j errs by at most
  e_j = 4 eps [ (36 + 2 j) mean_k |x_kj| + 4 (mu_j / s_j) |mean_k u_k| ] + sum_{i<j} e_i,
eps = 2^-53: sums of at most 20 terms per thread and 9 levels of a tree, the rounding of x, of u <= 1
(two roundings per move before) and of the standardisation constants; an error of an earlier
move shifts 4 g_j / n by no more than itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def _sweep(X, y, thr, inner):
    """Coordinate sweeps from zero in extended precision, and the first sweep's error bound."""
    L = np.longdouble
    n, p = X.shape
    Xl = X.astype(L)
    mu = Xl.mean(axis=0)
    s = np.sqrt(((Xl - mu) ** 2).mean(axis=0))
    x = (Xl - mu) / s
    b, tol, total = np.zeros(p, L), np.zeros(p), 0.0
    for sw in range(inner):
        eta = x @ b
        for j in range(p):
            u = y - 1 / (1 + np.exp(-eta))
            z = b[j] + 4 * (u @ x[:, j]) / n
            nb = max(z - thr, L(0)) if z > 0 else min(z + thr, L(0))
            eta += (nb - b[j]) * x[:, j]
            b[j] = nb
            if sw == 0:
                total += 4 * EPS * ((36 + 2 * j) * float(np.abs(x[:, j]).mean()) +
                                    4 * float(mu[j] / s[j]) * abs(float(u.mean())))
                tol[j] = total
    return b, tol


@pytest.mark.parametrize("n,p,freq,cases", [(10000, 6, 0.0005, 0.9), (5000, 8, 0.002, 0.9), (400, 5, 0.01, 0.95),
                                            (10000, 6, 0.9995, 0.1), (3000, 40, 0.3, 0.5), (3000, 20, 0.05, 0.9)])
def test_one_sweep_rounding(n, p, freq, cases):
    import torch
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    rng = np.random.default_rng([n, p])
    X = rng.binomial(2, freq, size=(n, p)).astype(np.uint8)
    X[0], X[1] = 1, 2 if freq > 0.5 else 0       # no marker without variance
    y = (rng.uniform(size=n) < cases).astype(np.uint8)
    lam = 50.0
    s = SpaSMC(SamplerConfig(n=n, p=p, N=64, a=1.0, lambdas=np.geomspace(10, 1, 2), move="rwm", sweeps=0, init_sweeps=0,
                             prec="fp64", seed=0), X, y)
    print(f"one sweep n={n} p={p} freq={freq} cases={cases}", flush=True)
    mode, _ = s.map_em(torch.zeros(1, p, dtype=torch.float64, device="cuda"), lam, 1, 1)
    ref, tol = _sweep(X, y.astype(np.longdouble), np.longdouble(4) / n * 2 / np.longdouble(lam), 1)
    err = np.abs(mode.cpu().numpy()[0].astype(np.longdouble) - ref).astype(float)
    tol = tol + EPS * np.abs(ref).astype(float) * 4
    print(f"  error {err.max():.2e}, at most {np.max(err / tol):.2f} of the bound")
    assert np.all(err <= tol)
    s.close()
