"""EM MAP estimates from start points that are not finite.  A linear predictor that is not a
number counts as sigma = 0, so the first sweep runs on the residuals y, the soft threshold sets
the coefficient that was not a number to zero, and the next sweep's fresh predictor is finite
again.  The reference below is the coordinate sweep of the oracle with that rule; tolerance as in
test_gpu_map.py (both sides differ in summation order only)."""
import numpy as np
import pytest
from scipy.special import expit

from oracle import em
from tests.gpu_util import dataset, particles

pytestmark = pytest.mark.gpu


def _map_em(Xs, y, b0, a, lam, outer, inner):
    n, p = Xs.shape
    modes = []
    for b in b0:
        b = b.copy()
        for _ in range(outer):
            thr = 4.0 / n * em.em_weights(b, a, lam)
            for _ in range(inner):
                eta = (b * Xs).sum(axis=1)
                for j in range(p):
                    z = b[j] + 4.0 / n * ((y - np.where(np.isnan(eta), 0.0, expit(eta))) @ Xs[:, j])
                    nb = z - thr[j] if z > thr[j] else z + thr[j] if z < -thr[j] else 0.0
                    delta = nb - b[j]             # not a number for an infinite coefficient: it moves
                    if delta != 0.0:
                        eta = eta + delta * Xs[:, j]
                    b[j] = nb
        modes.append(b)
    return np.stack(modes)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf], ids=["nan", "inf", "minus_inf"])
@pytest.mark.parametrize("n,p", [(100, 9), (700, 20), (6100, 12), (8300, 7)])
def test_map_em_from_non_finite_starts(n, p, value):
    import torch
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    cfg, X, y, Xs = dataset("n5000_p200_mala_bf16", n, p, 5)
    s = SpaSMC(SamplerConfig.from_workload(cfg, n=n, p=p, N=64, lambdas=np.geomspace(10.0, 1.0, 3), init_sweeps=0,
                                           sweeps=0, a=1.0), X, y)
    b0 = particles(4, p, seed=n, scale=0.3)
    b0[1, 0] = value
    b0[2, p // 2] = value
    b0[3, p - 1] = value
    for outer, inner in ((1, 1), (2, 2)):
        print(f"map_em {value} start n={n} p={p} outer={outer}", flush=True)
        mode, _ = s.map_em(torch.from_numpy(b0).cuda(), 0.4, outer, inner)
        with np.errstate(invalid="ignore"):
            ref = _map_em(Xs, y.astype(np.float64), b0, 1.0, 0.4, outer, inner)
        assert np.allclose(mode.cpu().numpy(), ref, rtol=0, atol=1e-9, equal_nan=True)
    s.close()
