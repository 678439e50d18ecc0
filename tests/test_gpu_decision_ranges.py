"""The FP64 MALA decision on every count of ranges that its gradient can be left in: one (few
individuals, with few and with many particles), 8 and 16 (few particles, many individuals);
trajectories against the oracle with the tolerances of test_fp64_tracks_oracle_ragged_shapes.
The device-side burn-in's step sizes: FP64 against the oracle; reduced precisions by what the rule
step <- step exp(clip(accepted / N - target, +-log 2)) leaves, whole numbers of acceptances, and
after one sweep, whose draws are the oracle's, by a number near the oracle's: log alpha is off by at
most 1e-4 of two log-likelihoods near n log 2, and log u has a density of at most one."""
import math

import numpy as np
import pytest

from oracle import smc
from tests.gpu_util import dataset

pytestmark = pytest.mark.gpu
TARGET = {"mala": 0.574, "rwm": 0.234}


def _run(cfg, X, y, **over):
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    return SpaSMC(SamplerConfig.from_workload(cfg, n=X.shape[0], p=X.shape[1], **over), X, y)


@pytest.mark.parametrize("n,p,N", [(90, 12, 40), (100, 33, 8200), (1030, 130, 20), (2100, 11, 17), (2050, 200, 16)])
def test_fp64_mala_tracks_oracle(n, p, N):
    cfg, X, y, Xs = dataset("n500_p10_rwm_fp64", n=n, p=p)
    cfg = cfg.replace(n=n, p=p, N=N, T=4, sweeps=3, init_sweeps=5, move="mala", lambdas=tuple(np.geomspace(2.0, 0.2, 4)))
    print(f"MALA n={n} p={p} N={N}", flush=True)
    r = smc.run_config(cfg, X, y)
    g = _run(cfg, X, y)
    stats = g.run()
    mean, _, logz = g.paths()
    beta, _ = g.particles()
    assert np.abs(mean - r.mean).max() <= 1e-8
    assert np.abs(beta.cpu().numpy() - r.state.beta).max() <= 1e-8
    assert np.allclose(logz, r.log_z, rtol=1e-10, atol=1e-9)
    assert np.allclose([s["accept_rate"] for s in stats[1:]], r.accept[1:], rtol=0, atol=1e-12)
    assert np.allclose([s["step"] for s in stats], r.step, rtol=1e-12)
    g.close()


@pytest.mark.parametrize("move,prec", [("mala", "bf16x2"), ("rwm", "bf16x2"), ("rwm", "fp8x3"), ("rwm", "fp8x4"),
                                       ("mala", "fp32"), ("rwm", "fp32")])
def test_burn_in_step_sizes(move, prec):
    cfg, X, y, Xs = dataset("n500_p10_rwm_fp64", n=400, p=37)
    n, p, N = 400, 37, 4111
    cfg = cfg.replace(n=n, p=p, N=N, T=2, sweeps=1, init_sweeps=1, move=move, lambdas=(2.0, 1.0))
    ref = smc.run_config(cfg, X, y, T_stop=1)
    step0 = cfg.step0()
    for k in (1, 2, 3, 7):
        print(f"burn-in {move} {prec} sweeps={k}", flush=True)
        g = _run(cfg, X, y, prec=prec, init_sweeps=k)
        moved = math.log(g.stats(1)["step"] / step0)
        g.close()
        # with c of the k sweeps clipped at +log 2, the others accepted this many in all
        counts = [N * (moved - c * math.log(2.0) + (k - c) * TARGET[move]) for c in range(k + 1)]
        assert any(-1e-6 <= v <= (k - c) * N + 1e-6 and abs(v - round(v)) <= 1e-6 for c, v in enumerate(counts)), counts
        if k == 1:
            assert abs(moved - math.log(ref.step[0] / step0)) <= 2 * 2e-4 * n * math.log(2.0)
    g = _run(cfg, X, y, prec=prec, init_sweeps=3, adapt=False)
    assert g.stats(1)["step"] == step0
    g.close()
