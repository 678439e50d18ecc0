"""Weighted summaries on both sides of the line between a workgroup per coefficient and passes over
all coefficients (few values of many coefficients), with and without tolerances: whole numbers of
weight, so quantiles and concentrations are compared exactly with the definition."""
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(v, w, levels, deltas):
    M, p = v.shape
    q = np.floor(np.ldexp(w / w.max(), 63 - int(np.ceil(np.log2(M))) if M > 1 else 63)).astype(np.uint64)
    C = int(sum(int(x) for x in q))
    quant, conc = np.empty((len(levels), p)), np.empty((len(deltas), p))
    for j in range(p):
        order = np.argsort(v[:, j], kind="stable")
        cum, run = [], 0
        for i in order:
            run += int(q[i])
            cum.append(run)
        for a, al in enumerate(levels):
            at = Fraction(float(al)) * C
            need = -(-at.numerator // at.denominator)
            quant[a, j] = v[order[next(k for k, c in enumerate(cum) if c >= need)], j]
        for b, de in enumerate(deltas):
            inside = sum(int(q[i]) for i in range(M) if abs(float(v[i, j])) < de)
            conc[b, j] = 1.0 - float(inside) / float(C)
    return quant, conc


@pytest.mark.parametrize("M,p,L,D,f64", [(1, 4700, 1, 0, False), (1, 4800, 1, 2, True), (3, 2300, 5, 1, False),
                                         (3, 2200, 5, 0, True), (40, 3100, 3, 0, False), (40, 3200, 3, 8, False),
                                         (33, 1700, 8, 8, True), (2, 66000, 1, 1, False)])
def test_both_forms_give_the_definition(M, p, L, D, f64):
    import torch
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    X = (np.arange(40)[:, None] % 3 * np.ones(3)).astype(np.uint8)
    s = SpaSMC(SamplerConfig(n=40, p=3, N=64, a=1.0, lambdas=np.geomspace(10, 1, 2), move="rwm", sweeps=0, init_sweeps=0,
                             prec="fp32", seed=0), X, (np.arange(40) % 2).astype(np.uint8))
    rng = np.random.default_rng([M, p])
    v = rng.normal(0.0, 0.1, size=(M, p)).astype(np.float64 if f64 else np.float32)
    v[rng.random((M, p)) < 0.1] = 0.0
    w = rng.gamma(0.5, 1.0, size=M)
    levels, deltas = np.linspace(0.05, 0.95, L), np.linspace(0.03, 0.2, D)
    print(f"summaries M={M} p={p} L={L} D={D} f64={f64}", flush=True)
    for rep in range(2):                          # the passes leave their scratch as they found it
        q, c = s.weighted_summaries(torch.from_numpy(v).cuda(), torch.from_numpy(w).cuda(), levels, deltas)
    cols = np.unique(np.r_[0:60, p // 2:p // 2 + 60, p - 60:p])
    qr, cr = _reference(v[:, cols], w, levels, deltas)
    assert np.array_equal(q.cpu().numpy()[:, cols], qr)
    assert np.array_equal(c.cpu().numpy()[:, cols], cr)
    s.close()
