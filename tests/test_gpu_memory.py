"""Device memory of a handle: the genotypes are n p bytes, and a handle whose calls need no adjoint
holds them once more as codes of the streamed contraction, not twice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_random_walk_handles_hold_no_adjoint_copy(prec):
    import torch
    from paper_1106_0322_amd import SamplerConfig, SpaSMC
    n, p = 100000, 255
    X = np.zeros((n, p), dtype=np.uint8)
    X[::3] = 1
    y = (np.arange(n) % 2).astype(np.uint8)
    kw = dict(N=64, a=1.0, lambdas=np.geomspace(10, 1, 2), move="rwm", sweeps=0, init_sweeps=0, prec=prec, seed=0)
    SpaSMC(SamplerConfig(n=50, p=3, **kw), X[:50, :3], y[:50]).close()      # the library itself is loaded
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    s = SpaSMC(SamplerConfig(n=n, p=p, **kw), X, y)
    s.loglik(torch.zeros(64, p, dtype=torch.float64, device="cuda"), prec)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    print(f"{prec}: {used / (n * p):.2f} n p bytes")
    assert used < 2.6 * n * p
    s.close()
