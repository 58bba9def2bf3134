"""SOGMM assignment where the bounds decide little: components 2 mm and 0.5 mm
thick on planes tens of metres wide, a third of the surfels metres off them (a
score of 1e5 and more, of which the bound's share exceeds what coplanar
components differ by), and surfels outside the bound's range.  Waves then score
every component, seen early (256 components and more) or at the end; each
surfel still gets the component of the full FP32 scan, with the rounding
allowance of that comparison."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, require_gpu
from oracle import geometry as GE
from paper_2604_10982_amd import psm
from test_gpu_geometry_bound import noise, records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("thick", [0.02, 0.002, 0.0005])
@pytest.mark.parametrize("k,n", [(64, 1500), (255, 513), (256, 1500), (512, 2000), (1999, 1100)])
def test_thin_coplanar_components(k, n, thick):
    require_gpu()
    rng = np.random.default_rng(k + n)
    plane = rng.integers(0, 3, k)
    mean = rng.uniform(-40.0, 40.0, (k, 3))
    mean[np.arange(k), plane] = rng.choice([-8.0, 8.0], k)
    var = np.full((k, 3), 1.5 ** 2)
    var[np.arange(k), plane] = thick ** 2
    cov = np.zeros((k, 6))
    cov[:, 0], cov[:, 3], cov[:, 5] = var.T
    w = rng.dirichlet(np.ones(k))
    near = rng.integers(0, k, n)
    x = mean[near] + rng.normal(0, 1, (n, 3)) * np.sqrt(var[near])
    off = rng.random(n) < 0.33
    x[off] = rng.uniform(-40.0, 40.0, (int(off.sum()), 3))
    x[128:192] = x[128:192] * 1e10  # a wave out of the margins' range
    mean, cov, w, x = (np.ascontiguousarray(a, np.float32) for a in (mean, cov, w, x))
    T = lambda a: torch.tensor(a, device=DEV)
    out = psm.geometry_loss(T(x), torch.ones(n, 2, device=DEV), torch.ones(n, 4, device=DEV), T(mean), T(cov), T(w),
                            0.4, return_assign=True)
    got = out["assign"].cpu().numpy()
    comp = records(mean, cov, w)
    s, e = GE.scores_f32(x, comp).astype(np.float64), noise(x, comp)
    best, i = s.argmin(1), np.arange(n)
    assert np.isfinite(s).all()
    assert (s[i, got] <= s[i, best] + e[i, got] + e[i, best]).all()
    assert (got == best).mean() > 0.99 - (64 / n)
