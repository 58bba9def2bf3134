"""SOGMM assignment through the matrix-core bound: whatever the shape of the
components, the number of them against the tiles of 16 and chunks of 256, the
number of surfels against the blocks of 512, and for components or surfels
outside the ranges of the bound, every surfel gets the component that a full
scan of the FP32 scores gives it.  The scan's records are formed here in FP64
from the same formula; either side's score may differ by the FP32 rounding of
record and score, at most 16 roundings of 2^-24 of the sum of |terms| each."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, require_gpu
from oracle import geometry as GE
from paper_2604_10982_amd import psm

pytestmark = pytest.mark.gpu


def records(mean, cov6, weight):
    c = np.asarray(cov6, np.float64)
    xx, xy, xz, yy, yz, zz = c.T
    adj = np.stack([yy * zz - yz * yz, xz * yz - xy * zz, xy * yz - xz * yy, xx * zz - xz * xz, xy * xz - xx * yz,
                    xx * yy - xy * xy], 1)
    det = xx * adj[:, 0] + xy * adj[:, 1] + xz * adj[:, 2]
    return {"mean": np.asarray(mean, np.float32), "P": (adj / det[:, None]).astype(np.float32),
            "c": (np.log(det) - 2.0 * np.log(np.asarray(weight, np.float64))).astype(np.float32)}


def noise(x, comp):
    d = np.abs(x[:, None, :].astype(np.float64) - comp["mean"][None].astype(np.float64))
    A = np.abs(GE.cov_matrix(comp["P"]))
    return (np.einsum("nki,kij,nkj->nk", d, A, d) + np.abs(comp["c"])[None]) * 16 * 2.0 ** -24


def components(kind, k, rng):
    sd = {"flat": (1.5, 1.5, 0.005), "needle": (4.0, 0.05, 0.001), "ball": (0.4, 0.4, 0.4), "far": (1.5, 1.0, 0.01),
          "odd": (1.0, 0.6, 0.02)}[kind]
    Q, _ = np.linalg.qr(rng.normal(size=(k, 3, 3)))
    S = np.einsum("kij,kj,klj->kil", Q, (np.asarray(sd) * rng.uniform(0.5, 2.0, (k, 3))) ** 2, Q)
    mean = rng.uniform(-4, 4, (k, 3)) + (700.0 if kind == "far" else 0.0)
    cov = np.stack([S[:, i, j] for i, j in GE.SYM], 1)
    w = rng.dirichlet(np.ones(k))
    if kind == "odd":
        w[1::17] = 0.0                                  # constant +inf: never taken
        cov[2::19] = np.nan                             # NaN scores: never taken
        cov[3::23] = (1e20, 0, 0, 1e20, 0, 1e20)        # wider than the bound covers
        cov[5::29] = (1.0, 0, 0, 1.0, 0, 1e-18)         # thinner than it covers
        mean[7::31] *= 1e10
    return mean.astype(np.float32), cov.astype(np.float32), w.astype(np.float32)


@pytest.mark.parametrize("kind", ["flat", "needle", "ball", "far", "odd"])
@pytest.mark.parametrize("k,n", [(1, 1), (15, 63), (16, 65), (17, 511), (255, 512), (257, 513), (1100, 700)])
def test_assignment_is_the_full_scan(kind, k, n):
    require_gpu()
    rng = np.random.default_rng(1000 * k + n)
    mean, cov, w = components(kind, k, rng)
    near = rng.integers(0, k, n)
    x = (np.where(np.abs(mean[near]) < 1e6, mean[near], 0) + rng.normal(0, 0.3, (n, 3))).astype(np.float32)
    if kind == "odd" and n > 60:
        x[3], x[17], x[40], x[59] = (np.nan, 0, 0), (1e12, 0, 1), (np.inf, 0, 0), (3e25, -3e25, 2e25)
    T = lambda a: torch.tensor(a, device=DEV)
    out = psm.geometry_loss(T(x), torch.ones(n, 2, device=DEV), torch.ones(n, 4, device=DEV), T(mean), T(cov), T(w),
                            0.4, return_assign=True)
    got = out["assign"].cpu().numpy()
    with np.errstate(all="ignore"):
        comp = records(mean, cov, w)
        s = GE.scores_f32(x, comp).astype(np.float64)
        e = noise(x, comp)
    s[~(s < np.inf)] = np.inf
    best = s.argmin(1)
    i = np.arange(n)
    none = ~np.isfinite(s[i, best])
    np.testing.assert_array_equal(got[none], 0)          # no finite score: component 0
    ok = ~none
    assert ok.sum() >= n - 4 or kind == "odd"
    sg, sb = s[i, got][ok], s[i, best][ok]
    assert (sg <= sb + e[i, got][ok] + e[i, best][ok]).all()
