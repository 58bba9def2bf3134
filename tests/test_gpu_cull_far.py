"""Sub-tile culling with the world's origin far from the camera.

The camera-space position R mu + t is a difference of large numbers there: in
FP32 the projected ellipse is off by fx 2^-24 (|R mu| + |t|) / z pixels (half a
pixel at 5 km), and a wave that culls by it would leave out surfels that blend.
The tile lists are FP32 by definition and lose a surfel near the tile's edge in
the same way, so the image is one tile and its outer two pixels are not
compared: inside, everything that the FP64 oracle blends has to be there."""
import numpy as np
import pytest

from gpu_helpers import decided, image_errors, np_out, require_gpu, stored_feat, to_dev
from paper_2604_10982_amd import psm, scenes
from paper_2604_10982_amd.scenes import Scene
import torch

pytestmark = pytest.mark.gpu

K = 8


def far_scene(dist, width, height, n=600, seed=17, f=1500.0):
    """Surfels of 0.2 to 2 px about a camera `dist` metres from the origin, turned."""
    rng = np.random.default_rng(seed)
    ang = rng.uniform(-1.0, 1.0, 3)
    cx, sx, cy, sy, cz, sz = *(g(ang[0]) for g in (np.cos, np.sin)), *(g(ang[1]) for g in (np.cos, np.sin)), *(
        g(ang[2]) for g in (np.cos, np.sin))
    R = (np.array([[1, 0, 0], [0, cx, -sx], [0, sx, cx]]) @ np.array([[cy, 0, sy], [0, 1, 0], [-sy, 0, cy]])
         @ np.array([[cz, -sz, 0], [sz, cz, 0], [0, 0, 1]])).astype(np.float32)
    centre = dist * rng.dirichlet(np.ones(3)) * rng.choice([-1.0, 1.0], 3)
    t = (-R.astype(np.float64) @ centre).astype(np.float32)
    z = rng.uniform(0.5, 4.0, n)
    px, py = rng.uniform(-2, width + 2, n), rng.uniform(-2, height + 2, n)
    mc = np.stack([(px - width / 2) * z / f, (py - height / 2) * z / f, z], -1)
    means = (mc - t.astype(np.float64)) @ R.astype(np.float64)  # R^T (mc - t)
    scales = np.exp(rng.uniform(np.log(0.2), np.log(2.0), (n, 2))) * (z / f)[:, None]
    c = np.float32
    sc = Scene(means.astype(c), scales.astype(c), rng.standard_normal((n, 4)).astype(c),
               rng.uniform(0.05, 0.9, n).astype(c), rng.uniform(0, 1, (n, 3)).astype(c),
               rng.standard_normal((n, 8)).astype(c))
    return sc, scenes.pinhole(width, height, f=f, R=R, t=t)


@pytest.mark.parametrize("tw", [8, 16, 32])
@pytest.mark.parametrize("flags", [0, psm.FLAG_LOWPASS, psm.FLAG_OPACITY_FOOTPRINT])
@pytest.mark.parametrize("dist", [0.0, 500.0, 2000.0, 5000.0])
def test_far_origin_keeps_contributors(orc, dist, flags, tw):
    require_gpu()
    sc, cam = far_scene(dist, tw, 256 // tw)
    t = to_dev(sc)
    out, _ = psm.forward(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"], cam, K,
                         flags=flags, launch=(0, 0, 0, 0, tw))
    torch.cuda.synchronize()
    lp = bool(flags & psm.FLAG_LOWPASS)
    feat = stored_feat(t)
    ref = orc.render(sc, cam, K, orc.TOPK, feat=feat, lowpass=lp)
    absf = orc.render(sc, cam, K, orc.TOPK, feat=np.abs(feat), lowpass=lp)["feat"]
    assert ref["ncontrib"].mean() > 3
    ok = decided(ref)
    ok[:2], ok[-2:], ok[:, :2], ok[:, -2:] = False, False, False, False
    assert ok.sum() > 80
    worst = image_errors(np_out(out), ref, absf, ok, 1e-5)
    assert max(worst.values()) <= 1.0, worst
