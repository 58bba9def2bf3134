"""Top-K feature adjoint where its blocks end: distinct selected surfels per
tile around the 16-slot blocks and 48-slot chunks, K around the halves a
pixel's selections are split into, channels around the passes of 16.  Feature
gradients and (through the dots) geometry gradients against the FP64 oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, decided, render, require_gpu, stored_feat, to_dev
from paper_2604_10982_amd import psm, scenes
from test_gpu_backward import grad_errors

pytestmark = pytest.mark.gpu


def _slots(ws, cam, K):
    """Distinct selected surfels of every tile."""
    sel = psm.read_selection(ws, psm.camera_struct(cam), psm.config_struct(K, "ellipse", "topk"))
    ids = sel["sel_id"].cpu().numpy().reshape(cam.height, cam.width, K)
    return [len(set(t[t >= 0].tolist())) for y in range(0, cam.height, 16) for x in range(0, cam.width, 16)
            for t in [ids[y:y + 16, x:x + 16]]]


@pytest.mark.parametrize("n,s,K,c,most", [(40, 0.30, 1, 8, 15), (150, 0.20, 9, 24, 63), (500, 0.12, 16, 40, 187),
                                          (900, 0.09, 17, 16, 281), (1500, 0.07, 32, 56, 536)])
def test_feature_adjoint_edges(orc, n, s, K, c, most):
    require_gpu()
    sc = scenes.uniform_box(n, c, seed=n, xy=1.0, z=(2.0, 5.0), scale_mu=np.log(s))
    cam = scenes.pinhole(71, 50, f=60.0)
    t = to_dev(sc)
    _, ws = render(t, cam, K, "ellipse", "topk")
    slots = _slots(ws, cam, K)
    print(f"[adjoint] n={n} K={K} c={c} slots {min(slots)}..{max(slots)}", flush=True)
    assert max(slots) == most  # the oracle's count: 0 to 15 slots here, past 48, 96 and 512 in the others
    feat = stored_feat(t)
    ok = decided(orc.render(sc, cam, K, orc.TOPK, feat=feat))
    g = scenes.upstream(cam.height, cam.width, sc.c, seed=1)
    for k in g:
        g[k][~ok] = 0.0
    ref = orc.backward(sc, cam, g, K=K, blend=orc.TOPK, feat=feat)
    gt = {k: torch.tensor(v, device=DEV) for k, v in g.items()}
    got = psm.backward(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"], cam, ws, gt, K,
                       "ellipse", "topk")
    torch.cuda.synchronize()
    worst = grad_errors({k: v.cpu().numpy().astype(np.float64) for k, v in got.items()}, ref)
    assert max(worst.values()) <= 1e-3, worst
