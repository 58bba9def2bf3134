"""Tiles in the order of their list lengths: beyond 1024 tiles every call orders
them, up to there only the persistent schedule does.  On both sides of that
line, with lists from empty to long, the schedules give the same images,
selection and gradients, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, OUTPUTS, render, require_gpu, to_dev
from paper_2604_10982_amd import psm, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blend", ["topk", "full"])
@pytest.mark.parametrize("w,h", [(512, 512), (512, 513), (1024, 1008), (40, 6400)])
def test_schedules_agree_around_the_ordering_line(w, h, blend):
    require_gpu()
    K = 8
    sc = scenes.uniform_box(6000, 16, seed=w + h, xy=1.2, z=(2.0, 5.0), scale_mu=np.log(0.05))
    cam = scenes.pinhole(w, h, f=0.6 * max(w, h))
    t = to_dev(sc)
    g = {k: torch.tensor(v, device=DEV) for k, v in scenes.upstream(h, w, sc.c, seed=1).items()}
    ref = None
    for s in (psm.SCHED_GRID, psm.SCHED_PERSISTENT):
        print(f"[order] {w}x{h} {blend} schedule {s}", flush=True)
        launch = (s, s, 0, 0, 16)
        out, ws = render(t, cam, K, "ellipse", blend, launch=launch)
        grad = psm.backward(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"], cam, ws, g, K,
                            "ellipse", blend, launch=launch)
        got = {k: out[k].clone() for k in OUTPUTS} | {"d_" + k: v.clone() for k, v in grad.items()}
        torch.cuda.synchronize()
        if ref is None:
            ref = got
            assert float(ref["alpha"].max()) > 0.5
            continue
        for k in ref:
            assert torch.equal(got[k], ref[k]), k
