"""Rotation gradients of surfels seen edge-on against recorded values.

A disk whose normal is nearly perpendicular to its viewing ray projects to an
ellipse of aspect 1 / |cos|.  The pixel offsets it covers lie along one axis
and the chain rule to its rotation takes differences of FP32 sums over them, so
the order of these sums shows in the gradient (4e-6 to 9e-6 of its norm here,
single elements of a large scene by 1e-3 and more) although no order is nearer
to the exact value.  The order is fixed per tile shape: golden/edge_on_quats.json holds the
values of a reduction of rounded products over the tile's rows by a tree of
lanes, recorded on an MI355X.  What may differ is the order of the sums that
the chain rule does not amplify (the normals, over 64 pixels: at most a few
2^-24 of the largest element they share a sum with), hence 2e-6 of the larger
of an element and the root mean square."""
import json
import os

import numpy as np
import pytest
import torch

from gpu_helpers import DEV, render, require_gpu, to_dev
from paper_2604_10982_amd import psm, scenes
from paper_2604_10982_amd.scenes import Scene

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "edge_on_quats.json")


def edge_on(n=48, c=8, seed=11):
    """n disks of about 30 px radius, |cos| of the viewing angle log-uniform in [1e-4, 1e-2]."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(18.0, 30.0, n)
    means = np.stack([rng.uniform(-0.4, 0.4, n) * z, rng.uniform(-0.3, 0.3, n) * z, z], -1)
    view = means / np.linalg.norm(means, axis=1, keepdims=True)
    side = np.cross(view, rng.standard_normal((n, 3)))
    side /= np.linalg.norm(side, axis=1, keepdims=True)
    cos = np.exp(rng.uniform(np.log(1e-4), np.log(1e-2), n)) * rng.choice([-1.0, 1.0], n)
    normal = cos[:, None] * view + np.sqrt(1 - cos[:, None] ** 2) * side
    # rotation e_z -> normal, then a spin about it
    q = np.concatenate([1 + normal[:, 2:], -normal[:, 1:2], normal[:, :1], np.zeros((n, 1))], 1)
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    half = rng.uniform(0, np.pi, n)
    spin = np.stack([np.cos(half), 0 * half, 0 * half, np.sin(half)], -1)
    q = np.stack([q[:, 0] * spin[:, 0] - q[:, 3] * spin[:, 3], q[:, 1] * spin[:, 0] + q[:, 2] * spin[:, 3],
                  q[:, 2] * spin[:, 0] - q[:, 1] * spin[:, 3], q[:, 3] * spin[:, 0] + q[:, 0] * spin[:, 3]], -1)
    scales = np.exp(rng.uniform(np.log(2.0), np.log(5.0), (n, 2)))
    f = np.float32
    sc = Scene(means.astype(f), scales.astype(f), np.ascontiguousarray(q, f), rng.uniform(0.1, 0.6, n).astype(f),
               rng.uniform(0, 1, (n, 3)).astype(f), rng.standard_normal((n, c)).astype(f))
    return sc, scenes.pinhole(200, 150, f=200.0)


def quat_gradients(tw):
    sc, cam = edge_on()
    t = to_dev(sc)
    launch = (0, 0, 0, 0, tw)
    _, ws = render(t, cam, 8, "ellipse", "topk", launch=launch)
    g = {k: torch.tensor(v, device=DEV) for k, v in scenes.upstream(cam.height, cam.width, sc.c, seed=3).items()}
    got = psm.backward(t["means"], t["scales"], t["quats"], t["opacity"], t["rgb"], t["feat"], cam, ws, g, 8,
                       "ellipse", "topk", launch=launch)
    return got["quats"].cpu().numpy()


@pytest.mark.parametrize("tw", [8, 16, 32, 64])
def test_edge_on_rotation_gradients_keep_their_sums(tw):
    require_gpu()
    with open(GOLDEN) as f:
        want = np.array(json.load(f)[str(tw)], np.uint32).view(np.float32).reshape(-1, 4).astype(np.float64)
    got = quat_gradients(tw).astype(np.float64)
    err = np.abs(got - want) / np.maximum(np.abs(want), np.sqrt(np.mean(want ** 2)))
    assert np.linalg.norm(want) > 0 and err.max() <= 2e-6, (err.max(), int(err.max(1).argmax()))
