"""Pair lists at the edges of the key stage's launch forms, bit-exact against
the oracle: the one-block sorts (surfel counts and pair capacities on both sides
of their bounds, pairs that fill one LDS chunk and more, tile ids of one and
two digits) and the wave-wide counting and emission of tall and wide
footprints (surfels covering hundreds of tiles next to single-tile ones)."""
import numpy as np
import pytest

from gpu_helpers import render, require_gpu, to_dev
from paper_2604_10982_amd import psm, scenes

pytestmark = pytest.mark.gpu


def _check(orc, sc, cam, mode, capacity, tw=16):
    t = to_dev(sc)
    _, ws = render(t, cam, 4, mode, "topk", capacity=capacity, launch=(0, 0, 0, 0, tw))
    got = psm.read_pairs(ws, psm.camera_struct(cam), psm.config_struct(4, mode, "topk", tile_w=tw))
    ref = orc.keystage(sc, cam, mode, tile=(tw, 256 // tw))
    np.testing.assert_array_equal(got["count"].numpy(), ref["count"])
    assert got["P"] == ref["P"]
    np.testing.assert_array_equal(got["tile"].numpy(), ref["tile"])
    np.testing.assert_array_equal(got["id"].numpy(), ref["id"])
    st = got["stats"]
    assert st.visible == int((ref["cull"] == 0).sum())
    return ref["P"]


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 16384, 16385])
def test_depth_sort_bounds(orc, n):
    require_gpu()
    sc = scenes.uniform_box(n, 8, seed=n)
    sc.means[: n // 3, 2] = sc.means[0, 2]  # equal depths: ties by id
    _check(orc, sc, scenes.pinhole(200, 120), "ellipse", 8 * n + 4096)


@pytest.mark.parametrize("size", [(16, 16), (250, 250), (600, 400)])  # 1, 256 and 950 tiles
@pytest.mark.parametrize("capacity", [32768, 32769])
def test_pair_sort_bounds(orc, size, capacity):
    require_gpu()
    sc = scenes.uniform_box(4000, 8, seed=3, scale_mu=np.log(0.02 if size[0] > 300 else 0.12))
    p = _check(orc, sc, scenes.pinhole(*size), "ellipse", capacity)
    assert p <= 32768
    if size == (250, 250):
        assert p > 16384  # more than one chunk of the one-block sort


@pytest.mark.parametrize("mode", ["sphere", "aabb", "ellipse"])
@pytest.mark.parametrize("tw", [8, 16, 64])
def test_wide_footprints(orc, mode, tw):
    require_gpu()
    sc = scenes.uniform_box(3000, 8, seed=9, xy=2.0, z=(0.5, 8.0))
    rng = np.random.default_rng(2)
    sc.scales[:] = np.exp(rng.uniform(np.log(0.005), np.log(1.5), sc.scales.shape))
    _check(orc, sc, scenes.pinhole(1111, 1203), mode, None, tw)
