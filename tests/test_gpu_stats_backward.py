"""The statistics read-back and the backward write no common byte of the
workspace beyond the status block, so a read-back on another stream cannot
change a running backward (nor be changed by it).  Shown without any overlap in
time: a byte that the read-back changed after one backward, and the next
backward changed again, would be written by both.  The scene has a surfel of
more than 64 pairs, so every reduction of the backward runs."""
import pytest
import torch

from gpu_helpers import DEV, require_gpu, to_dev
from paper_2604_10982_amd import psm, scenes
from test_gpu_heavy_reduce import _scene

pytestmark = pytest.mark.gpu

STATUS_BYTES = 256


def test_read_back_and_backward_share_no_memory():
    require_gpu()
    sc, cam, K = _scene(), scenes.pinhole(320, 180, f=240.0), 4
    t = to_dev(sc)
    args = [t[k] for k in ("means", "scales", "quats", "opacity", "rgb", "feat")]
    cs, cfg = psm.camera_struct(cam), psm.config_struct(K)
    _, ws = psm.forward(*args, cam, K)
    assert int(psm.read_pairs(ws, cs, cfg)["count"].max()) > 64
    ws.buf.zero_()  # read_pairs read the statistics already
    psm.forward(*args, cam, K, ws=ws)
    gt = {k: torch.tensor(v, device=DEV) for k, v in scenes.upstream(cam.height, cam.width, sc.c, seed=2).items()}
    first = psm.backward(*args, cam, ws, gt, K)
    after = [ws.buf.clone()]
    st = psm.read_stats(ws, sc.n, cs, cfg, sc.c, ws.capacity)
    after.append(ws.buf.clone())
    second = psm.backward(*args, cam, ws, gt, K)
    after.append(ws.buf.clone())
    assert st.selected_unique > 0
    both = (after[0] != after[1]) & (after[1] != after[2])
    off = (-ws.buf.data_ptr()) % 256
    assert int((after[0] != after[1])[off + STATUS_BYTES:].sum()) > 0  # the read-back's bitmap
    assert int(both[off + STATUS_BYTES:].sum()) == 0
    for k in first:
        assert torch.equal(first[k], second[k]), k
