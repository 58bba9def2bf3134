"""Label logits by 16-byte loads or, where an array starts off that alignment,
by single channels: the channels are summed in the same order, so labels are
the same bits, for channel counts with and without a remainder of 16 and
surfel counts around a wave's 16."""
import pytest
import torch

from gpu_helpers import DEV, TORCH_DTYPES, require_gpu
from paper_2604_10982_amd import psm
from test_gpu_labels import T, queries, surfels

pytestmark = pytest.mark.gpu


def _off(t):
    """The same values one element off the allocation's alignment."""
    flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
    flat[1:] = t.reshape(-1)
    return flat[1:].view(t.shape)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,nq,c", [(1, 3, 4), (15, 16, 16), (17, 33, 20), (200, 64, 48), (65, 130, 60)])
def test_labels_same_bits_at_any_alignment(n, nq, c, dtype):
    require_gpu()
    means, f = surfels(n, c)
    qf, qm, qp = (T(a) for a in queries(nq, c))
    tf = T(f).to(TORCH_DTYPES[dtype]).contiguous()
    ref = psm.instance_labels(T(means), tf, qf, qm, qp)
    assert torch.isfinite(ref).all()
    for a, b in ((_off(tf), qf), (tf, _off(qf)), (_off(tf), _off(qf))):
        assert torch.equal(psm.instance_labels(T(means), a, b, qm, qp), ref)
