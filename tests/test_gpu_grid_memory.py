"""Device memory the grid holds."""
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


def _held(n, dims=(1, 1, 1)):
    """Bytes of device memory the grid's resources take, and those still gone
    after it."""
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with grid(n, zmarch_min=None, dims=dims):
        igg.timing_enable(True)  # makes the grid's device resources
        held = free - torch.cuda.mem_get_info()[0]
    return held, free - torch.cuda.mem_get_info()[0]


def test_one_rank_holds_no_halo_buffers(monkeypatch):
    """A rank that is its own neighbour fills its halo from its own points: the
    32 send and receive planes (FP64, of the largest field) are allocated where
    the slabs pack, and for several ranks."""
    say("grid memory")
    _held((16, 16, 16))  # what the runtime allocates once
    n = (600, 500, 8)
    plane = 601 * 501 * 8
    held, after = _held(n)
    assert held < 8 * plane and after < plane
    monkeypatch.setenv("IGG_SLAB_PACK", "1")
    held, after = _held(n)
    assert held >= 32 * plane and after < 8 * plane
    monkeypatch.delenv("IGG_SLAB_PACK")
    held, after = _held(n, (1, 2, 1))
    assert held >= 64 * plane and after < 8 * plane
