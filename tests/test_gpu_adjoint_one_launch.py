"""The adjoint step in one launch (the default on one rank) against the chain
with a separate halo update (IGG_SCHEDULE=2)."""
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


# the smallest rows, broken vectors of every remainder, rows just past one
# tile of each width (128 and 256 points), and one that takes half-wide tiles
@pytest.mark.parametrize("n", [(5, 5, 6), (17, 7, 6), (67, 37, 29), (130, 66, 20), (257, 40, 13), (259, 20, 12),
                               (300, 33, 20)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0), (0, 0, 1), (1, 1, 0), (0, 1, 1)])
@pytest.mark.parametrize("zmin", [0, None])
def test_one_launch_equals_the_chain(n, periods, zmin, monkeypatch):
    """lam_n (every point, edges too) and gCi, bit for bit, both forms, from
    fields without valid halos and outputs holding other values."""
    say("adjoint one launch", n, periods, zmin)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    d = [1.0 / (m - 1) for m in n]
    dt = min(v * v for v in d) / 6.1 / 0.75
    size = n[0] * n[1] * n[2]
    for ol in ((2, 2, 2), (3, 2, 4)):
        for dtype in (torch.float64, torch.float32):
            f = [torch.rand(size + 8, device="cuda", dtype=torch.float64, generator=g).to(dtype)[q:q + size].view(n[::-1])
                 for q in range(5)]
            for step in (igg.diffusion_step_adjoint, igg.diffusion_flux_step_adjoint):
                for split in (None, (16, 5, 5)):
                    out = []
                    for sched in ("2", None):
                        if sched is None:
                            monkeypatch.delenv("IGG_SCHEDULE", raising=False)
                        else:
                            monkeypatch.setenv("IGG_SCHEDULE", sched)
                        with grid(n, periods, ol, zmarch_min=zmin):
                            ln, gC = f[0].clone(), f[4].clone()
                            step(ln, f[1], f[2], f[3], gC, 1.0, dt, *d, split=split)
                            out.append((ln, gC))
                    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), (ol, dtype, split)
