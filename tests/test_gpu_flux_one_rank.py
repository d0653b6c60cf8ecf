"""The flux form's one-rank path (the default) against the chain with slabs
(IGG_SCHEDULE=2)."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


# the smallest rows, broken vectors of every remainder, rows just past one
# tile of each width, and one that takes half-wide tiles
@pytest.mark.parametrize("n", [(5, 5, 6), (18, 7, 6), (67, 37, 29), (130, 66, 20), (257, 40, 13), (300, 33, 20)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("zmin", [0, None])
def test_one_rank_equals_the_chain(n, periods, zmin, monkeypatch):
    """T2 and the three face fields, every point, bit for bit, from fields
    without valid halos and outputs holding other values."""
    say("flux one rank", n, periods, zmin)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    d = [1.0 / (m - 1) for m in n]
    dt = min(v * v for v in d) / 6.1 / 0.75
    for ol in ((2, 2, 2), (3, 2, 4)):
        for dtype in (torch.float64, torch.float32):
            T, Ci, T2 = (torch.rand(n[::-1], device="cuda", dtype=dtype, generator=g) for _ in range(3))
            q = [torch.rand_like(a) for a in diffusion.FluxProblem.face_arrays(T)]
            out = []
            for sched, split in (("2", None), ("2", (16, 5, 5)), (None, None), (None, (16, 5, 5))):
                if sched is None:
                    monkeypatch.delenv("IGG_SCHEDULE", raising=False)
                else:
                    monkeypatch.setenv("IGG_SCHEDULE", sched)
                with grid(n, periods, ol, zmarch_min=zmin):
                    res = [T2.clone()] + [a.clone() for a in q]
                    igg.diffusion_flux_step(res[0], T, Ci, *res[1:], 1.0, dt, *d, split=split)
                    out.append(res)
            for res in out[1:]:
                assert all(torch.equal(a, b) for a, b in zip(res, out[0])), (ol, dtype)
