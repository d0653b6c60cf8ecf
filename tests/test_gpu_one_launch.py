"""The step in one launch (the default on one rank) against the same step as
a chain of launches with a separate halo update (IGG_SCHEDULE=2)."""
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}


# the smallest rows, rows of broken vectors of every remainder, rows a few
# points past one tile and past half a tile of each type (64, 128 and 256
# points), tall and flat grids
@pytest.mark.parametrize("n", [(5, 5, 6), (17, 7, 6), (33, 20, 18), (67, 37, 29), (130, 66, 40), (257, 70, 23),
                               (259, 40, 50), (523, 33, 20)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0), (0, 0, 1), (1, 1, 0), (0, 1, 1)])
@pytest.mark.parametrize("zmin", [0, None])
def test_one_launch_equals_the_chain(n, periods, zmin, monkeypatch):
    """Every point of T2, halos and edges included, bit for bit, from fields
    without valid halos and a T2 holding other values, split and unsplit,
    overlaps of 2 and wider ones, bases not aligned to a vector."""
    say("one launch", n, periods, zmin)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    d = [1.0 / (m - 1) for m in n]
    dt = min(v * v for v in d) / 6.1 / 0.75
    size = n[0] * n[1] * n[2]

    def field(dtype, lo, hi, shift):
        flat = torch.rand(size + 8, device="cuda", dtype=torch.float64, generator=g) * (hi - lo) + lo
        return flat.to(dtype)[shift:shift + size].view(n[::-1])

    for ol in ((2, 2, 2), (3, 2, 4)):
        for name, dtype in DT.items():
            T, Ci, Z = field(dtype, 1.6, 1.8, 1), field(dtype, 0.25, 0.75, 3), field(dtype, 0.0, 1.0, 2)
            for rnd in (None, igg.rounding("stochastic", 3, 5)) if name == "f16" else (None,):
                for split in (None, (16, 5, 4)):
                    out = []
                    for sched in ("2", None):
                        if sched is None:
                            monkeypatch.delenv("IGG_SCHEDULE", raising=False)
                        else:
                            monkeypatch.setenv("IGG_SCHEDULE", sched)
                        with grid(n, periods, ol, zmarch_min=zmin):
                            T2 = Z.clone()
                            igg.diffusion_step(T2, T, Ci, 1.0, dt, *d, split=split, rnd=rnd)
                            out.append(T2)
                    assert torch.equal(out[0], out[1]), (ol, name, rnd is not None, split)


def test_small_and_marching_kernels_agree_at_the_rule():
    """The bytes at which the small-grid kernel hands over to the z-march
    (88 MiB in three arrays): both sides of the line, both kernels."""
    for n in ((150, 160, 160), (165, 160, 160)):
        say("rule", n)
        d = [1.0 / (m - 1) for m in n]
        T = torch.rand(n[::-1], device="cuda", dtype=torch.float64) + 1.0
        Ci = torch.rand(n[::-1], device="cuda", dtype=torch.float64) * 0.5 + 0.25
        out = []
        for zmin in (None, 0, 1 << 40):
            with grid(n, (1, 1, 1), zmarch_min=zmin):
                T2 = torch.zeros_like(T)
                igg.diffusion_step(T2, T, Ci, 1.0, 1e-6, *d)
                out.append(T2)
        assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
