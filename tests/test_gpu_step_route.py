"""Which kernels a step on one rank takes (the small-grid kernel by the bytes of
the inner points, slabs and z-march above), and the bits of the general path
where the slabs leave a thin region or none."""
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402
from gpu_graph import kernels  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
MIB = {"f64": 90, "f32": 90, "f16": 25}  # of three arrays


def _fields(n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    T = (torch.rand(n[::-1], device="cuda", dtype=torch.float32, generator=g) + 1.0).to(DT[dtype])
    Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float32, generator=g) * 0.5 + 0.25).to(DT[dtype])
    T2 = (torch.rand(n[::-1], device="cuda", dtype=torch.float32, generator=g) + 1.0).to(DT[dtype])
    d = [1.0 / (m - 1) for m in n]
    return T2, T, Ci, (1.0, min(v * v for v in d) / 6.1 / 0.75, *d)


# either side of the bound for each type, within 3% of it, and planes of four
# and of five inner rows at any size
@pytest.mark.parametrize("dtype,n", [("f64", (158, 160, 160)), ("f64", (161, 160, 160)), ("f32", (200, 202, 198)),
                                     ("f32", (200, 206, 200)), ("f16", (176, 160, 160)), ("f16", (178, 160, 160)),
                                     ("f64", (1500, 6, 1500)), ("f64", (1200, 7, 1200))])
def test_the_kernel_does_not_depend_on_the_split(dtype, n):
    """One launch in all cases: of the small-grid kernel up to the bound, else
    of the z-march kernel."""
    points = (n[0] - 2) * (n[1] - 2) * (n[2] - 2)
    small = n[1] <= 6 or 3 * points * DT[dtype].itemsize <= MIB[dtype] << 20
    with grid(n, (1, 0, 1), zmarch_min=None):
        T2, T, Ci, c = _fields(n, dtype)
        igg.diffusion_step(T2, T, Ci, *c)
        for split in (None, (16, 2, 2), (16, 40, 2), (16, n[1] // 2, n[2] // 2 - 4)):
            say("step route", dtype, n, split)
            names = kernels(lambda: igg.diffusion_step(T2, T, Ci, *c, split=split))
            assert len(names) == 1
            assert ("k_step_small" if small else "k_step_zmarch") in names[0], (split, names)


def _same_as_general(n, periods, overlaps, dtype, zmin, monkeypatch, want):
    """The default step, one launch of the kernel `want`, against one chain of
    step and halo update (schedule 2): every point, halos included."""
    out = []
    rnd = igg.rounding("stochastic", 3, 5) if dtype == "f16" else None
    for sched in (None, "2"):
        with monkeypatch.context() as m:
            if sched:
                m.setenv("IGG_SCHEDULE", sched)
            with grid(n, periods, overlaps, zmarch_min=zmin):
                T2, T, Ci, c = _fields(n, dtype)
                for split in (None, tuple(max(o, 2) for o in overlaps)):
                    igg.diffusion_step(T2, T, Ci, *c, split=split, rnd=rnd)
                    out.append(T2.clone())
                if sched is None:
                    names = kernels(lambda: igg.diffusion_step(T2, T, Ci, *c, split=None, rnd=rnd))
                    assert len(names) == 1 and want in names[0], names
    for o in out[1:]:
        assert torch.equal(o, out[0])


PERIODS = [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0), (1, 1, 0), (0, 0, 1), (0, 1, 1)]


# grids whose z slabs are all there is (with a period in z), or leave one plane
@pytest.mark.parametrize("periods", PERIODS)
@pytest.mark.parametrize("dtype,n", [("f64", (2003, 1012, 4)), ("f32", (4001, 1012, 4)), ("f16", (2203, 1002, 4)),
                                     ("f64", (2003, 1012, 5))])
def test_flat_grids(dtype, n, periods, monkeypatch):
    say("flat", dtype, n, periods)
    want = "k_step_slab" if n[2] == 4 and periods[2] else "k_step_zmarch"
    _same_as_general(n, periods, (2, 2, 2), dtype, None, monkeypatch, want)


# the same on a few thousand points (every grid marches), overlaps above 2 too
@pytest.mark.parametrize("periods", PERIODS)
@pytest.mark.parametrize("n,overlaps", [((43, 20, 13), (2, 2, 2)), ((43, 20, 13), (2, 3, 4)), ((19, 20, 7), (2, 3, 4)),
                                        ((20, 4, 9), (2, 2, 2)), ((21, 9, 3), (3, 5, 2))])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
def test_slabs_only_where_a_period_needs_them(dtype, n, overlaps, periods, monkeypatch):
    say("slabs", dtype, n, overlaps, periods)
    _same_as_general(n, periods, overlaps, dtype, 0, monkeypatch, "k_step_")


# FP16 rows of at most 64 points, whose stochastic stores take one point per
# lane, and one more, against 4-point vectors (every region marched)
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 1, 0), (1, 0, 1)])
@pytest.mark.parametrize("nx", [34, 50, 65, 66, 67])
def test_short_rows_with_stochastic_stores(nx, periods):
    n = (nx, 400, 380)
    say("short rows, stochastic", n, periods)
    out = []
    for zmin in (None, 0):
        with grid(n, periods, zmarch_min=zmin):
            T2, T, Ci, c = _fields(n, "f16")
            for mode, one in (("stochastic", nx <= 66 and zmin is None), ("nearest", False)):
                rnd = igg.rounding(mode, 3, 5)
                igg.diffusion_step(T2, T, Ci, *c, rnd=rnd)
                out.append(T2.clone())
                name = kernels(lambda: igg.diffusion_step(T2, T, Ci, *c, rnd=rnd))[0]
                assert "k_step_zmarchIDF16_Li%dE" % (1 if one else 4) in name, name
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
