"""The tiles of the flux step and of the adjoint across rows of every fit: 64, 128
and 256 points wide, begun at a whole vector or at the first inner point; and
which kernel short rows take."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402
from gpu_graph import kernels, launches  # noqa: E402


def _fields(n, dtype, ranks=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))

    def rand():
        return [(torch.rand(n[::-1], device="cuda", dtype=torch.float32, generator=g) + 0.5).to(dtype)
                for _ in range(ranks)]

    d = [1.0 / (m - 1) for m in n]
    return [rand() for _ in range(5)], (1.0, min(v * v for v in d) / 6.1 / 1.5, *d)


def _outputs(n, periods, dtype, zmin, dims=(1, 1, 1)):
    """Every output of a flux step and of one adjoint step of either form."""
    ranks = dims[0] * dims[1] * dims[2]
    with grid(n, periods, zmarch_min=zmin, dims=dims):
        F, c = _fields(n, dtype, ranks)
        q = [diffusion.FluxProblem.face_arrays(t) for t in F[0]]
        qs = [[x[k] for x in q] for k in range(3)]
        igg.diffusion_flux_step_ranks(F[0], F[1], F[2], *qs, *c)
        out = F[0] + qs[0] + qs[1] + qs[2]
        for step in (igg.diffusion_step_adjoint_ranks, igg.diffusion_flux_step_adjoint_ranks):
            lam, g = [t.clone() for t in F[3]], [t.clone() for t in F[4]]
            step(lam, F[3], F[1], F[2], g, *c, split=None)
            out += lam + g
        torch.cuda.synchronize()
    return out


# rows of 2 to 64 inner points, of one tile and a point more or less, where a
# tile from the first inner point on saves one, and of several tiles
@pytest.mark.parametrize("nx", [4, 23, 34, 65, 66, 67, 68, 129, 130, 131, 132, 162, 163, 194, 257, 258, 259, 260, 386,
                                387, 514])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("periods,dims", [((1, 1, 1), (1, 1, 1)), ((0, 1, 0), (1, 1, 1)), ((1, 0, 1), (2, 1, 1))])
def test_tiles_equal_one_point_per_thread(nx, dtype, periods, dims):
    """Every region through the z-march kernels, against the kernels without
    tiles that small grids take: all points, halos included."""
    n = (nx, 21, 9)
    say("row tiles", n, dtype, periods, dims)
    for a, b in zip(_outputs(n, periods, dtype, 0, dims), _outputs(n, periods, dtype, None, dims)):
        assert torch.equal(a, b)


# a row of the bound and one more, with more points than the bounds in bytes
@pytest.mark.parametrize("form,dtype,row", [("adjoint", torch.float64, 40), ("adjoint", torch.float32, 64),
                                            ("flux", torch.float64, 40), ("flux", torch.float32, 88)])
def test_short_rows_take_the_small_grid_kernel(form, dtype, row):
    for more in (0, 1):
        n = (row + 2 + more, 450, 210 if row < 88 else 150)
        say("short rows", form, dtype, n)
        with grid(n, (1, 1, 0), zmarch_min=None):
            F, c = _fields(n, dtype)
            F = [f[0] for f in F]
            q = diffusion.FluxProblem.face_arrays(F[0])

            def call():
                if form == "adjoint":
                    igg.diffusion_step_adjoint(*F, *c)
                else:
                    igg.diffusion_flux_step(*F[:3], *q, *c)

            call()
            name = kernels(call)[0]
            assert ("_small" in name) == (more == 0) and ("_zmarch" in name) == (more == 1), name


# the last plane with which five arrays of inner points fit 84 MiB (FP64 in rows
# that fill tiles of 128 points) or 96, and one plane more
@pytest.mark.parametrize("dtype,nx,nz", [(torch.float64, 130, 136), (torch.float64, 136, 148),
                                         (torch.float32, 130, 309)])
@pytest.mark.parametrize("step", [igg.diffusion_step_adjoint, igg.diffusion_flux_step_adjoint])
def test_adjoint_of_the_small_grid_bound(step, dtype, nx, nz):
    for more in (0, 1):
        n = (nx, 130, nz + more)
        say("adjoint at the small-grid bound", dtype, n)
        with grid(n, (1, 1, 1), zmarch_min=None):
            F, c = _fields(n, dtype)
            F = [f[0] for f in F]
            step(*F, *c)
            name = kernels(lambda: step(*F, *c))[0]
            assert ("_small" in name) == (more == 0) and ("_zmarch" in name) == (more == 1), name


# 32 tiles of 128 x 4 points over 256 planes: fewer than 2048 work-groups of 6
# planes, so the least chunk, 4 planes
@pytest.mark.parametrize("step", [igg.diffusion_step_adjoint, igg.diffusion_flux_step_adjoint])
def test_adjoint_marches_four_planes_at_least(step):
    n = (130, 130, 258)
    say("adjoint chunks", n)
    with grid(n, (1, 1, 1), zmarch_min=None):
        F, c = _fields(n, torch.float64)
        F = [f[0] for f in F]
        step(*F, *c)
        name, groups = launches(lambda: step(*F, *c))[0]
        assert "k_adj_zmarch" in name and groups == 32 * 256 // 4, (name, groups)


@pytest.mark.parametrize("form,dtype,row", [("adjoint", torch.float64, 36), ("adjoint", torch.float32, 36),
                                            ("flux", torch.float64, 40), ("flux", torch.float32, 20)])
def test_short_rows_of_ranks_take_the_box_kernel(form, dtype, row):
    for more in (0, 1):
        n = (row + 2 + more, 450, 300)
        say("short rows of ranks", form, dtype, n)
        with grid(n, (1, 1, 0), zmarch_min=None, dims=(2, 1, 1)):
            F, c = _fields(n, dtype, 2)
            q = [diffusion.FluxProblem.face_arrays(t) for t in F[0]]

            def call():
                if form == "adjoint":
                    igg.diffusion_step_adjoint_ranks(*F, *c, split=None)
                else:
                    igg.diffusion_flux_step_ranks(*F[:3], *[[x[k] for x in q] for k in range(3)], *c)

            call()
            name = kernels(call)[0]
            assert ("_boxes" in name) == (more == 0) and ("_zmarch" in name) == (more == 1), name
