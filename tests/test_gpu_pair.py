"""Two steps in one launch (diffusion_run, diffusion.forward): the bits of
single steps, in both buffers, at the edges of the kernels' tiles."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}


# rows of whole and of broken vectors, one and several tiles across (64
# vectors: 128 FP64 or 256 FP32 points), the smallest marching row (16) and
# the smallest grid, columns of one tile and of several, blocks of 16 x 4 x 4
# and (1.1e6 points) of 16 x 8 x 8
@pytest.mark.parametrize("n", [(3, 3, 3), (16, 3, 4), (17, 4, 3), (33, 20, 18), (64, 37, 29), (130, 66, 40),
                               (257, 70, 23), (523, 33, 20), (107, 103, 101)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("zmin", [0, None])
def test_pairs_equal_single_steps(n, periods, dtype, zmin):
    """diffusion_run against a loop of diffusion_step: T_nt and, in the other
    buffer, T_{nt-1}, bit for bit, halos included; Ci without a valid halo
    (no step reads it), T0 without one too; FP16 with stochastic rounding."""
    say("pairs", n, periods, dtype, zmin)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    with grid(n, periods, zmarch_min=zmin):
        T0 = (torch.randn(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 1e-2 + 1.7).to(DT[dtype])
        Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 0.5 + 0.25).to(DT[dtype])
        d = [1.0 / (m - 1) for m in n]
        dt = min(v * v for v in d) / 6.1 / 0.75
        seed = 3 if dtype == "f16" else None

        def rnd(it):
            return None if seed is None else igg.rounding("stochastic", seed, 7 + it)

        for nt in (6, 9, 16):
            a, b = T0.clone(), T0.clone()
            for it in range(nt):
                igg.diffusion_step(b, a, Ci, 1.0, dt, *d, split=None, rnd=rnd(it))
                a, b = b, a
            for graph in (False,) if seed is not None else (False, True, True):
                x, y = T0.clone(), T0.clone()
                out = igg.diffusion_run(x, y, Ci, 1.0, dt, *d, nt, split=None, rnd=rnd(0), graph=graph)
                other = y if out is x else x
                assert (out is x) == (nt % 2 == 0)
                assert torch.equal(out, a) and torch.equal(other, b), (nt, graph)
            out = diffusion.forward(T0.clone(), Ci, nt, 1.0, dt, *d, split=None, sr_seed=seed, counter0=7)
            assert torch.equal(out, a)


def test_fullsize_pairs_equal_single_steps():
    """Tiles of every position at a size the marching kernel is meant for,
    with broken vectors and several rounds of work-groups."""
    n = (301, 257, 203)
    say("pairs", n)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    for dtype in (torch.float64, torch.float32):
        with grid(n, (1, 1, 0), zmarch_min=None):
            T0 = (torch.randn(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 1e-2 + 1.7).to(dtype)
            Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 0.5 + 0.25).to(dtype)
            d = [1.0 / (m - 1) for m in n]
            dt = min(v * v for v in d) / 6.1 / 0.75
            a, b = T0.clone(), T0.clone()
            for _ in range(10):
                igg.diffusion_step(b, a, Ci, 1.0, dt, *d)
                a, b = b, a
            out = diffusion.forward(T0.clone(), Ci, 10, 1.0, dt, *d)
            assert torch.equal(out, a)


def test_refused_calls_stay_refused():
    """T sharing memory with Ci is refused at the step that would write it."""
    n = (40, 36, 34)
    with grid(n, zmarch_min=None):
        T = torch.rand(n[::-1], device="cuda", dtype=torch.float64)
        with pytest.raises(igg.IggError) as e:
            igg.diffusion_run(T, T.clone(), T, 1.0, 1e-5, 0.1, 0.1, 0.1, 20, graph=False)
        assert e.value.code == igg.IGG_ERR_ALIAS
