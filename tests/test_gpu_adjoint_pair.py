"""Two adjoint steps in one launch: the bits of two single steps."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


def _fields(n, periods, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))

    def rand(lo, hi):
        t = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * (hi - lo) + lo).to(dtype)
        igg.update_halo(t)
        return t

    lam, T0, Tobs, Ci, gCi = rand(-1, 1), rand(1, 2), rand(1, 2), rand(0.25, 0.75), rand(-1, 1)
    for d, per in enumerate(periods):
        if not per:
            for k in (0, n[d] - 1):
                lam.select(2 - d, k).zero_()
    return lam, T0, Tobs, Ci, gCi


def _compare(n, periods, dtype):
    lam, T0, _, Ci, gCi = _fields(n, periods, dtype)
    d = [1.0 / (m - 1) for m in n]
    c = (1.0, min(v * v for v in d) / 6.1 / 0.75, *d)
    T1 = T0.clone()
    igg.diffusion_step(T1, T0, Ci, *c, split=None)
    g1, g2 = gCi.clone(), gCi.clone()
    mid, one, two = torch.zeros_like(lam), torch.zeros_like(lam), torch.zeros_like(lam)
    igg.diffusion_step_adjoint(mid, lam, T1, Ci, g1, *c, split=None)
    igg.diffusion_step_adjoint(one, mid, T0, Ci, g1, *c, split=None)
    if igg.adjoints_per_launch(lam) == 1:
        with pytest.raises(igg.IggError):
            igg.diffusion_step_adjoint_pair(two, lam, T0, Ci, g2, *c, split=None)
        return False
    igg.diffusion_step_adjoint_pair(two, lam, T0, Ci, g2, *c, split=None)
    assert torch.equal(two, one)
    assert torch.equal(g2, g1)
    return True


# rows of whole and of broken vectors, one and several tiles across, the
# smallest marching row (16) and the smallest grid, columns of one tile and of
# several; with the default bounds blocks below 2^19 points, marching in FP64
# (107 x 103 x 101) or single steps above
@pytest.mark.parametrize("n", [(3, 3, 3), (16, 3, 4), (17, 4, 3), (33, 20, 18), (64, 37, 29), (130, 66, 40),
                               (257, 70, 23), (523, 33, 20), (107, 103, 101)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0), (1, 0, 0), (0, 1, 1)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("zmin", [0, None])
def test_pair_equals_two_steps(n, periods, dtype, zmin):
    say("adjoint pair", n, periods, dtype, zmin)
    with grid(n, periods, zmarch_min=zmin):
        pts = (n[0] - 2) * (n[1] - 2) * (n[2] - 2)
        march = n[0] >= 16 if zmin == 0 else pts >= 1 << 20 and dtype == torch.float64
        assert _compare(n, periods, dtype) == (march or (zmin is None and pts < 1 << 19))


def test_fullsize_pair_equals_two_steps():
    """Tiles of every position at sizes the marching kernel is meant for."""
    for n in ((301, 257, 203), (256, 256, 256)):
        for dtype in (torch.float64, torch.float32):
            say("adjoint pair", n, dtype)
            with grid(n, (1, 1, 0), zmarch_min=None):
                assert _compare(n, (1, 1, 0), dtype)


def test_gradient_with_pairs_equals_single_steps(monkeypatch):
    n, nt = (70, 41, 33), 11
    for sched in (("periodic", 4), ("store_all",), ("binomial", 3)):
        say("gradient", sched)
        with grid(n, (1, 1, 1)):
            _, T0, Tobs, Ci, _ = _fields(n, (1, 1, 1), torch.float64)
            d = [1.0 / (m - 1) for m in n]
            p = diffusion.Problem(1.0, min(v * v for v in d) / 6.1 / 0.75, *d)
            L, gT, gC, sw = diffusion.loss_and_grad(T0, Ci, Tobs, p, nt, sched)
            with monkeypatch.context() as m:
                m.setattr(igg, "adjoints_per_launch", lambda T: 1)
                L1, gT1, gC1, sw1 = diffusion.loss_and_grad(T0, Ci, Tobs, p, nt, sched)
            assert any(op[0] == "adjoint2" for op in sw.rev) and not any(op[0] == "adjoint2" for op in sw1.rev)
            assert L == L1 and torch.equal(gT, gT1) and torch.equal(gC, gC1)
            assert sw.adjoints == sw1.adjoints == nt
