"""Kernel timing switched on or off between the halves of a sweep: the sweep
keeps the plan it was made with, pairs of steps or single ones."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


# blocks (pairs below the marching bounds) and, with every region marching,
# the z-march kernels; the FP32 size has pairs in the forward sweep alone
@pytest.mark.parametrize("n,dtype,zmin", [((40, 36, 34), torch.float64, None), ((40, 36, 34), torch.float32, 0),
                                          ((90, 84, 82), torch.float32, None)])
@pytest.mark.parametrize("on_first", [False, True])
def test_timing_may_change_between_forward_and_backward(n, dtype, zmin, on_first):
    nt = 13
    pts = (n[0] - 2) * (n[1] - 2) * (n[2] - 2)
    say("sweep timing", n, dtype, zmin, on_first)
    with grid(n, (1, 0, 1), zmarch_min=zmin):
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        T0 = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) + 1.0).to(dtype)
        Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 0.5 + 0.25).to(dtype)
        igg.update_halo(T0, Ci)
        d = [1.0 / (m - 1) for m in n]
        prob = diffusion.Problem(1.0, min(v * v for v in d) / 6.1 / 0.75, *d)
        w = torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g).to(dtype)

        def grads(switch):
            a, c = T0.clone().requires_grad_(), Ci.clone().requires_grad_()
            if switch:
                igg.timing_enable(on_first)
            out = diffusion.DiffusionSolve.apply(a, c, prob, nt, ("periodic", 4))
            if switch:
                igg.timing_read()
                igg.timing_enable(not on_first)
            (out * w).sum().backward()
            return a.grad, c.grad

        want = grads(False)
        got = grads(True)
        ms, launches, points, _ = igg.timing_read()
        igg.timing_enable(False)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        if not on_first:  # the reverse half was timed: nt adjoint steps at least
            assert ms > 0.0 and launches > 0 and points >= nt * pts and points % pts == 0
