"""Which launches take two steps, the kernels that take them on either side of
every bound, and the state between two steps where it is stored too."""
import pytest

from paper_2211_15716_amd import diffusion, igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402
from gpu_graph import kernels  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
MARCH = 1 << 21  # forward pairs march from this many inner points on


def _points(n):
    return (n[0] - 2) * (n[1] - 2) * (n[2] - 2)


def _steps_per_launch(n, dtype, zmin):
    """Blocks below the marching bound, marching above it in rows of 16 points
    and more, FP64 and FP32."""
    if _points(n) < (MARCH if zmin is None else zmin):
        return 2
    return 2 if dtype != "f16" and n[0] >= 16 else 1


def _fields(n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    T = (torch.randn(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 1e-2 + 1.7).to(DT[dtype])
    Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 0.5 + 0.25).to(DT[dtype])
    igg.update_halo(T)
    d = [1.0 / (m - 1) for m in n]
    return T, Ci, (1.0, min(v * v for v in d) / 6.1 / 0.75, *d)


SIZES = [(3, 3, 3), (16, 3, 4), (17, 4, 3), (33, 20, 18), (64, 37, 29), (130, 66, 40), (257, 70, 23), (523, 33, 20),
         (107, 103, 101)]


# blocks of 16 x 8 x 8 and (from 2^20 points on) of 32 x 8 x 8, marching rows of
# whole and of broken vectors
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("zmin", [0, None])
def test_pair_with_the_state_between(n, periods, dtype, zmin):
    """diffusion_step_pair with and without mid against two diffusion_step
    calls: T_{n+1} and T_{n+2}, every point; Ci without a valid halo; FP16 with
    stochastic rounding at two counters.  Refused where pairs do not apply."""
    say("pair with mid", n, periods, dtype, zmin)
    with grid(n, periods, zmarch_min=zmin):
        T, Ci, c = _fields(n, dtype)
        assert igg.steps_per_launch(T) == _steps_per_launch(n, dtype, zmin)
        rnd = [igg.rounding("stochastic", 3, 7 + q) if dtype == "f16" else None for q in (0, 1)]
        one, two = T.clone(), T.clone()
        igg.diffusion_step(one, T, Ci, *c, split=None, rnd=rnd[0])
        igg.diffusion_step(two, one, Ci, *c, split=None, rnd=rnd[1])
        mid, out, alone = T.clone(), T.clone(), T.clone()
        if igg.steps_per_launch(T) == 1:
            with pytest.raises(igg.IggError) as e:
                igg.diffusion_step_pair(out, mid, T, Ci, *c, split=None, rnd=rnd[0])
            assert e.value.code == igg.IGG_ERR_STATE
            return
        igg.diffusion_step_pair(out, mid, T, Ci, *c, split=None, rnd=rnd[0])
        igg.diffusion_step_pair(alone, None, T, Ci, *c, split=None, rnd=rnd[0])
        assert torch.equal(mid, one) and torch.equal(out, two) and torch.equal(alone, two)


def test_where_pairs_do_not_apply(monkeypatch):
    n = (40, 36, 34)
    T = torch.zeros(n[::-1], device="cuda", dtype=torch.float64)
    for periods, overlaps, steps in (((1, 1, 1), (2, 2, 3), 1), ((1, 1, 0), (2, 2, 3), 2), ((0, 0, 0), (3, 4, 5), 2)):
        with grid(n, periods, overlaps, zmarch_min=None):
            assert igg.steps_per_launch(T) == igg.adjoints_per_launch(T) == steps
    with grid(n, dims=(1, 2, 1), zmarch_min=None):
        assert igg.steps_per_launch(T) == igg.adjoints_per_launch(T) == 1
    for key, value in (("IGG_SCHEDULE", "2"), ("IGG_X_EXCHANGE", "halo"), ("IGG_SLAB_PACK", "1")):
        with monkeypatch.context() as m:
            m.setenv(key, value)
            with grid(n, zmarch_min=None):
                assert igg.steps_per_launch(T) == igg.adjoints_per_launch(T) == 1


# inner points just below and at 2^20 (block shapes) and 2^21 (marching)
@pytest.mark.parametrize("n,kernel", [((66, 130, 129), "k_step2_block"), ((66, 130, 130), "k_step2_block"),
                                      ((130, 130, 129), "k_step2_block"), ((130, 130, 130), "k_step2_zmarch")])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
def test_forward_pairs_at_the_bounds(n, kernel, dtype):
    say("forward pair bounds", n, dtype)
    with grid(n, (1, 0, 1), zmarch_min=None):
        T, Ci, c = _fields(n, dtype)
        march = kernel == "k_step2_zmarch"
        assert igg.steps_per_launch(T) == (1 if march and dtype == "f16" else 2)
        rnd = igg.rounding("stochastic", 3, 0) if dtype == "f16" else None
        x, y = T.clone(), T.clone()
        names = kernels(lambda: igg.diffusion_run(x, y, Ci, *c, 10, split=None, rnd=rnd, graph=False))
        if march and dtype == "f16":
            assert len(names) == 10
        else:
            assert len(names) == 6 and all(kernel in k for k in names[1:5])
        a, b = T.clone(), T.clone()
        for it in range(10):
            igg.diffusion_step(b, a, Ci, *c, split=None,
                               rnd=igg.rounding("stochastic", 3, it) if dtype == "f16" else None)
            a, b = b, a
        out = igg.diffusion_run(x, y, Ci, *c, 10, split=None, rnd=rnd, graph=False)
        assert torch.equal(out, a) and torch.equal(y, b)


# FP64: blocks below 3 * 2^18 inner points, marching above; FP32: blocks below
# 2^19, single steps below 7 * 2^18, marching above
@pytest.mark.parametrize("n,dtype,kernel", [((98, 96, 88), "f64", "k_adj2_block"), ((98, 96, 92), "f64", "k_adj2_zmarch"),
                                            ((82, 82, 82), "f32", "k_adj2_block"), ((84, 82, 82), "f32", None),
                                            ((124, 124, 124), "f32", None), ((126, 124, 124), "f32", "k_adj2_zmarch")])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 1, 0)])
def test_adjoint_pairs_at_the_bounds(n, dtype, kernel, periods):
    say("adjoint pair bounds", n, dtype, periods)
    with grid(n, periods, zmarch_min=None):
        T0, Ci, c = _fields(n, dtype)
        g = torch.Generator(device="cuda")
        g.manual_seed(9)
        lam, gCi = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g).to(DT[dtype]) for _ in range(2))
        for d, per in enumerate(periods):
            if not per:
                for q in (0, n[d] - 1):
                    lam.select(2 - d, q).zero_()
        igg.update_halo(lam, Ci)
        assert igg.adjoints_per_launch(lam) == (1 if kernel is None else 2)
        T1, mid, one, two = T0.clone(), *(torch.zeros_like(lam) for _ in range(3))
        g1, g2 = gCi.clone(), gCi.clone()
        igg.diffusion_step(T1, T0, Ci, *c, split=None)
        igg.diffusion_step_adjoint(mid, lam, T1, Ci, g1, *c, split=None)
        igg.diffusion_step_adjoint(one, mid, T0, Ci, g1, *c, split=None)
        if kernel is None:
            with pytest.raises(igg.IggError):
                igg.diffusion_step_adjoint_pair(two, lam, T0, Ci, g2, *c, split=None)
            return
        igg.diffusion_step_adjoint_pair(two, lam, T0, Ci, g2, *c, split=None)
        assert torch.equal(two, one) and torch.equal(g2, g1)
        names = kernels(lambda: igg.diffusion_step_adjoint_pair(two, lam, T0, Ci, g2, *c, split=None))
        assert len(names) == 1 and kernel in names[0]


# blocks in both sweeps; marching; FP32 with pairs in the forward sweep alone
# (whose launches store the states between)
@pytest.mark.parametrize("n,dtype,zmin", [((40, 36, 34), "f64", None), ((43, 36, 34), "f32", None),
                                          ((41, 30, 28), "f64", 0), ((40, 30, 29), "f32", 0),
                                          ((90, 84, 82), "f32", None)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
def test_gradient_with_pairs(n, dtype, zmin, periods, monkeypatch):
    nt = 13
    with grid(n, periods, zmarch_min=zmin):
        T0, Ci, c = _fields(n, dtype)
        igg.update_halo(Ci)
        Tobs = (T0 + 0.25 * Ci).to(DT[dtype])
        prob = diffusion.Problem(*c)
        for sched in (("periodic", 4), ("store_all",), ("binomial", 3), ("sqrt",)):
            say("gradient with pairs", n, dtype, zmin, periods, sched)
            L, gT, gC, sw = diffusion.loss_and_grad(T0, Ci, Tobs, prob, nt, sched)
            with monkeypatch.context() as m:
                m.setattr(igg, "adjoints_per_launch", lambda T: 1)
                m.setattr(igg, "steps_per_launch", lambda T: 1)
                L1, gT1, gC1, one = diffusion.loss_and_grad(T0, Ci, Tobs, prob, nt, sched)
            assert sw.pairs and not one.pairs and one.adjoint_launches == nt
            assert sw.adjoints == one.adjoints == nt and sw.advance_launches < one.advance_launches
            assert (sw.adjoint_launches < nt) == (igg.adjoints_per_launch(T0) == 2)
            assert L == L1 and torch.equal(gT, gT1) and torch.equal(gC, gC1)
