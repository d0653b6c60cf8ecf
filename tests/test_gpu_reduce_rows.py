"""Reductions and the adjoint seed over rows of every remainder of a vector,
and the one-launch halo update of mixed fields."""
import math

import numpy as np
import pytest

import oracle
from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}


# inner rows of 1 to 9 points, of one and two passes of a wave (64 vectors of
# 2, 4 or 8 points) and a few more, more rows than waves take in one turn
@pytest.mark.parametrize("n", [(3, 3, 3), (4, 5, 3), (9, 4, 6), (11, 40, 30), (130, 9, 8), (131, 170, 160),
                               (517, 6, 5), (1031, 5, 4)])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
def test_reductions_and_seed(n, dtype):
    """Maxima and minima exact; sums within a rounding per point of FP64 of
    the exactly rounded sum; the no-allocation form and the seed's loss with
    the same bits as igg.reduce."""
    say("reduce", n, dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    a = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) - 0.4).to(DT[dtype])
    b = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) + 0.5).to(DT[dtype])
    x, y = a.double().cpu().numpy(), b.double().cpu().numpy()
    xi, yi = x[1:-1, 1:-1, 1:-1].ravel(), y[1:-1, 1:-1, 1:-1].ravel()
    with grid(n, (1, 1, 1)):
        out = torch.zeros(1, device="cuda", dtype=torch.float64)

        def both(op, two):
            v = igg.reduce(op, a, b if two else None)
            igg.reduce_noalloc(op, a, out, b if two else None)
            assert out.item() == v or (math.isnan(v) and math.isnan(out.item()))
            return v

        assert both(igg.RED_MAX, False) == x.max() and both(igg.RED_MIN, False) == x.min()
        assert both(igg.RED_MAX_ABS, False) == np.abs(xi).max()
        assert both(igg.RED_MAX_ABS_DIFF, True) == np.abs(xi - yi).max()
        for op, two, t in ((igg.RED_SUM, False, xi), (igg.RED_SUM_RATIO, True, xi / yi), (igg.RED_DOT, True, xi * yi),
                           (igg.RED_HALF_SQDIFF, True, 0.5 * (xi - yi) ** 2)):
            tol = 2.0 ** -53 * (len(t) + 1) * np.abs(t).sum()
            assert abs(both(op, two) - math.fsum(t)) <= tol, op
        a[0, 0, 0] = float("nan")
        assert math.isnan(both(igg.RED_MAX, False)) and math.isnan(both(igg.RED_MIN, False))
        a[0, 0, 0] = 0
        lam = torch.full_like(a, 7.0)
        L = igg.adjoint_seed(lam, a, b, halo=False, loss=True)
        assert L == igg.reduce(igg.RED_HALF_SQDIFF, a, b)
        want = torch.zeros_like(a)
        c = torch.float64 if dtype == "f64" else torch.float32
        want[1:-1, 1:-1, 1:-1] = (a.to(c) - b.to(c)).to(a.dtype)[1:-1, 1:-1, 1:-1]
        assert torch.equal(lam, want)


@pytest.mark.parametrize("n", [(3, 3, 3), (5, 4, 6), (18, 9, 7), (67, 30, 20)])
@pytest.mark.parametrize("periods", [(1, 1, 1), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (0, 1, 1), (0, 0, 0)])
@pytest.mark.parametrize("extra", [0, 2])
def test_halo_of_mixed_fields(n, periods, extra):
    """One call with cell and face fields of three types against the oracle's
    dimension-ordered halo update, every point (edges and corners too)."""
    say("halo", n, periods, extra)
    n = tuple(m + extra for m in n)
    ol = (2 + extra, 2, 2 + extra // 2)
    rng = np.random.default_rng(sum(n))
    shapes = [n, (n[0] + 1, n[1], n[2]), (n[0], n[1] + 1, n[2]), (n[0], n[1], n[2] + 1), n, n]
    types = [torch.float64, torch.float64, torch.float32, torch.float16, torch.float32, torch.float16]
    fields = [torch.from_numpy(rng.uniform(size=s[::-1])).to("cuda").to(t) for s, t in zip(shapes, types)]
    want = []
    for f, s in zip(fields, shapes):
        h = f.double().cpu().numpy().copy()
        oracle.halo(h, tuple(o + (m - c) for o, m, c in zip(ol, s, n)), periods)
        want.append(h)
    with grid(n, periods, ol):
        igg.update_halo(*fields)
        for f, h in zip(fields, want):
            assert np.array_equal(f.double().cpu().numpy(), h)
