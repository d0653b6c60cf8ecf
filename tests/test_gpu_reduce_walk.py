"""Reductions and the adjoint seed where a field's vectors meet its rows and
planes: rows of a vector and a point fewer or more, one chunk of a work-group and
several, more chunks than work-groups; nothing outside the region counts."""
import math

import numpy as np
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}


# (3 to 17 points a row around vectors of 2, 4 and 8; chunks of 2048 to 16384
# points; 1024 chunks are 2.1 to 16.8 million points)
@pytest.mark.parametrize("n", [(3, 3, 4), (4, 7, 5), (5, 4, 9), (7, 9, 5), (8, 6, 5), (9, 7, 6), (15, 4, 8),
                               (16, 5, 7), (17, 3, 3), (4093, 5, 4), (64, 64, 17), (172, 171, 160), (262, 259, 257)])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
def test_only_the_region_counts(n, dtype):
    """Sums, absolute maxima and the seed see the inner points only: the halo is
    NaN.  Maxima and minima see every point: the extremes are the field's last
    points.  Sums within a rounding per point of FP64 of the exact sum."""
    say("reduce walk", n, dtype)
    rng = np.random.default_rng(sum(n))
    x, y = (rng.uniform(lo, 1.5, n[::-1]).astype(np.float32) for lo in (-0.4, 0.5))
    a, b = (torch.from_numpy(v).to("cuda").to(DT[dtype]) for v in (x, y))
    x, y = a.double().cpu().numpy(), b.double().cpu().numpy()
    inside = np.zeros(x.shape, bool)
    inside[1:-1, 1:-1, 1:-1] = True
    xi, yi = x[inside], y[inside]
    halo = torch.from_numpy(~inside).to("cuda")
    ah, bh = a.masked_fill(halo, float("nan")), b.masked_fill(halo, float("nan"))
    with grid(n, (1, 1, 1)):
        for op, two, t in ((igg.RED_SUM, False, xi), (igg.RED_SUM_RATIO, True, xi / yi), (igg.RED_DOT, True, xi * yi),
                           (igg.RED_HALF_SQDIFF, True, 0.5 * (xi - yi) ** 2)):
            v = igg.reduce(op, ah, bh if two else None)
            assert abs(v - math.fsum(t)) <= 2.0 ** -53 * (len(t) + 1) * np.abs(t).sum(), op
        assert igg.reduce(igg.RED_MAX_ABS, ah) == np.abs(xi).max()
        assert igg.reduce(igg.RED_MAX_ABS_DIFF, ah, bh) == np.abs(xi - yi).max()
        c = torch.float64 if dtype == "f64" else torch.float32
        for T, O, want in ((None, None, torch.zeros_like(a)), (ah, None, a), (ah, bh, (a.to(c) - b.to(c)).to(a.dtype))):
            lam = torch.full_like(a, 7.0)
            igg.adjoint_seed(lam, T, O, halo=False)
            assert torch.equal(lam, want.masked_fill(halo, 0.0))
        lam = torch.full_like(a, 7.0)
        L = igg.adjoint_seed(lam, ah, bh, halo=False, loss=True)
        assert L == igg.reduce(igg.RED_HALF_SQDIFF, ah, bh)
        for q in range(1, 9):
            e = a.clone()
            e.view(-1)[-q] = 3.0
            assert igg.reduce(igg.RED_MAX, e) == 3.0
            e.view(-1)[-q] = -3.0
            assert igg.reduce(igg.RED_MIN, e) == -3.0
