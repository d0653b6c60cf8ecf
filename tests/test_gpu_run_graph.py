"""The time loop's kept graph (diffusion_run with graph=True), which is
captured on the second call in a row with the same arguments, buffers
included, and replayed from then on."""
import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}


def _problem(n, dtype="f64"):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(n))
    T0 = (torch.randn(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 1e-2 + 1.7).to(DT[dtype])
    Ci = (torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) * 0.5 + 0.25).to(DT[dtype])
    igg.update_halo(T0, Ci)
    d = [1.0 / (m - 1) for m in n]
    return T0, Ci, (1.0, min(v * v for v in d) / 6.1 / 0.75, *d)


def _steps(T0, Ci, c, nt, split=None):
    """T_nt and T_{nt-1} by single steps."""
    a, b = T0.clone(), T0.clone()
    for _ in range(nt):
        igg.diffusion_step(b, a, Ci, *c, split=split)
        a, b = b, a
    return a, b


@pytest.mark.parametrize("nt", [8, 37])
def test_a_captured_stream_records_the_steps(nt):
    """diffusion_run with graph=True inside a caller's capture records its
    launches there, on the first call with these arguments and on later ones,
    which outside a capture would replay the kept graph: every replay of the
    caller's graph advances the state."""
    n = (40, 36, 34)
    with grid(n, zmarch_min=None):
        T0, Ci, c = _problem(n)
        T, T2 = T0.clone(), T0.clone()
        for warm in (0, 2):
            say("capture", nt, warm)
            for _ in range(warm):
                igg.diffusion_run(T, T2, Ci, *c, nt, graph=True)
            g = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(g):
                out = igg.diffusion_run(T, T2, Ci, *c, nt, graph=True)
            for replay in range(3):
                x = T0 * (1.0 + 0.125 * replay)
                want, before = _steps(x, Ci, c, nt)
                T.copy_(x)
                T2.copy_(x)
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, want), (warm, replay)
                assert torch.equal(T2 if out is T else T, before), (warm, replay)
