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


def _calls(T0, Ci, c, nt, split, want, before, calls=4):
    """The same call again and again on the same buffers, their contents reset:
    the first runs directly, the second captures, the others replay."""
    T, T2 = T0.clone(), T0.clone()
    launches = []
    for call in range(calls):
        T.copy_(T0)
        T2.copy_(T0)
        out = igg.diffusion_run(T, T2, Ci, *c, nt, split=split, graph=True)
        launches.append(igg.timing_read()[1])
        assert torch.ones(100, device="cuda").sum().item() == 100.0
        assert (out is T) == (nt % 2 == 0)
        assert torch.equal(out, want), (nt, call)
        assert torch.equal(T2 if out is T else T, before), (nt, call)
    return launches


@pytest.mark.parametrize("n,split,dtype", [((32, 32, 32), (16, 2, 2), "f64"), ((66, 40, 36), (16, 2, 2), "f32"),
                                           ((48, 40, 36), None, "f64"), ((160, 140, 120), (16, 2, 2), "f64"),
                                           ((40, 34, 30), (16, 2, 2), "f16")])
@pytest.mark.parametrize("periods", [(1, 1, 1), (0, 1, 0)])
@pytest.mark.parametrize("sched", [None, "0", "1", "2", "3"])
def test_repeated_calls_equal_single_steps(n, split, dtype, periods, sched, monkeypatch):
    """Under every schedule, with pairs of steps (the default and schedule 3)
    and without, nt below, at and above what one graph holds."""
    if sched is not None:
        monkeypatch.setenv("IGG_SCHEDULE", sched)
    say("kept graph", n, split, dtype, periods, sched)
    with grid(n, periods, zmarch_min=None):
        T0, Ci, c = _problem(n, dtype)
        assert igg.steps_per_launch(T0) == (2 if sched in (None, "3") else 1)
        for nt in (2, 6, 7, 16, 37, 70):
            want, before = _steps(T0, Ci, c, nt, split)
            _calls(T0, Ci, c, nt, split, want, before)


def test_calls_from_the_second_on_replay_a_graph():
    """Kernel timing counts the launches made directly: all of the first call's,
    and of the later ones only those a graph of 16 steps leaves over."""
    n, nt = (40, 36, 34), 37
    with grid(n, zmarch_min=None):
        T0, Ci, c = _problem(n)
        want, before = _steps(T0, Ci, c, nt)
        igg.timing_enable(True)
        assert _calls(T0, Ci, c, nt, None, want, before) == [nt] + 3 * [nt - 32]
        igg.timing_enable(False)


@pytest.mark.parametrize("where", ["side:300", "inner:300", "halo:300"])
@pytest.mark.parametrize("pack", ["1", "2", "0"])
def test_held_back_stream_in_the_kept_graph(where, pack, monkeypatch):
    """A wait longer than a step put into one stream of the schedules, fork and
    join inside the graph: replays give the bits of single steps."""
    n, nt, split = (260, 140, 72), 7, (16, 2, 2)
    monkeypatch.setenv("IGG_SLAB_PACK", pack)
    monkeypatch.setenv("IGG_SCHEDULE", "2")
    with grid(n, zmarch_min=None):
        T0, Ci, c = _problem(n)
        want, before = _steps(T0, Ci, c, nt, split)
    monkeypatch.setenv("IGG_TEST_DELAY", where)
    for sched in ("1", "0", "2", "3"):
        monkeypatch.setenv("IGG_SCHEDULE", sched)
        say("held back", where, "pack", pack, "schedule", sched)
        with grid(n, zmarch_min=None):
            _calls(T0, Ci, c, nt, split, want, before)


def test_other_arguments_while_replays_are_queued():
    """A call with other arguments puts the kept graph aside while its replays
    may be queued still; 40 graphs in turn, more than are put aside before they
    are destroyed."""
    n, nt = (128, 128, 128), 34
    with grid(n, zmarch_min=None):
        T0, Ci, c = _problem(n)
        want = [_steps(T0, Ci, c, calls * nt)[0] for calls in (3, 6)]
        T, T2 = [T0.clone() for _ in range(2)], [T0.clone() for _ in range(2)]
        for turn in range(40):  # directly, captured, replayed
            say("graph", turn)
            k = turn % 2
            if turn % 4 < 2:
                T[k].copy_(T0)
                T2[k].copy_(T0)
            for _ in range(3):
                igg.diffusion_run(T[k], T2[k], Ci, *c, nt, graph=True)
            if turn % 4 == 3:
                assert all(torch.equal(t, want[1]) for t in T), turn
        torch.cuda.synchronize()
    assert not torch.equal(*want)
