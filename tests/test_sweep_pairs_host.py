"""The checkpointing executor with two steps per launch, on CPU tensors."""
import numpy as np
import pytest

from paper_2211_15716_amd import checkpoint as ck
from paper_2211_15716_amd import diffusion, igg

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sched", [("store_all",), ("periodic", 1), ("periodic", 4), ("periodic", 5), ("sqrt",),
                                   ("binomial", 1), ("binomial", 4)])
@pytest.mark.parametrize("nt", [0, 1, 2, 3, 7, 20, 33])
def test_sweep_with_pairs_sees_every_state(sched, nt, monkeypatch):
    """Forward result, the state each adjoint step sees, step count and
    buffers as with single steps; no pair from T0, no buffer read and written
    by one launch."""
    rng = np.random.default_rng(nt)
    T0 = torch.from_numpy(rng.uniform(0.0, 1.0, (5, 6, 7)))
    Ci = torch.from_numpy(rng.uniform(0.0, 1.0, (5, 6, 7)))
    copy, seen, made, pairs = T0.clone(), [], [], []

    def f(T):
        return 0.5 * T + Ci

    def step(T2, T, C, *a, **k):
        assert T2 is not T and T2 is not T0
        T2.copy_(f(T))

    def step_pair(T2, mid, T, C, *a, **k):
        assert T2 is not T and T2 is not T0 and T is not T0 and mid is not T and mid is not T2
        pairs.append(mid is not None)
        if mid is not None:
            assert mid is not T0
            mid.copy_(f(T))
        T2.copy_(f(f(T)))

    def counting(g):
        def h(x):
            made.append(g(x))
            return made[-1]
        return h

    monkeypatch.setattr(igg, "steps_per_launch", lambda T: 2)
    monkeypatch.setattr(igg, "diffusion_step", step)
    monkeypatch.setattr(igg, "diffusion_step_pair", step_pair)
    monkeypatch.setattr(igg, "diffusion_step_adjoint", lambda ln, lp, Tn, *a, **k: seen.append(Tn.clone()))
    clone = diffusion._clone
    monkeypatch.setattr(diffusion, "_clone", counting(clone))
    monkeypatch.setattr(diffusion, "_fresh_like", counting(clone))
    monkeypatch.setattr(diffusion, "_zeros_like", lambda x: torch.zeros_like(x))
    states = [T0.clone()]
    for _ in range(nt):
        states.append(f(states[-1]))
    ops = ck.make(sched[0], nt, sched[1] if len(sched) > 1 else None)
    sw = diffusion.Sweep(diffusion.Problem(1.0, 0.1, 1.0, 1.0, 1.0), Ci, T0, ops)
    assert torch.equal(sw.forward(nt), states[nt])
    sw.reverse(torch.zeros_like(T0))
    assert torch.equal(T0, copy) and len(seen) == nt
    for q, s in enumerate(seen):
        assert torch.equal(s, states[nt - 1 - q]), q
    assert sw.advances == sum(op[2] - op[1] for op in ops if op[0] == "advance") + (nt > 0)
    assert len(made) <= 3 + sw.peak - 1
    assert bool(pairs) == (nt >= 7 and sched != ("periodic", 1)), pairs


def test_only_problems_own_step_is_paired(monkeypatch):
    """A subclass or instance with a step of its own keeps it."""
    monkeypatch.setattr(igg, "steps_per_launch", lambda T: 2)
    T = torch.zeros(4, 4, 4)

    class Sourced(diffusion.Problem):
        def step(self, out, T, Ci, stream=None):
            pass

    args = (1.0, 0.1, 1.0, 1.0, 1.0)
    assert diffusion._pairs(diffusion.Problem(*args), T)
    assert not diffusion._pairs(Sourced(*args), T)
    assert not diffusion._pairs(diffusion.RankProblem(*args), [T])
    assert not diffusion._pairs(diffusion.FluxProblem(*args), T)
    own = diffusion.Problem(*args)
    own.step = lambda out, T, Ci, stream=None: None
    assert not diffusion._pairs(own, T)


@pytest.mark.parametrize("sched", [("store_all",), ("periodic", 1), ("periodic", 5), ("sqrt",), ("binomial", 1),
                                   ("binomial", 4)])
@pytest.mark.parametrize("nt", [1, 2, 3, 8, 21])
def test_sweep_with_adjoint_pairs_sees_every_state(sched, nt, monkeypatch):
    """The states the adjoint steps see, one or two a launch, as with single
    steps; no launch writes the adjoint state it reads."""
    T0, Ci, seen = torch.full((3, 3, 3), 0.5, dtype=torch.float64), torch.rand(3, 3, 3, dtype=torch.float64), []

    def f(T):
        return 0.5 * T + Ci

    def adjoint(ln, lp, Tn, *a, **k):
        assert ln is not lp
        seen.append(Tn.clone())

    def adjoint_pair(ln, lp, T, *a, **k):
        assert ln is not lp and T is not T0
        seen.extend((f(T), T.clone()))

    monkeypatch.setattr(igg, "steps_per_launch", lambda T: 1)
    monkeypatch.setattr(igg, "adjoints_per_launch", lambda T: 2)
    monkeypatch.setattr(igg, "diffusion_step", lambda T2, T, *a, **k: T2.copy_(f(T)))
    monkeypatch.setattr(igg, "diffusion_step_adjoint", adjoint)
    monkeypatch.setattr(igg, "diffusion_step_adjoint_pair", adjoint_pair)
    for name in ("_clone", "_fresh_like"):
        monkeypatch.setattr(diffusion, name, lambda x: x.clone())
    monkeypatch.setattr(diffusion, "_zeros_like", lambda x: torch.zeros_like(x))
    states = [T0.clone()]
    for _ in range(nt):
        states.append(f(states[-1]))
    ops = ck.make(sched[0], nt, sched[1] if len(sched) > 1 else None)
    sw = diffusion.Sweep(diffusion.Problem(1.0, 0.1, 1.0, 1.0, 1.0), Ci, T0, ops)
    assert torch.equal(sw.forward(nt), states[nt])
    sw.reverse(torch.zeros_like(T0))
    assert sw.adjoints == nt and len(seen) == nt
    assert sw.advances <= sum(op[2] - op[1] for op in ops if op[0] == "advance") + 1
    assert set(sw.store) <= {0}
    assert all(torch.equal(s, states[nt - 1 - q]) for q, s in enumerate(seen))
    assert any(op[0] == "adjoint2" for op in sw.rev) or nt < 8 or sched[0] == "binomial"
