"""Calls that return a reduction's value to the host, made by several threads
at once."""
import threading

import pytest

from paper_2211_15716_amd import igg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_common import grid, say  # noqa: E402


def test_threads_do_not_share_partial_results():
    """Four threads, each with a stream and a field of its own, whose maximum
    and sum differ from the others': every call returns its own field's
    value, the same bits each time."""
    n, nthreads, calls = (66, 130, 66), 4, 150
    say("reduce threads", n)
    with grid(n, zmarch_min=None):
        g = torch.Generator(device="cuda")
        g.manual_seed(1)
        A = [torch.rand(n[::-1], device="cuda", dtype=torch.float64, generator=g) + 2.0 * t for t in range(nthreads)]
        want = [(igg.reduce(igg.RED_MAX, a), igg.reduce(igg.RED_SUM, a)) for a in A]
        assert len(set(want)) == nthreads
        streams = [torch.cuda.Stream() for _ in A]
        torch.cuda.synchronize()
        wrong, start = [], threading.Barrier(nthreads)

        def work(t):
            start.wait()
            for _ in range(calls):
                got = tuple(igg.reduce(op, A[t], stream=streams[t]) for op in (igg.RED_MAX, igg.RED_SUM))
                if got != want[t]:
                    wrong.append((t, got))

        ts = [threading.Thread(target=work, args=(t,)) for t in range(nthreads)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not wrong, (len(wrong), wrong[:4])


@pytest.mark.parametrize("own_stream", [False, True])
def test_earlier_work_is_complete_when_a_value_returns(own_stream):
    """Copies to pinned memory put into the stream before igg.reduce or
    igg.diffusion_dt have arrived when the value is returned, without a
    synchronisation, and an event recorded before the call has happened."""
    n = (256, 128, 128)
    say("reduce order", own_stream)
    with grid(n, zmarch_min=None):
        T = torch.empty(n[::-1], device="cuda", dtype=torch.float64)
        T2 = torch.empty_like(T)
        Ci = torch.full_like(T, 0.5)
        pinned = torch.zeros(n[::-1], dtype=torch.float64, pin_memory=True)
        s = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            for q in range(1, 9):
                T.fill_(float(q))
                for _ in range(4):
                    igg.diffusion_step(T2, T, Ci, 1.0, 1e-6, 0.1, 0.1, 0.1)
                pinned.copy_(T2, non_blocking=True)
                e = torch.cuda.Event()
                e.record()
                if q % 2:
                    assert igg.reduce(igg.RED_MAX, T) == q
                else:
                    igg.diffusion_dt(Ci, 1.0, 0.1, 0.1, 0.1)
                assert e.query()
                assert pinned[1:-1, 1:-1, 1:-1].eq(q).all()
