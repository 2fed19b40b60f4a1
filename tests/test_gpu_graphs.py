"""Steps that replay graphs, and steps that a caller captures.  A context
outside the one-launch path and below 8192 bodies captures eight steps once 64
of one tau were taken, and replays them in later calls of nine steps or more;
with profiling on every step is launched by itself.  The same calls on both
give the same bits, through a remainder after the last replay, another tau and
another kick shape; and a caller's own graph of a call, before and after the
context has one, gives those of the call."""
import sys

import numpy as np
import pytest

from paper_1007_3458_amd import inputs

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def Q():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_1007_3458_amd import qsym
    qsym.lib()
    return qsym


def crowd(n, seed):
    return inputs.make_disk(f"crowd{n}", seed, n - 4, 1e-6, 4.5, 6.0, "uniform", "uniform", 0.05, 0.01)


def equal(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a.get_state(), b.get_state()))


@pytest.mark.parametrize("kind", ["hybrid", "swapped", "sweep"])
@pytest.mark.parametrize("nsys", [1, 2])
def test_graphs_equal_single_launches(Q, kind, nsys):
    systems = [crowd(300 + 7 * k, 6 + k) for k in range(nsys)]
    kw = dict(sweep=1) if kind == "sweep" else {}
    a, b = Q.Context(systems, **kw), Q.Context(systems, **kw)
    b.profile(True)

    def both(tau, n):
        say("graphs", kind, nsys, tau, n)
        for c in (a, b):
            (c.step_swapped if kind == "swapped" else c.step)(tau, n)
        assert equal(a, b)
        assert np.array_equal(a.energy(), b.energy())   # the context's own work between replays
        sa, sb = a.stats(), b.stats()
        for k in ("steps", "n_candidates", "n_encounters", "n_sets", "substeps", "total_encounters",
                  "total_substeps", "kepler_iters", "status"):
            assert sa[k] == sb[k], k

    for n in (64, 21, 9, 8, 1, 17):           # captured in the second; two replays and four steps
        both(0.01, n)
    for n in (60, 20, 20):                    # another tau: captured again in the third
        both(0.02, n)
    for c in (a, b):                          # another shape: the graph is made anew
        c.set_kick_shape(2, 128, 512, 0)
    both(0.02, 30)
    both(0.01, 12)
    both(0.02, 70)
    both(0.02, 25)
    a.close()
    b.close()


@pytest.mark.parametrize("n", [104, 300])
@pytest.mark.parametrize("before", [(1,), (40, 40), (64, 21)])
@pytest.mark.parametrize("kind", ["hybrid", "swapped"])
def test_step_in_a_callers_capture(Q, n, before, kind):
    """Replayed three times, with the context's own calls between."""
    import torch
    say("capture", n, before, kind)
    s = crowd(n, 9)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a, b = Q.Context(s), Q.Context(s)
        step = [c.step_swapped if kind == "swapped" else c.step for c in (a, b)]
        for k in before:
            for f in step:
                f(0.01, k)
        a.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            step[0](0.01, 20)
        assert equal(a, b)                    # recorded, not run
        for k in (0, 3, 21):
            g.replay()
            step[1](0.01, 20)
            if k:
                for f in step:
                    f(0.01, k)
            torch.cuda.synchronize()
            assert equal(a, b)
            assert np.array_equal(a.energy(), b.energy())
        assert a.stats()["steps"] == b.stats()["steps"]
        a.close()
        b.close()
