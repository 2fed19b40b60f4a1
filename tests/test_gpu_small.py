"""Small systems' steps in one launch against the step's kernels launched one
by one (profiling turns the former off): states, energies, encounter pairs,
set ids, r_crit and statistics equal bit for bit, since both run the same
arithmetic in the same order.  Sizes at the edges of the 64-body chunks and
of the kick's tiles, both step kinds, every mode; segments that overflow in
the middle of a call; calls longer than one launch."""
import sys

import numpy as np
import pytest

from paper_1007_3458_amd import inputs

pytestmark = pytest.mark.gpu

STATS = ["steps", "n_candidates", "n_encounters", "n_sets", "max_set", "substeps", "total_encounters",
         "total_substeps", "kepler_iters", "kepler_max", "kepler_hist", "status", "whole_system",
         "fallbacks", "overflows", "global_sets", "kepler_restarts"]


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


def crowd(n, seed, m=1e-6, a=(4.5, 6.0)):
    k = min(n, 4)
    s = inputs.make_disk(f"crowd{n}", seed, max(n, 4) - 4, m, *a, "uniform", "uniform", 0.05, 0.01)
    return s if n >= 4 else inputs.System(s.name, 1.0, 1.0, s.m[:k], s.q[:k], s.v[:k])


def both(Q, systems, calls, swapped=False, skip=(), **kw):
    """The same calls on both paths; everything that a caller can read, compared."""
    got = []
    for one_by_one in (False, True):
        ctx = Q.Context(systems, **kw)
        ctx.profile(one_by_one)
        for tau, k in calls:
            (ctx.step_swapped if swapped else ctx.step)(tau, k)
        q, v = ctx.get_state(check=False)
        st = ctx.stats()
        out = dict(q=q, v=v)
        if st["status"] == 0:
            out.update(E=ctx.energy(), rcrit=ctx.set_rcrit(),
                       cand=np.array(sorted(map(tuple, ctx.candidates(cap=10 ** 6)))) if not st["fallbacks"]
                       else 0)
            out["pairs"], out["sid"] = ctx.encounters()
        got.append((out, {k: st[k] for k in STATS if k not in skip}))
        ctx.close()
    (a, sa), (b, sb) = got
    assert sa == sb
    for k in b:
        assert np.array_equal(a[k], b[k], equal_nan=k != "cand"), k
    return sa


@pytest.mark.parametrize("n", [1, 2, 4, 5, 63, 64, 65, 104, 128, 129, 192, 193, 255, 256])
@pytest.mark.parametrize("precision", [0, 1])
def test_sizes(Q, n, precision):
    """One system up to 192 bodies; larger ones take the one launch from 16
    systems on."""
    say("sizes", n, precision)
    systems = [crowd(n, n)] + ([inputs.enhanced_outer(k) for k in range(15)] if n > 192 else [])
    st = both(Q, systems, [(0.05, 3), (0.05, 1)], precision=precision)
    if n >= 63:
        assert st["n_encounters"] > 0
    both(Q, systems, [(0.05, 3), (0.05, 1)], swapped=True, precision=precision)


@pytest.mark.parametrize("kw", [dict(hill_mode=1), dict(kepler_mode=1), dict(kepler_mode=2),
                                dict(planet_mass=1e-5, aE=4.0), dict(aE=0.0), dict(pair_capacity=3),
                                dict(aE=6.0, aH=4.0)])
def test_modes(Q, kw):
    """Every mode over a context of uneven systems, empty ones among them."""
    systems = [crowd(n, 20 + n) for n in (104, 1, 256, 65, 4)]
    empty = inputs.System("none", 1.0, 1.0, np.zeros(0), np.zeros((0, 3)), np.zeros((0, 3)))
    systems = [systems[0], empty] + systems[1:] + [inputs.two_planet_encounter(40), empty]
    systems += [inputs.enhanced_outer(k) for k in range(12)]
    say("modes", kw)
    st = both(Q, systems, [(0.05, 4), (-0.02 if kw.get("aE") == 0.0 else 0.03, 2)], **kw)
    if "planet_mass" in kw:
        assert st["whole_system"] > 0
    if "pair_capacity" in kw:
        assert st["fallbacks"] > 0


@pytest.mark.parametrize("n", [193, 255, 256])
@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(hill_mode=1, kepler_mode=1),
                                dict(planet_mass=1e-5, aE=4.0)])
def test_many_systems_of_most_bodies(Q, n, kw):
    """Systems of nearly as many bodies as the one launch holds take it where
    there are enough of them; small and empty ones beside them."""
    say("most bodies", n, kw)
    empty = inputs.System("none", 1.0, 1.0, np.zeros(0), np.zeros((0, 3)), np.zeros((0, 3)))
    systems = [crowd(n, 60 + k) for k in range(48)] + [inputs.enhanced_outer(1), empty, crowd(65, 7)]
    st = both(Q, systems, [(0.05, 3), (0.03, 1)], **kw)
    assert st["n_encounters"] > 0
    both(Q, systems, [(0.05, 3)], swapped=True, **kw)


@pytest.mark.parametrize("n,nsys", [(192, 512), (128, 1024), (104, 1)])
def test_autotune_keeps_the_one_launch(Q, n, nsys):
    """Full-matrix shapes only, since symmetric ones would cost the context
    its one-launch steps."""
    base = [inputs.batch_system(k, n) for k in range(32)]
    ctx = Q.Context([base[k % 32] for k in range(nsys)])
    ctx.autotune(0.05)
    say("autotune", n, nsys, ctx.kick_shape(0), ctx.kick_shape(1))
    assert ctx.kick_shape(0)["sym"] == 0 and ctx.kick_shape(1)["sym"] == 0
    ctx.step(0.05, 2)
    ctx.sync()
    ctx.close()


@pytest.mark.parametrize("jchunk", [128, 256, 512])
def test_kick_chunks(Q, jchunk):
    """Full-matrix shapes of other j-chunks: the same partial sums."""
    s = [crowd(250, 9)] + [crowd(130, k) for k in range(15)]
    got = []
    for one_by_one in (False, True):
        ctx = Q.Context(s)
        ctx.set_kick_shape(2, 128, jchunk, 1)
        ctx.profile(one_by_one)
        ctx.step(0.05, 3)
        got.append(ctx.get_state())
        ctx.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


def test_many_systems_and_long_calls(Q):
    """More systems than compute units, and more steps than one launch takes."""
    say("many systems")
    sizes = np.random.default_rng(3).integers(2, 120, 300)
    both(Q, [inputs.batch_system(k, int(n)) for k, n in enumerate(sizes)], [(0.05, 5)])
    say("long call")
    st = both(Q, [inputs.small(4)], [(0.05, 600)])
    assert st["steps"] == 600


@pytest.mark.parametrize("nsys", [1, 3])
def test_segment_overflow(Q, nsys):
    """A crowd that outgrows its encounter segment during the call: every
    system of the context stays at that step's start, later steps do nothing,
    and a new state steps again."""
    rng = np.random.default_rng(5)
    n = 180
    # bodies that fall together: encounters grow until the segment is full
    base = crowd(n, 31, m=1e-9, a=(20.0, 20.4))
    s = base.copy()
    s.q[4:] = base.q[4] + rng.normal(size=(n - 4, 3)) * 0.5
    s.v[4:] = base.v[4] - 0.5 * (s.q[4:] - base.q[4])
    systems = [inputs.small(2), s, inputs.small(3)][:nsys] if nsys > 1 else [s]
    say("segment overflow", nsys)
    st = both(Q, systems, [(0.05, 40), (0.05, 3)],
              skip=("n_sets", "max_set", "substeps", "total_encounters", "total_substeps",
                    "kepler_iters", "kepler_hist", "kepler_max"))
    assert st["status"] & 2 and 0 < st["steps"] < 40
    assert st["overflows"] == 43 - st["steps"]
    ctx = Q.Context(systems)
    ctx.step(0.05, 40)
    with pytest.raises(Q.QsymError):
        ctx.sync()
    m, h = (np.concatenate([getattr(x, k) for x in systems]) for k in "mh")
    q, v = (np.concatenate([getattr(x, k) for x in systems]) for k in "qv")
    ctx.set_state(m, h, q, v)
    ctx.step(0.05, 1)
    ctx.sync()
    ctx.close()
