"""Sets on one workgroup at the edges of its waves: one thread keeps each
member, lane groups of the whole workgroup form the pair sums."""
import sys

import numpy as np
import pytest

from paper_1007_3458_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_1007_3458_amd import qsym
    qsym.lib()
    return qsym


def one_set(n):
    """n bodies in one set: light bodies and one on a nearly parabolic orbit,
    whose osculating Hill radius takes them all in."""
    base = inputs.make_disk(f"set{n}", 21, n - 1, 1e-9, 4.5, 6.0, "uniform", "uniform", 0.05, 0.01,
                            planets=False)
    r = np.array([5.0, 0.1, 0.0])
    v = np.array([0.0, 0.99995 * np.sqrt(2.0 / np.linalg.norm(r)), 0.0])
    return inputs.System(f"set{n}", 1.0, 1.0, np.concatenate([base.m, [1e-6]]),
                         np.vstack([base.q, r]), np.vstack([base.v, v]))


def test_member_edges(Q, orc):
    """Sets of 17 members (the smallest on a workgroup) to 256 (the largest),
    on both sides of 32, 64 and 128, in one context; time-step factors that
    take several substeps.  Substeps equal, states to 1e-12 (the step's bound
    against the oracle: rounding of some thousand operations a body)."""
    opts = dict(eta=2e-5, eta_s=2e-3)
    systems = [one_set(n) for n in (17, 32, 33, 64, 65, 128, 129, 256)]
    print("workgroup sets", [s.n for s in systems], flush=True)
    sys.stdout.flush()
    ctx = Q.Context(systems, **opts)
    ctx.step(0.05, 1)
    ctx.sync()
    st = ctx.stats()
    qg, vg = ctx.get_state()
    off = ctx.offsets
    substeps = 0
    for k, s in enumerate(systems):
        qo, vo, res = orc.step(orc.make_params(**opts), 0.05, s.m, s.h, s.q, s.v)
        assert res.rc == 0 and res.stats["max_set"] == s.n and res.stats["substeps"] > 2
        substeps += res.stats["substeps"]
        for g, o in ((qg, qo), (vg, vo)):
            err = np.linalg.norm(g[off[k]:off[k + 1]] - o, axis=1) / np.linalg.norm(o, axis=1)
            assert err.max() < 1e-12
    assert st["status"] == 0 and st["substeps"] == substeps and st["n_sets"] == len(systems)
    ctx.close()


def _mixed(n, far):
    """One set of n bodies, and `far` bodies further out in sets of their own."""
    s = one_set(n)
    o = inputs.make_disk(f"far{far}", 4, far, 3e-7, 400.0, 440.0, "uniform", "uniform", 0.02, 0.01,
                         planets=False)
    return inputs.System(f"mixed{n}", 1.0, 1.0, np.concatenate([s.m, o.m]), np.vstack([s.q, o.q]),
                         np.vstack([s.v, o.v]))


@pytest.mark.parametrize("n", [511, 512, 513, 900])
def test_partition_places(Q, orc, n):
    """Members are placed by counts up to a largest set of 512 and by a sort
    beyond it; with a large set among small ones, ids and members equal the
    oracle's, states to 1e-12."""
    s = _mixed(n, 300)
    print("partition", s.n, flush=True)
    opts = dict(aE=3.0)
    qo, vo, res = orc.step(orc.make_params(**opts), 0.05, s.m, s.h, s.q, s.v)
    size = np.bincount(res.label[res.label >= 0])
    assert res.rc == 0 and size.max() == n and (size > 0).sum() > 3
    ctx = Q.Context(s, **opts)
    ctx.step(0.05, 1)
    ctx.sync()
    st = ctx.stats()
    assert st["status"] == 0 and st["max_set"] == n and st["n_sets"] == (size > 0).sum()
    pairs, sid = ctx.encounters()
    assert len(pairs) == res.stats["n_encounters"]
    # ids by smallest member, as the oracle's labels in ascending order
    want = np.full(s.n, -1)
    roots = np.unique(res.label[res.label >= 0])
    want[res.label >= 0] = np.searchsorted(roots, res.label[res.label >= 0])
    assert np.array_equal(sid, want)
    for g, o in zip(ctx.get_state(), (qo, vo)):
        assert (np.linalg.norm(g - o, axis=1) / np.linalg.norm(o, axis=1)).max() < 1e-12
    ctx.close()
