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
