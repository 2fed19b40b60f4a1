"""The state's way in and out of device memory and the energy: one kernel
each, or copies where the caller's arrays rule the kernel out."""
import ctypes

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


def disk(n, seed=5):
    return inputs.make_disk(f"calls{n}", seed, max(n, 4) - 4, 1e-6, 4.5, 6.0, "uniform", "uniform", 0.05,
                            0.01)


def raw(t, shift):
    """The doubles of t in device memory, `shift` bytes past an aligned address."""
    import torch
    buf = torch.zeros(t.numel() * 8 + 8, dtype=torch.uint8, device="cuda")
    buf[shift:shift + t.numel() * 8] = t.contiguous().view(-1).view(torch.uint8)
    return buf


@pytest.mark.parametrize("n", [4, 63, 64, 255, 256, 257, 1029])
@pytest.mark.parametrize("shift", [0, 4])
def test_device_state_calls(Q, n, shift):
    """set_state and get_state with device arrays, aligned (one kernel) and
    four bytes off (copies), carry the bits of the host calls; so does a step
    after them (its first drift takes the momentum that set_state forms)."""
    import torch
    print("state calls", n, shift, flush=True)
    s = disk(n)
    ref, ctx = Q.Context(s), Q.Context(s)
    other = disk(n, 6)
    h = ref.h
    ref.set_state(other.m, h, other.q, other.v)
    dev = [raw(torch.tensor(np.ascontiguousarray(x), device="cuda"), shift)
           for x in (other.m, h, other.q.T, other.v.T)]
    torch.cuda.synchronize()
    L, DEV = Q.lib(), Q.QSYM_DEVICE
    assert L.qsym_set_state(ctx.ctx, *[ctypes.c_void_p(b.data_ptr() + shift) for b in dev], DEV) == 0
    for steps in (0, 2):
        if steps:
            ref.step(0.02, steps)
            ctx.step(0.02, steps)
        out = [raw(torch.zeros(3 * n, dtype=torch.float64, device="cuda"), shift) for _ in range(2)]
        torch.cuda.synchronize()
        at = [ctypes.c_void_p(b.data_ptr() + shift) for b in out]
        # either array alone, then both
        assert L.qsym_get_state(ctx.ctx, at[0], None, DEV) == 0
        assert L.qsym_get_state(ctx.ctx, None, at[1], DEV) == 0
        one = [b.clone() for b in out]
        assert L.qsym_get_state(ctx.ctx, at[0], at[1], DEV) == 0
        for a, b, want in zip(one, out, ref.get_state()):
            assert torch.equal(a, b)
            got = b[shift:shift + 24 * n].clone().view(torch.float64).view(3, n).T
            assert np.array_equal(got.cpu().numpy(), want)
    # q and v in one array: the copies' order decides, v last
    assert L.qsym_get_state(ctx.ctx, at[0], at[0], DEV) == 0
    got = out[0][shift:shift + 24 * n].clone().view(torch.float64).view(3, n).T
    assert np.array_equal(got.cpu().numpy(), ref.get_state()[1])
    ref.close()
    ctx.close()


def test_nonfinite_status_reaches_every_call(Q):
    """A non-finite state is reported by energy and get_state from the status
    that their kernels carry out, and a new state clears it."""
    import torch
    s = disk(300)
    ctx = Q.Context(s)
    dev = [torch.tensor(np.ascontiguousarray(x), device="cuda") for x in (s.m, ctx.h, s.q.T, s.v.T)]
    bad = dev[3].clone()
    bad[0, 7] = float("nan")
    out = torch.zeros(2, 3, s.n, dtype=torch.float64, device="cuda")
    ctx.set_state_device(dev[0], dev[1], dev[2], bad)
    ctx.step(0.02, 1)
    with pytest.raises(Q.QsymError):
        ctx.energy()
    rc = Q.lib().qsym_get_state(ctx.ctx, out[0].data_ptr(), out[1].data_ptr(), Q.QSYM_DEVICE)
    assert rc != 0
    ctx.set_state_device(*dev)
    ctx.energy()
    assert Q.lib().qsym_get_state(ctx.ctx, out[0].data_ptr(), out[1].data_ptr(), Q.QSYM_DEVICE) == 0
    assert np.array_equal(out[1].cpu().numpy().T, s.v)
    ctx.close()


def test_profiled_device_load_is_the_kernels_time(Q):
    """The momentum phase of a profiled set_state holds its kernel alone, from
    device arrays (one kernel) as by copies (the momentum kernel after them),
    not the wait of the host that follows: both are a launch between two
    events, so the smaller of many agree within half and 2 us."""
    import torch
    s = disk(1029)
    ctx = Q.Context(s)
    ctx.profile(True)
    cols = [torch.tensor(np.ascontiguousarray(x), device="cuda") for x in (s.m, ctx.h, s.q.T, s.v.T)]
    least = []
    for shift in (0, 4):
        dev = [raw(x, shift) for x in cols]
        torch.cuda.synchronize()
        at, us = [ctypes.c_void_p(b.data_ptr() + shift) for b in dev], []
        for _ in range(40):
            before = ctx.stats()["phase_us"][10]
            assert Q.lib().qsym_set_state(ctx.ctx, *at, Q.QSYM_DEVICE) == 0
            us.append(ctx.stats()["phase_us"][10] - before)
        least.append(min(us))
    print("momentum phase us: one kernel, copies", least, flush=True)
    assert 0.0 < least[0] <= 1.5 * least[1] + 2.0
    ctx.close()


def test_energy_short_waves(Q, orc):
    """Energies whose waves hold 16 columns or a few more: systems at the
    edges of the 64- and 128-body blocks, alone and together, to 1e-13 (the
    bound of the energy against the oracle)."""
    systems = [disk(n, n) for n in (4, 5, 63, 64, 65, 127, 128, 129, 193, 320)]
    for group in [systems] + [[s] for s in systems]:
        print("energy", [s.n for s in group], flush=True)
        ctx = Q.Context(group)
        E = ctx.energy()
        ctx.close()
        for s, e in zip(group, E):
            Eo = orc.energy(s.G, s.m0, s.m, s.q, s.v)
            assert abs(e - Eo) <= 1e-13 * abs(Eo)
