"""Passes whose route depends on the size: the force operator and its transpose
at every kind of transform length, and checkpoints copied in one launch or, into
a buffer that is not aligned, one by one."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import log, new_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 16), (32, 64), (48, 96), (64, 128), (96, 192), (128, 256),
                                   (192, 384), (256, 512), (384, 768), (512, 1024)],
                         ids=lambda s: f"{s[0]}p{s[1]}m")
def test_force_tangent_and_its_transpose_agree(shape):
    """<v, J u> = <J^T v, u> for the force's derivative J at a clustered state,
    v = J u so that nothing cancels: J u from set_tangent, J^T v as the part of
    x_bar that step_vjp of a last step adds, K2 (df/dx)^T p_bar.  Both sides
    are float32 fields with errors below 5e-6 of their norms."""
    np_side, nm = shape
    box, a0, a1 = float(np_side), 0.5, 0.55
    wl = W.Workload("pair", np_side, nm, box, 0.1, 1.0, 4, 16, 2.0, (1.0,))
    gen = torch.Generator().manual_seed(4)
    if nm < 1024:
        x = torch.from_numpy(W.clustered_positions(np_side, nm, box, seed=3)).float()
    else:  # (minutes of numpy)
        x = torch.rand((3, np_side ** 3), generator=gen) * box
    u = torch.randn(x.shape, generator=gen)
    from paper_2012_07266_amd._lib import PM_MODE_TANGENT
    log(f"force and transpose {shape}")
    with new_sim(wl, torch.float32, modes=PM_MODE_TANGENT) as sim:
        sim.set_state(x, torch.zeros_like(x), a1)
        u = u.to(sim.device)
        sim.set_tangent(u, torch.zeros_like(u), 0.0)
        v = sim.get_tangent()[2]
        x_bar = torch.zeros_like(v)
        p_bar = v.clone()
        sim.step_vjp(a0, a1, -1.0, x_bar, p_bar, None)
        ah = 0.5 * (a0 + a1)
        k2 = (sim.background(a1)[1] - sim.background(ah)[1]) / sim.background(a1)[0]
        sim.sync()
    lhs = float((v.double() ** 2).sum())
    rhs = float((x_bar.double() * u.double()).sum()) / k2
    log(f"<v, Ju> {lhs:.8e}, <J^T v, u> {rhs:.8e}")
    assert lhs > 0 and abs(rhs - lhs) <= 2e-5 * lhs


@pytest.mark.parametrize("force", [False, True], ids=["state", "force"])
@pytest.mark.parametrize("shape", [(16, 16), (16, 32), (48, 96), (512, 1024)],
                         ids=lambda s: f"{s[0]}p{s[1]}m")
def test_checkpoint_into_any_buffer(shape, force):
    """Saved into aligned memory and 4 bytes off it, a checkpoint is the same
    bytes, and restores the same state and force."""
    from paper_2012_07266_amd import Simulation, lib
    np_side, nm = shape
    log(f"checkpoint copies {shape} force={force}")
    x = torch.rand((3, np_side ** 3), generator=torch.Generator().manual_seed(7)) * 32.0
    with Simulation(np_side, nm, 32.0, 32, 2.0, (1.0,), ckpt_force=force) as sim:
        sim.set_state(x, 0.01 * x, 0.5)
        sim.step(0.5, 0.55)
        want = [t.clone() for t in sim.get_state()]
        n = int(lib().pm_checkpoint_bytes(sim._h))
        bufs = [torch.zeros(n + 64, dtype=torch.uint8, device=sim.device) for _ in range(2)]
        for off, b in zip((0, 4), bufs):
            assert lib().pm_checkpoint_save(sim._h, ctypes.c_void_p(b.data_ptr() + off)) == 0
        assert torch.equal(bufs[0][:n], bufs[1][4:4 + n])
        assert not bufs[0][n:].any() and not bufs[1][4 + n:].any()
        for off, b in zip((0, 4), bufs):
            sim.set_state(0.9 * x, x, 0.6)
            assert lib().pm_checkpoint_load(sim._h, ctypes.c_void_p(b.data_ptr() + off),
                                            ctypes.c_double(0.55)) == 0
            assert all(torch.equal(a, b) for a, b in zip(sim.get_state(), want))
            sim.step(0.55, 0.6)
            got = sim.get_state()
            if off == 0:
                first = [t.clone() for t in got]
            assert all(torch.equal(a, b) for a, b in zip(got, first))
        sim.sync()
    assert np.isfinite(first[0].cpu().numpy()).all()
