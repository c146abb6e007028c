"""Routes of the shell projection that depend on how many images a shell has,
by itself, in a run and in a batch."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import log, new_sim

pytestmark = pytest.mark.gpu


def a_of_chi(sim, chi):
    """The scale factor at distance chi (bisection on the library's own chi)."""
    lo, hi = 0.05, 1.0
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if sim.background(mid)[2] > chi else (lo, mid)
    return 0.5 * (lo + hi)


def test_shell_with_more_images_than_32_bits_count():
    """Every particle in one plane across the line of sight, inside a shell
    0.03 cells deep: 128^2 replicas of 64^3 images, 4.6e9 bin entries, where
    the mean density gives 5 a particle.  The map is linear in the particles,
    so it is that of one half of them plus that of the other, less the empty
    shell's; each of those has fewer than 2^32 entries.  The images' sums are
    exact, so each map is rounded once: 2^-24 of its value, three maps and two
    additions, 1e-6 in all."""
    n, box, cell = 64 ** 3, 6.0, 6.0 / 128
    wl = W.Workload("plane", 64, 128, box, 0.1, 1.0, 4, 4096, 22.0, (1.5,))
    gen = torch.Generator().manual_seed(21)
    x = torch.rand((3, n), generator=gen, dtype=torch.float64) * box
    x[2] = 47.36 * cell
    log("shell with more images than 32 bits count")
    with new_sim(wl, torch.float32) as sim:
        plane = 333 * box + 47.36 * cell
        a_near, a_far = (a_of_chi(sim, plane + d * cell) for d in (-0.015, 0.015))
        half = torch.arange(n) % 2 == 0
        maps = []
        for gone in (None, half, ~half, half | ~half):
            y = x.clone()
            if gone is not None:
                y[2, gone] = 100.36 * cell
            sim.set_state(y, torch.zeros_like(y), a_near)
            k = sim.new_maps()
            sim.lens(a_far, a_near, k)
            sim.sync()
            maps.append(k.double())
            log(f"mean of the map {float(maps[-1].mean()):.4e}")
    full, a, b, empty = maps
    inner = full[:, 8:-8, 8:-8]
    assert float(inner.min()) > 0.25 * float(inner.mean()) > 0
    want = a + b - empty
    worst = float(((full - want).abs() / want.abs()).max())
    log(f"largest relative difference {worst:.2e}")
    assert worst <= 1e-6
