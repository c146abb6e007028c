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


@pytest.mark.parametrize("npix", [96, 512])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_batched_shells_of_every_route_equal_each_run_alone(dtype, npix):
    """Slots whose shells outgrow the bins (walked), fit them, and overflow
    them (every particle on the line of sight), stepped together; 96 and 512
    pixels are the smallest and the largest side of a walk's regions.  float32
    maps are the same bits as each run's alone, float64 sums differ in their
    order (some 10^4 additions a pixel)."""
    from paper_2012_07266_amd.sim import Batch
    # box, field of view, particles
    slots = [(48.0, 8.0, "clustered"), (256.0, 1.0, "clustered"), (32.0, 0.2, "axis"),
             (40.0, 6.0, "clustered")]
    a = np.linspace(0.55, 0.8, 4)
    log(f"batched routes {dtype} {npix}")
    sims, maps, want = [], [], []
    for i, (box, fov, kind) in enumerate(slots):
        wl = W.Workload(f"s{i}", 16, 32, box, 0.1, 1.0, 4, npix, fov, (1.0,))
        x = W.clustered_positions(16, 32, box, seed=61 + i)
        if kind == "axis":
            gen = np.random.Generator(np.random.Philox(key=62))
            x[:2] = 0.5 * box + gen.normal(0.0, 0.02 * box / 16, size=x[:2].shape)
        x = torch.from_numpy(x)
        with new_sim(wl, dtype) as sim:
            sim.set_state(x, torch.zeros_like(x), a[0])
            k = sim.new_maps()
            sim.steps(a, k)
            sim.sync()
            want.append((k.clone(), *(t.clone() for t in sim.get_state())))
        sims.append(new_sim(wl, dtype))
        sims[-1].set_state(x, torch.zeros_like(x), a[0])
        maps.append(sims[-1].new_maps())
    with Batch(sims[0], len(slots)) as b:
        for sim, k in zip(sims[:3], maps):
            b.attach(sim, a, k)
        b.step()
        b.attach(sims[3], a, maps[3])  # walks alone in its last step
        while b.step():
            pass
        for sim in sims:
            b.detach(sim)
    for i, (sim, k, w) in enumerate(zip(sims, maps, want)):
        x, p = sim.get_state()
        sim.sync()
        sim.close()
        e = float((k - w[0]).abs().max() / w[0].abs().max())
        log(f"slot {i}: largest difference over the largest value {e:.1e}")
        assert float(w[0].abs().max()) > 0
        if dtype == torch.float32:
            assert torch.equal(k, w[0]) and torch.equal(x, w[1]) and torch.equal(p, w[2]), i
        else:
            assert e <= 1e-12, i
            assert float((x - w[1]).abs().max()) <= 1e-10 * slots[i][0], i


# np, nm, box, npix, fov, z_src, a0, a1, dtype: shells that outgrow the bins'
# own scratch by so much that no cut into thinner shells fits (float64), or
# that are better walked (float32, pencils of 26 cells)
KEPT = {"no_cut_fits": (16, 32, 48.0, 64, 22.0, (1.0,), 0.52, 0.56, torch.float64),
        "wide_pencils": (64, 128, 42.0, 2048, 6.0, (1.5, 2.0), 0.45, 0.4509, torch.float32)}


@pytest.mark.parametrize("name", list(KEPT))
def test_walked_shell_keeps_the_force_meshes(name):
    """A projection that walks its shell uses no scratch, so a reverse step
    after it finds the step's force meshes and paints no density."""
    np_side, nm, box, npix, fov, zs, a0, a1, dtype = KEPT[name]
    wl = W.Workload(name, np_side, nm, box, 0.1, 1.0, 4, npix, fov, zs)
    x = torch.from_numpy(W.clustered_positions(np_side, nm, box, seed=71))
    log(f"force meshes kept {name}")
    with new_sim(wl, dtype) as sim:
        sim.set_state(x, torch.zeros_like(x), a0)
        sim.step(a0, a1)
        k = sim.new_maps()
        sim.lens(a0, a1, k)
        x_bar = torch.zeros((3, sim.n_particles), dtype=dtype, device=sim.device)
        p_bar = torch.ones_like(x_bar)
        sim.sync()
        sim.profile(True)
        sim.step_vjp(a0, a1, -1.0, x_bar, p_bar, None)
        launches = {n: c for n, (_, c) in sim.profile_read().items()}
        sim.profile(False)
        log(f"launches of the reverse step {launches}")
        assert float(k.abs().max()) > 0 and float(x_bar.abs().max()) > 0
        assert launches.get("vjp_readout") == 1
        assert "paint" not in launches


@pytest.mark.parametrize("shape", [(128, 256), (192, 384)], ids=["128p256m", "192p384m"])
def test_inverse_and_dual_axis1_passes_are_named_as_launched(shape):
    """Up to 256 the two passes are one launch, above they are two, and the
    per-kernel times carry their names."""
    np_side, nm = shape
    wl = W.Workload("passes", np_side, nm, float(np_side), 0.1, 1.0, 4, 64, 2.0, (1.0,))
    a = np.linspace(0.6, 0.7, 3)
    x = torch.rand((3, np_side ** 3), generator=torch.Generator().manual_seed(9)) * wl.box
    log(f"axis-1 passes {shape}")
    with new_sim(wl, torch.float32) as sim:
        sim.set_state(x, torch.zeros_like(x), a[0])
        sim.sync()
        sim.profile(True)
        sim.steps(a, sim.new_maps())
        launches = {n: c for n, (_, c) in sim.profile_read().items()}
        sim.profile(False)
    log(f"launches of two steps {launches}")
    merged = {"fft_c2c_axis1_inv_dual": 2}
    apart = {"fft_c2c_axis1_inv": 2, "fft_c2c_axis1_dual": 2}
    for n, c in {**merged, **apart}.items():
        assert launches.get(n, 0) == (c if n in (merged if nm <= 256 else apart) else 0)
