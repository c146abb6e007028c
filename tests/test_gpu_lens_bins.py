"""The projection with its images sorted by map region first: shells whose
images fit the sort's scratch, fit only with the meshes, outgrow both, and
overflow it because they crowd into a few regions, each against the oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import cosmo_of, log, new_sim, rel_rms, to_np

pytestmark = pytest.mark.gpu

# np, nm, box, npix, fov, z_src, a_far, a_near, rotation seed, particles
CASES = {
    # a map that no region side divides, two planes, one inside the shell
    "odd_map": (32, 64, 128.0, 203, 3.0, (0.55, 1.0), 0.6, 0.7, None, "clustered"),
    # the same with rotated replicas
    "odd_map_rotated": (32, 64, 128.0, 203, 3.0, (0.55, 1.0), 0.6, 0.7, 77, "clustered"),
    # 1024 regions of 32 x 32 pixels, a shell that ends at the observer.
    # float64 only: within a few Mpc/h of the observer an ulp of a float32
    # position is a sizeable part of a 28" pixel
    "to_observer": (32, 32, 96.0, 1024, 8.0, (0.5,), 0.85, 1.0, None, "clustered"),
    # the smallest map and mesh (one tile, one unit in the box)
    "smallest": (16, 16, 256.0, 16, 1.0, (1.0,), 0.6, 0.7, None, "clustered"),
    # about 4 images per particle: they fit with the meshes only
    "needs_meshes": (16, 32, 48.0, 64, 2.0, (1.0,), 0.55, 0.75, None, "clustered"),
    # over 60 images per particle: by regions, or (float64) as thinner shells
    "too_many": (16, 32, 48.0, 48, 8.0, (1.0,), 0.55, 0.75, None, "clustered"),
    # every particle on the line of sight: each replica's 4096 images fall
    # on the map, 25 times what the mean density gives
    "overflow": (16, 16, 32.0, 32, 0.2, (1.0,), 0.55, 0.8, None, "axis"),
}


def particles(np_side, nm, box, kind):
    x = W.clustered_positions(np_side, nm, box, seed=51)
    if kind == "axis":
        gen = np.random.Generator(np.random.Philox(key=52))
        x[:2] = 0.5 * box + gen.normal(0.0, 0.02 * box / np_side, size=x[:2].shape)
    return x


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_binned_shell_matches_oracle(dtype, name):
    """Tolerances as for the other static shells: float64 round-off; float32
    1e-4 of the maps and 1e-5 of the particle term (about 10^4 additions a
    pixel, each rounded to 6e-8)."""
    from oracle import lens
    if name == "to_observer" and dtype == torch.float32:
        pytest.skip("float32 positions do not resolve the pixels next to the observer")
    np_side, nm, box, npix, fov, zs, a_far, a_near, seed, kind = CASES[name]
    wl = W.Workload(name, np_side, nm, box, 0.1, 1.0, 4, npix, fov, zs)
    c = cosmo_of(wl)
    x = particles(np_side, nm, box, kind)
    if dtype == torch.float32:  # the oracle takes the positions the library is given
        x = x.astype(np.float32).astype(np.float64)
        x[x >= box] = 0.0
    geom = lens.MapGeometry(npix, fov, zs, c, rotation_seed=seed)
    kp = lens.project_shell(x, a_far, a_near, c, box, np_side, geom, include_mean=False)
    ko = lens.project_shell(x, a_far, a_near, c, box, np_side, geom)
    log(f"binned shell {name} {dtype}")
    with new_sim(wl, dtype) as sim:
        if seed is not None:
            sim.set_replica_rotation(seed)
        sim.set_state(torch.from_numpy(x), torch.from_numpy(np.zeros_like(x)), a_near)
        maps = []
        for _ in range(2):  # the second projection finds the first's scratch
            k = sim.new_maps()
            sim.lens(a_far, a_near, k)
            maps.append(to_np(k))
        sim.sync()
    for kg in maps:
        e_part = float(np.sqrt(np.mean((kg - ko) ** 2) / np.mean(kp ** 2)))
        log(f"kappa rel-rms {rel_rms(kg, ko):.2e}, vs particle term {e_part:.2e}")
        assert rel_rms(kg, ko) <= (1e-10 if dtype == torch.float64 else 1e-4)
        assert e_part <= (1e-12 if dtype == torch.float64 else 1e-5)


# a_i, a_f, steps: shells of 64^3 particles on 128^3 meshes whose pencils of
# 64 of 2048 pixels are 22 cells wide, wider than a tile: with images that
# outgrow the sort's scratch (5 a particle) and that fit it (0.8); and such
# shells on both sides of that width (16.2 to 15.7 cells, 1.7 a particle)
FAR = {"many_images": (0.45, 0.4518, 2), "few_images": (0.45, 0.4503, 2),
       "both_widths": (0.555, 0.567, 16)}


@pytest.mark.parametrize("name", list(FAR))
def test_far_shells_beside_the_transform_match_the_steps(name):
    """The images of a far shell are walked by regions in a run and binned in
    a projection by itself.  The images' values and their fixed-point sums are
    the same on both routes, so the float32 maps are equal bit for bit."""
    a_i, a_f, steps = FAR[name]
    wl = W.Workload(name, 64, 128, 42.0, a_i, a_f, steps, 2048, 5.0, (1.5, 2.0))
    x = torch.from_numpy(particles(64, 128, 42.0, "clustered"))
    a = np.linspace(a_i, a_f, steps + 1)
    log(f"far shells {name}")
    with new_sim(wl, torch.float32) as sim:
        k1, k2 = sim.new_maps(), sim.new_maps()
        sim.set_state(x, torch.zeros_like(x), a_i)
        for a0, a1 in zip(a[:-1], a[1:]):
            sim.step(a0, a1)
            sim.lens(a0, a1, k1)
        sim.set_state(x, torch.zeros_like(x), a_i)
        sim.steps(a, k2)
        sim.sync()
        assert float(k1.abs().max()) > 0
        assert torch.equal(k1, k2)
