"""lbm_get_stats at the edges of its kernels: rows narrower and wider than a
wavefront, walls (a population that streams into a wall comes back as its
opposite), and particle counts on both sides of the 1 024 from which each
particle has one wavefront instead of a workgroup.  The sums are formed again
on the host in binary64 from the populations, the particles and the exchange
records that the library returns; both sides add up to N terms of size 1 with
rounding 2^-53, so they agree to 1e-12 of the sum of magnitudes."""
import numpy as np
import pytest

from paper_1011_2613_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim, shape, count, storage, wall", [
    (2, (63, 41), 1, "fp64", True), (2, (130, 65), 3, "fp16s", False), (2, (700, 500), 1023, "fp64", True),
    (2, (700, 500), 1024, "fp32s", False), (3, (65, 33, 20), 5, "fp64", True), (3, (20, 64, 31), 0, "fp32s", True)])
def test_stats_equal_the_sums_of_the_state(gpu_lib, dim, shape, count, storage, wall):
    print("stats", dim, shape, count, storage, wall, flush=True)
    w = I.Workload("t", dim, shape, 0.7, wall, 3.0, count, 20.0, 4, 100.0, 0.9, 0, seed=9, v0=5e-3,
                   fluid_force=(1e-5, 2e-6, 0.0))
    sim = gpu_lib.simulation_for(w, storage=storage)
    if not count:
        sim.set_particles()
    sim.step(7)
    st, rho_u = sim.stats(), sim.macro()
    N = float(np.prod(shape))
    rho, u = (a.reshape(-1) if a.ndim == dim else a.reshape(dim, -1) for a in rho_u)
    assert abs(st["mass"] - rho.sum()) <= 1e-12 * N
    for d in range(dim):
        assert abs(st["fluid_momentum"][d] - (rho * u[d]).sum()) <= 1e-12 * N
    x, v, _ = sim.particles()
    F, _ = sim.forces()
    if count:
        m = 20.0 * (np.pi * 9.0 if dim == 2 else 4.0 / 3.0 * np.pi * 27.0)
        assert np.abs(st["particle_momentum"] - m * v.sum(0)).max() <= 1e-12 * m * np.abs(v).sum()
        assert np.abs(st["mean_drag"] - F.mean(0)).max() <= 1e-12 * np.abs(F).sum()
        # every particle's eps shares add up to its sampled volume
        vol = 9.0 * np.pi if dim == 2 else 36.0 * np.pi
        assert abs(st["solid_fraction"] * N - count * vol) <= 0.1 * count * vol
    else:
        assert st["solid_fraction"] == 0.0 and st["np"] == 0
    sim.close()
