"""Footprint and force kernels at the edges of their choices, against the FP64
oracle bit for bit: particles from a fraction of a cell to the largest allowed,
boxes cut into 1 .. 256 segments, 16, 64, 256 and 1 024 threads per particle in
the force sums, particles at walls and across periodic edges, lattices so
narrow that several rows share an owner-count word, and particle counts on both
sides of the choices (2 048 units, 16 384 discs)."""
import numpy as np
import pytest

from paper_1011_2613_amd import inputs as I
from tests.parity_util import compare, make_pair

pytestmark = pytest.mark.gpu


def particles(dim, shape, radii, seed, wall):
    """Particles with the given radii, placed as spheres of the largest."""
    R = max(radii)
    n = len(radii)
    pos = I.place_particles(dim, shape, R, n, seed, wall_y=wall)
    vel = I.random_velocities(dim, n, 0.01, seed + 1)
    om = np.zeros((n, 3))
    om[:, 2] = 1e-3
    if dim == 3:
        om[:, 0] = -5e-4
    return pos, vel, om, np.array(radii), np.full(n, 8.0), np.zeros(n, np.uint8)


CASES = [
    # dim, shape, radii, samples, wall, steps
    (3, (96, 90, 94), [30.0], 4, False, 2),            # one large sphere: 256 segments, 1 024 threads
    (3, (70, 66, 64), [16.0], 3, True, 3),
    (2, (140, 150), [62.0], 2, False, 2),              # the largest disc
    (2, (60, 200), [20.3, 11.0, 5.0], 8, True, 4),
    (3, (40, 44, 36), [0.1, 0.4, 1.0, 2.5, 4.9, 6.0], 4, False, 4),
    (2, (7, 40), [2.4, 1.1, 0.2], 5, False, 4),        # rows narrower than an owner-count word
    (3, (6, 9, 30), [1.9, 0.7], 8, True, 4),
    (3, (33, 31, 29), [3.0] * 20, 1, False, 6),
    (2, (640, 650), [3.2] * 2047, 4, False, 2),        # last count with segments
    (2, (640, 650), [3.2] * 2048, 4, True, 2),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_forces_and_fields_equal_the_oracle(gpu_lib, case):
    dim, shape, radii, S, wall, steps = CASES[case]
    print("footprints", CASES[case][:2], len(radii), "particles, largest", max(radii), flush=True)
    parts = particles(dim, shape, radii, 300 + case, wall)
    orc, gpu = make_pair(gpu_lib, dim, shape, 0.7, wall_y=wall, fluid_force=(1e-5, 0, 0),
                         particle_accel=(0, -1e-5, 0), samples=S, kn=50.0, restitution=0.9, particles=parts,
                         max_radius=max(radii))
    for _ in range(steps):
        orc.step(1)
        gpu.step(1)
    errs = compare(orc, gpu)
    assert all(e == 0.0 for e in errs.values()), errs
    # the exchange records behind the lists, node by node
    assert np.array_equal(gpu.q(), orc.q()[:dim])
    # two steps replayed as a graph after the single ones
    orc.step(4)
    gpu.step(4)
    errs = compare(orc, gpu)
    assert all(e == 0.0 for e in errs.values()), errs


def test_particle_count_does_not_change_a_particle(gpu_lib):
    """16 383 and 16 384 equal discs (64 and 16 lanes per disc): the discs that
    both runs share give the same forces bit for bit."""
    shape, R = (1500, 1400), 4.0
    s = 10.0  # a square grid of discs, each off its node by a seeded offset
    gx, gy = int(shape[0] // s), int(shape[1] // s)
    k = np.arange(16384)
    off = I.uniform(77, 0, 2 * len(k)).reshape(-1, 2)
    pos = np.stack([s * (k % gx) + 4.2 + 1.5 * off[:, 0], s * (k // gx) + 4.2 + 1.5 * off[:, 1], 0.0 * k], 1)
    assert k[-1] // gx < gy
    out = []
    for n in (16383, 16384):
        sim = gpu_lib.Simulation(2, shape, 0.7, samples=8, kn=10.0, max_particles=n, max_radius=R,
                                 fluid_force=(1e-5, 0, 0))
        sim.set_particles(pos[:n], vel=I.random_velocities(2, n, 0.005, 78), radius=np.full(n, R), rho_s=np.full(n, 5.0))
        sim.step(1)
        out.append([a[:16383 - 200] for a in sim.forces()])
        sim.close()
    # the last disc changes its own surroundings only; the others' first step is local
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("dim", [2, 3])
def test_cell_list_carried_between_steps(gpu_lib, dim):
    """The plain step files each particle in the next step's cell list; steps
    with every phase timed, with neighbour lists or with the slab pipeline
    build their own.  Contacts across all switches, and after the particle set
    and a saved state are replaced, equal the oracle bit for bit."""
    shape = (60, 80) if dim == 2 else (30, 44, 28)
    R = 3.0
    n = 40 if dim == 2 else 60
    radii = [R] * n
    parts = particles(dim, shape, radii, 500 + dim, True)
    parts[1][:] *= 20.0  # fast enough to change cells and touch within some steps
    orc, gpu = make_pair(gpu_lib, dim, shape, 0.7, wall_y=True, particle_accel=(0, -1e-4, 0), samples=4, kn=40.0,
                         restitution=0.9, particles=parts, max_radius=R)
    touched = 0
    switches = [lambda: None, lambda: gpu.set_timing(True), lambda: gpu.set_timing(False),
                lambda: gpu.set_neighbour_list(5, 1.0), lambda: gpu.set_neighbour_list(0),
                lambda: gpu.set_pipeline(2), lambda: gpu.set_pipeline(1), lambda: gpu.set_timing(True, lattice_only=True)]
    for k, switch in enumerate(switches):
        print("cell list, %dD, switch %d" % (dim, k), flush=True)
        switch()
        for chunk in (1, 4, 3):
            orc.step(chunk)
            gpu.step(chunk)
            errs = compare(orc, gpu)
            assert all(e == 0.0 for e in errs.values()), (k, errs)
            touched += int(np.count_nonzero(np.abs(orc.contact_forces()).sum(axis=1)))
    assert touched > 0
    import os
    import tempfile
    path = os.path.join(tempfile.mkdtemp(), "state")
    gpu.save(path)
    gpu.step(6)
    orc.step(3)
    gpu.load_state(path)
    gpu.step(3)
    errs = compare(orc, gpu)
    assert all(e == 0.0 for e in errs.values()), errs
