"""Rows whose last workgroup would hold idle wavefronts take tiles of one
wavefront, dealt to the workgroups in turn: the same bits as a chosen workgroup
width, at row lengths on both sides of the choice, with rows of tiles that cross
workgroups, and in the slabs of the pipeline."""
import numpy as np
import pytest

from paper_1011_2613_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(257, 9, 5), (300, 11, 7), (320, 8, 9), (385, 9, 6), (449, 7, 5), (512, 7, 6), (700, 9, 6),
          (1300, 23), (321, 64), (300, 7)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", ["fp64", "fp32s", "fp16s"])
def test_same_bits_as_a_chosen_width(gpu_lib, shape, storage):
    print("row tiles", shape, storage, flush=True)
    dim = len(shape)
    R = 1.4
    pos = I.place_particles(dim, shape, R, 6, 3, wall_y=True)
    vel = I.random_velocities(dim, 6, 0.01, 4)
    out = []
    for width in (0, 64):
        sim = gpu_lib.Simulation(dim, shape, 0.8, storage=storage, wall_y=True, fluid_force=(1e-5, 0, 0),
                                 max_particles=6, max_radius=R)
        sim.set_particles(pos, vel, np.zeros((6, 3)), np.full(6, R), np.full(6, 3.0))
        sim.set_lattice_block(width)
        sim.step(5)
        out.append((sim.get_f(), sim.q()) + sim.forces() + sim.particles())
        sim.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))


def test_slabs_of_the_pipeline(gpu_lib):
    shape, R = (300, 96, 12), 2.0
    pos = I.place_particles(3, shape, R, 40, 3, wall_y=True)
    vel = I.random_velocities(3, 40, 0.01, 4)
    out = []
    for slabs in (1, 4):
        sim = gpu_lib.Simulation(3, shape, 0.8, wall_y=True, max_particles=40, max_radius=R)
        sim.set_particles(pos, vel, np.zeros((40, 3)), np.full(40, R), np.full(40, 3.0))
        sim.set_pipeline(slabs)
        sim.step(6)
        out.append((sim.get_f(),) + sim.forces() + sim.particles())
        sim.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
