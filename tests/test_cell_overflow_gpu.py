"""When a DEM cell of more than its 16 places fails a run: at the step whose
contacts (or whose neighbour lists, on a rebuild) are read from it, and no
sooner.  One disc among many small ones sets the cell edge; 16 discs rest in a
cell and a heavy 17th crosses its border at a known step.  Until then every
field equals the oracle, whose contact search has no cells."""
import numpy as np
import pytest

from tests.parity_util import compare, make_pair

pytestmark = pytest.mark.gpu
CELL_OVERFLOW = -8


def crowd(shape, edge, extra=0):
    """Discs of radius 0.4 around the cell (1, 1) of cells of this edge: 16 at
    rest inside, one that is inside from its third step on, `extra` far away;
    and the disc of radius 6 that the edge comes from."""
    width = [shape[d] / (shape[d] // edge) for d in range(2)]
    pos = [[width[0] + 2.2 + 2.5 * (k % 4), width[1] + 2.2 + 2.5 * (k // 4), 0.0] for k in range(16)]
    pos.append([2 * width[0] + 0.25, width[1] + 6.0, 0.0])
    pos.append([2 * width[0] + 12.0, 2 * width[1] + 12.0, 0.0])
    for k in range(extra):
        pos.append([5.0 + 9.0 * (k % 160), 80.0 + 9.0 * (k // 160), 0.0])
    n = len(pos)
    vel = np.zeros((n, 3))
    vel[16, 0] = -0.1
    radius = np.full(n, 0.4)
    radius[17] = 6.0
    fixed = np.ones(n, np.uint8)
    fixed[16] = 0
    rho = np.full(n, 5.0)
    rho[16] = 1e7
    return np.array(pos), vel, np.zeros((n, 3)), radius, rho, fixed


def expect_overflow(gpu_lib, gpu):
    with pytest.raises(gpu_lib.LbmError) as err:
        gpu.step(1)
    assert err.value.code == CELL_OVERFLOW


@pytest.mark.parametrize("timing", [False, True])
def test_overflow_fails_the_step_that_reads_the_cell(gpu_lib, timing):
    print("crowded cell, timing", timing, flush=True)
    parts = crowd((64, 64), 12)
    orc, gpu = make_pair(gpu_lib, 2, (64, 64), 0.8, samples=4, kn=10.0, particles=parts, max_radius=6.0)
    gpu.set_timing(timing)
    for steps in (1, 2):  # the disc is inside at the end of the third step
        orc.step(steps)
        gpu.step(steps)
        errs = compare(orc, gpu)
        assert all(e == 0.0 for e in errs.values()), errs
    assert gpu.particles()[0][16, 0] < 25.6
    expect_overflow(gpu_lib, gpu)


def test_overflow_with_a_thread_per_disc(gpu_lib):
    parts = crowd((1500, 1200), 12, extra=16400)
    gpu = gpu_lib.Simulation(2, (1500, 1200), 0.8, samples=2, kn=10.0, max_particles=len(parts[0]), max_radius=6.0)
    gpu.set_particles(*parts)
    gpu.step(3)
    assert gpu.particles()[0][16, 0] < 24.0
    expect_overflow(gpu_lib, gpu)
    gpu.close()


@pytest.mark.parametrize("timing", [False, True])
def test_lists_fail_only_when_they_are_built(gpu_lib, timing):
    """The lists of the first step last until the disc has moved 0.49 skin, so
    the cells of the third to fifth state are not read."""
    print("crowded cell with lists, timing", timing, flush=True)
    parts = crowd((64, 64), 13)
    orc, gpu = make_pair(gpu_lib, 2, (64, 64), 0.8, samples=4, kn=10.0, particles=parts, max_radius=6.0)
    gpu.set_neighbour_list(100, 1.0)
    gpu.set_timing(timing)
    for steps in (4, 1):
        orc.step(steps)
        gpu.step(steps)
        errs = compare(orc, gpu)
        assert all(e == 0.0 for e in errs.values()), errs
    assert gpu.particles()[0][16, 0] < 32.0 and gpu.neighbour_list[2] == 1
    expect_overflow(gpu_lib, gpu)
