"""Particle counts on both sides of the choices that the footprint and the force
kernel make by count, against the FP64 oracle bit for bit: segments per box (4,
2 or 1), threads per particle in the force sums, and workgroups per particle."""
import numpy as np
import pytest

from paper_1011_2613_amd import inputs as I
from tests.parity_util import compare, make_pair

pytestmark = pytest.mark.gpu

CASES = [
    # dim, shape, radius, count; the choice at this count
    (2, (500, 480), 6.3, 1023),       # box of 196 nodes in 4 segments
    (2, (500, 480), 6.3, 1024),       # 2
    (2, (520, 530), 4.7, 2047),       # box of 121 nodes in 2 segments
    (2, (520, 530), 4.7, 2048),       # 1
    (2, (1300, 1280), 9.1, 4095),     # 260 list entries: 256 threads per disc
    (2, (1300, 1280), 9.1, 4096),     # 64
    (3, (76, 78, 74), 5.0, 128),      # 523 list entries: 2 workgroups per sphere
    (3, (76, 78, 74), 5.0, 129),      # 1
    (3, (148, 146, 150), 4.0, 4095),  # 268 list entries: 256 threads per sphere
    (3, (148, 146, 150), 4.0, 4096),  # 64
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_counts_at_the_choices_equal_the_oracle(gpu_lib, case):
    dim, shape, R, n = CASES[case]
    print("particle choices", dim, shape, R, n, flush=True)
    # cells of a lattice of places, each particle off its node by a seeded offset
    per = [int(s // (2 * R + 1.05)) for s in shape[:dim]]
    assert np.prod(per) >= n
    step = [s / c for s, c in zip(shape, per)]
    k = np.arange(n)
    at = [k % per[0], k // per[0] % per[1], k // (per[0] * per[1])][:dim]
    jitter = I.uniform(900 + case, 0, dim * n).reshape(dim, n) * 1.0
    pos = np.zeros((n, 3))
    for d in range(dim):
        pos[:, d] = np.mod(step[d] * at[d] + 0.3 + jitter[d], shape[d])
    vel = I.random_velocities(dim, n, 0.01, 901)
    om = np.zeros((n, 3))
    om[:, 2] = 1e-3
    parts = (pos, vel, om, np.full(n, R), np.full(n, 8.0), np.zeros(n, np.uint8))
    orc, gpu = make_pair(gpu_lib, dim, shape, 0.7, fluid_force=(1e-5, 0, 0), particle_accel=(0, -1e-5, 0), samples=3,
                         kn=50.0, particles=parts, max_radius=R)
    orc.step(2)
    gpu.step(2)
    errs = compare(orc, gpu)
    assert all(e == 0.0 for e in errs.values()), errs
    assert np.array_equal(gpu.q(), orc.q()[:dim])
