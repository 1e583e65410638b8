"""Solid velocity of half-precision storage, whose kernel branches on what its
wavefronts need: nodes with several owners, the minimum image, and the division
(zeros and numbers near underflow divide, the rest multiply by a reciprocal and
correct).  The first step starts from populations that are exactly zero, so q is
a linear image of the solid velocity; it is compared node by node with the FP64
oracle.

Tolerance: V goes through at most 12 binary32 roundings of terms no larger than
vmax = |v| + |omega| (R + 1), the sums of Omega_i c_i through at most 40 more,
none amplified (beta <= 1, the weights times 3 sum to 1 per component):
64 * 2^-24 vmax covers both."""
import numpy as np
import pytest

from tests.parity_util import make_pair

pytestmark = pytest.mark.gpu

KINDS = {  # factors of v and omega, and one of both
    "moving": (1.0, 1.0, 1.0),
    "one_axis": ((1.0, 0.0, 0.0), 0.0, 1.0),  # zero components: the division
    "tiny": (1.0, 1.0, 1e-33),                # below the range of the correction
    "at_rest": (0.0, 0.0, 1.0),
}


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("dim,shape,samples", [(2, (67, 45), 8), (3, (35, 33, 34), 4), (3, (24, 40, 26), 1)])
def test_first_exchange_follows_the_oracle(gpu_lib, dim, shape, samples, kind):
    print("solid velocity", dim, shape, samples, kind, flush=True)
    fv, fw, scale = KINDS[kind]
    R = 4.3
    half = 0.5 * np.array(shape[:dim] + (0,) * (3 - dim), dtype=float)
    # a touching pair (shared nodes) inside, one particle across the periodic
    # edges, and three about one point
    off = np.array([R + 0.05, 0.3, 0.2 if dim == 3 else 0.0])
    up = np.array([0.0, 2 * R + 2, 0.0])
    pos = np.array([half - off, half + off, [0.4, 0.3, 0.2], half + up,
                    half + up + [1.96 * R, 0, 0], half + up + [0.98 * R, 1.7 * R, 0]])
    pos[:, dim:] = 0.0
    pos = np.mod(pos, np.array(shape[:dim] + (1,) * (3 - dim), dtype=float))
    rng = np.random.default_rng(7)
    vel, om = 0.02 * rng.standard_normal((6, 3)) * fv, 2e-3 * rng.standard_normal((6, 3)) * fw
    if dim == 2:
        vel[:, 2] = 0.0
        om[:, :2] = 0.0
    rest = (np.full(6, R), np.full(6, 5.0), np.zeros(6, np.uint8))
    orc, gpu = make_pair(gpu_lib, dim, shape, 0.8, wall_y=False, fluid_force=(0, 0, 0),
                         particle_accel=(0, 0, 0), samples=samples, kn=1.0, restitution=0.9,
                         particles=(pos, vel, om) + rest, max_radius=R, storage="fp16s")
    gpu.set_particles(pos, vel * scale, om * scale, *rest)
    orc.step(1)
    gpu.step(1)
    # from rest sum_i Omega_i c_i is linear in V (the even terms cancel), so the
    # oracle, whose populations w_i + g_i hold no 1e-33, runs unscaled
    ref, got = orc.q()[:dim] * scale, gpu.q()
    vel, om = vel * scale, om * scale
    vmax = float(np.max(np.linalg.norm(vel, axis=1) + np.linalg.norm(om, axis=1) * (R + 1)))
    assert np.max(np.abs(got - ref)) <= 64 * 2.0**-24 * vmax
    assert kind == "at_rest" or np.max(np.abs(ref)) > 0.05 * vmax
