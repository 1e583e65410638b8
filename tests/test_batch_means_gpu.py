"""Mean and shell velocities of ensemble boxes whose node count is below, not a
multiple of and far above the 128 x 256 threads that share a box, against the
same sums over the box's populations on the host.  Both sides round in binary64
(2^-53) over at most N L terms of size 1e-2, so they agree to 1e-13."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


def test_mean_and_shell_velocity(gpu_lib):
    boxes = [{"edge": 4}, {"edge": 5}, {"edge": 33, "pos": [[3.2, 30.7, 16.4], [20.1, 5.5, 2.2]], "radius": 4.3},
             {"edge": 21, "pos": [[20.9, 0.1, 10.6]], "radius": 9.5}]
    for k, b in enumerate(boxes):
        b.update(tau=0.7 + 0.1 * k, fluid_force=(1e-5, -2e-6, 3e-6), init_velocity=(0.01, 0.004 * k, -0.003))
    batch = gpu_lib.Batch(boxes, samples=4)
    batch.run(25)
    U, Us = batch.mean_velocity(), batch.shell_velocity()
    c, _ = O.velocities(3)
    c = np.asarray(c, dtype=np.float64).reshape(-1, np.asarray(c).shape[-1])
    c = c if c.shape[0] == 19 else c.T
    s0 = 0
    for k, b in enumerate(boxes):
        L = b["edge"]
        f = batch.get_f(k)
        j = np.tensordot(c.T[:3], f, axes=(1, 0))  # [3][z][y][x]
        print("box of edge %d: %s" % (L, U[k]), flush=True)
        assert np.abs(U[k] - j.reshape(3, -1).mean(1)).max() <= 1e-13
        u = j / f.sum(0)
        g = np.arange(L, dtype=np.float64)
        for p, x in enumerate(b.get("pos", [])):
            d = [g - x[a] for a in range(3)]
            d = [np.where(v > 0.5 * L, v - L, np.where(v <= -0.5 * L, v + L, v)) for v in d]
            r2 = d[2][:, None, None] ** 2 + d[1][None, :, None] ** 2 + d[0][None, None, :] ** 2
            R = b["radius"]
            m = (r2 >= (R + 1.0) ** 2) & (r2 <= 4.0 * R * R)
            for q in b["pos"]:  # no sub-cell sample of any sphere: the cell lies outside
                e = [np.abs(np.mod(g - q[a] + 0.5 * L, L) - 0.5 * L) for a in range(3)]
                off = (np.arange(4) + 0.5) / 4 - 0.5
                near = [np.min(np.abs(np.abs(v)[:, None] + off[None]) ** 2, axis=1) for v in e]
                m &= near[2][:, None, None] + near[1][None, :, None] + near[0][None, None, :] > R * R
            assert m.sum() > 0
            assert np.abs(Us[s0 + p] - u[:, m].mean(1)).max() <= 1e-13
        s0 += len(b.get("pos", []))
