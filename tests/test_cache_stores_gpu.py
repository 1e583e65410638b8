"""Populations stored through the caches (state arrays of 48 to 280 MB together)
or with the non-temporal hint (below and above): the same bits.  A periodic box
repeated along an axis holds copies of the single box, and the two lie on
different sides of a line."""
import numpy as np
import pytest

from paper_1011_2613_amd import ensemble

pytestmark = pytest.mark.gpu

CASES = [  # shape (x, y[, z]) and storage; the repeat doubles the last axis
    ((44, 44, 41), "fp64"), ((52, 50, 66), "fp32s"), ((70, 66, 76), "fp16s"), ((360, 500), "fp64"),
    ((80, 80, 142), "fp64"), ((112, 112, 146), "fp32s"), ((1300, 1490), "fp64"),
]


@pytest.mark.parametrize("shape,storage", CASES)
def test_repeated_box_holds_copies(gpu_lib, shape, storage):
    print("stores", shape, storage, flush=True)
    dim = len(shape)
    Q, size = (9 if dim == 2 else 19), {"fp64": 8, "fp32s": 4, "fp16s": 2}[storage]
    nbytes = 2 * Q * size * int(np.prod(shape))
    inside = [48e6 <= b <= 280e6 for b in (nbytes, 2 * nbytes)]
    assert inside[0] != inside[1]
    rng = np.random.default_rng(5)
    out = []
    f0 = None
    for rep in (1, 2):
        full = shape[:-1] + (shape[-1] * rep,)
        sim = gpu_lib.Simulation(dim, full, 0.7, storage=storage, fluid_force=(1e-5, 2e-5, 0))
        sim.set_particles()
        if f0 is None:
            f0 = sim.get_f() * (1.0 + 0.05 * rng.random((Q,) + sim.field_shape))
        sim.set_f(np.concatenate([f0] * rep, axis=1))
        sim.step(5)  # two steps as a graph twice, and one alone
        out.append(sim.get_f())
        sim.close()
    n = out[0].shape[1]
    assert np.array_equal(out[1][:, :n], out[0]) and np.array_equal(out[1][:, n:], out[0])


def test_batched_box_among_others(gpu_lib):
    box = next(b for b in ensemble.sample_boxes(64, 4) if b["edge"] == 32)
    drag = []
    for copies in (1, 12, 60):  # 5, 60 and 299 MB
        batch = gpu_lib.Batch([box] * copies, samples=4)
        batch.run(6)
        F, X = batch.get_drag()
        m = len(box["pos"])
        for k in (0, copies - 1):
            drag.append((F[k * m:(k + 1) * m], X[k * m:(k + 1) * m]))
    for F, X in drag[1:]:
        assert np.array_equal(F, drag[0][0]) and np.array_equal(X, drag[0][1])
