"""Reads of forces and particles through the pinned memory of a context: as many
particles at a time as it holds (1 MiB), host and device destinations, and
several threads on one context."""
import ctypes as C
import threading

import numpy as np
import pytest

from paper_1011_2613_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 2, 170, 14563, 14564, 29200])  # 1 MiB holds 14 563 particles of 72 bytes
def test_reads_return_what_was_set(gpu_lib, count):
    print("reads", count, flush=True)
    import torch
    side = 8 * int(np.ceil(np.sqrt(count))) + 8
    k = np.arange(count)
    pos = np.stack([4.0 + 8.0 * (k % (side // 8)), 4.0 + 8.0 * (k // (side // 8)), 0.0 * k], 1)
    rng = np.random.default_rng(count)
    vel = np.concatenate([rng.standard_normal((count, 2)), np.zeros((count, 1))], 1)
    om = np.concatenate([np.zeros((count, 2)), rng.standard_normal((count, 1))], 1)
    sim = gpu_lib.Simulation(2, (side, side), 0.8, max_particles=count, max_radius=2.0)
    sim.set_particles(pos, vel, om, np.full(count, 2.0), np.full(count, 2.0))
    for got, want in zip(sim.particles(), (pos, vel, om)):
        assert np.array_equal(got, want)
    # the same on the device
    out = [torch.full((count, 3), 7.0, dtype=torch.float64, device=sim.device) for _ in range(3)]
    torch.cuda.synchronize()
    rc = gpu_lib.load().lbm_get_particles(sim._ctx, *[C.c_void_p(t.data_ptr()) for t in out], gpu_lib.LBM_DEVICE)
    assert rc == 0
    for got, want in zip(out, (pos, vel, om)):
        assert np.array_equal(got.cpu().numpy(), want)
    assert gpu_lib.load().lbm_get_particles(sim._ctx, *[C.c_void_p(t.data_ptr()) for t in out], 9) != 0
    sim.close()


def test_reads_from_threads_and_streams(gpu_lib):
    import torch
    w = I.workload("C1")
    sim = gpu_lib.simulation_for(w)
    sim.step(3)
    want = sim.particles() + sim.forces()
    rho, u = (t.cpu().numpy() for t in sim.macro_device())
    bad = []

    def reader():
        for _ in range(50):
            if not all(np.array_equal(a, b) for a, b in zip(sim.particles() + sim.forces(), want)):
                bad.append("particles")
            with torch.cuda.stream(torch.cuda.Stream()):
                r, v = (t.cpu().numpy() for t in sim.macro_device())
            if not (np.array_equal(r, rho) and np.array_equal(v, u)):
                bad.append("macro")

    threads = [threading.Thread(target=reader) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    sim.close()
