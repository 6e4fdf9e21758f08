"""Reads into pinned host memory, which the kernels write in place, against reads through the
staging array of ordinary memory: the same values, no tolerance."""
import ctypes

import numpy as np
import pytest
import torch

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu


def ptr(a):
    return None if a is None else a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
@pytest.mark.parametrize("nx,ny", [(64, 32), (778, 333)])
def test_reads_into_pinned_memory(nx, ny, storage):
    print(f"[case] pinned read {nx}x{ny} {storage}", flush=True)
    w = workloads.Workload(name="read", nx=nx, ny=ny, u_wall=0.02, nu_f=0.05, eta_ratio=20.0,
                           xi=0.8, n_beads=4, radius=1.5, l0=3.0, k_s=0.45, k_b=2e-3,
                           theta0=0.3, cx=nx / 2, cy=ny / 2, steps=0, storage=storage)
    lib = _lib.lib()
    with _lib.simulation_from_workload(w, storage=storage) as sim:
        sim.step(7)
        n = nx * ny
        ordinary = np.zeros((13, ny, nx))
        # an odd offset into a larger pinned array, which keeps its other values
        whole = torch.full((13 * n + 9,), -7.0, dtype=torch.float64, pin_memory=True).numpy()
        pinned = whole[5:5 + 13 * n].reshape(13, ny, nx)
        for out in (ordinary, pinned):
            _lib.check(lib.fpd_read_fields(sim.h, *[ptr(out[i]) for i in range(4)]))
            _lib.check(lib.fpd_read_populations(sim.h, ptr(out[4:])))
        assert np.array_equal(pinned, ordinary)
        assert np.all(whole[:5] == -7.0) and np.all(whole[5 + 13 * n:] == -7.0)
        # some outputs only, and pinned ones beside ordinary ones
        pinned[:4] = 0.0
        _lib.check(lib.fpd_read_fields(sim.h, None, ptr(pinned[1]), None, ptr(pinned[3])))
        other = np.zeros((ny, nx))
        _lib.check(lib.fpd_read_fields(sim.h, ptr(pinned[0]), ptr(other), None, None))
        assert np.array_equal(pinned[[0, 1, 3]], ordinary[[0, 1, 3]])
        assert np.array_equal(other, ordinary[1]) and not pinned[2].any()
        # up to the end of the pinned array
        tail = whole[-n:].reshape(ny, nx)
        _lib.check(lib.fpd_read_fields(sim.h, ptr(tail), None, None, None))
        assert np.array_equal(tail, ordinary[0])
