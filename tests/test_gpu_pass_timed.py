"""FPD_FLAG_TIME_KERNELS times the path that fpd_step takes: on a lattice of passes one lattice pass
for four steps, each step's bead kernel, and the steps left over as single ones; the same bits."""
import numpy as np
import pytest

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu


def channel(storage, beads):
    return workloads.Workload(name="timed", nx=2048, ny=520, u_wall=0.02, nu_f=0.05,
                              eta_ratio=20.0, xi=0.8, n_beads=beads, radius=1.5, l0=3.0, k_s=0.45,
                              k_b=2e-3, theta0=0.7, cx=1000.0, cy=260.0, steps=0, storage=storage)


@pytest.mark.parametrize("storage,beads", [("f64", 8), ("f32", 8), ("bf16dev", 8), ("f32", 0)])
def test_timed_passes(storage, beads):
    w = channel(storage, beads)
    print(f"[case] timed passes {storage} {beads} beads", flush=True)
    with _lib.simulation_from_workload(w, flags=_lib.FPD_FLAG_TIME_KERNELS) as a, \
            _lib.simulation_from_workload(w) as b:
        for n in (31, 8, 2, 600):            # 7, 2, 0 and 150 passes; 3, 0, 2 and 0 single steps
            a.step(n)
            b.step(n)
        assert a.steps == b.steps == 641
        for x, y in zip((a.populations(), *a.beads()), (b.populations(), *b.beads())):
            assert np.array_equal(x, y)
        ms_lat, n_lat, ms_bead, n_bead = a.kernel_times()
        assert n_lat == 7 + 2 + 150 + 3 + 2 and n_bead == (641 if beads else 0)
        assert ms_lat > 0 and (ms_bead > 0) == (beads > 0)
        a.reset_kernel_times()
        a.step(40)
        ms_lat, n_lat, _, _ = a.kernel_times()
        # (far within these bounds: a pass reads and writes every population at least once)
        copy = 2 * 9 * w.nx * w.ny * {"f64": 8, "f32": 4, "bf16dev": 2}[storage] / 6.6e12 * 1e3
        assert n_lat == 10 and 0.5 * copy < ms_lat / n_lat < 40 * copy
