"""Unstable runs on the path of passes: a bead that outruns its patch is not pulled from it.  The run
is reported by health bits, and the other members of a batch keep their results."""
import numpy as np
import pytest

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu


def channel(nx, ny, storage, **over):
    kw = dict(name="unstable", nx=nx, ny=ny, u_wall=0.02, nu_f=0.05, eta_ratio=20.0, xi=0.8,
              n_beads=8, radius=1.5, l0=3.0, k_s=0.45, k_b=2e-3, theta0=0.7, cx=nx / 2 + 0.3,
              cy=ny / 2, steps=0, storage=storage)
    kw.update(over)
    return workloads.Workload(**kw)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
def test_unstable_member_leaves_a_batch_that_takes_passes(storage):
    good, bad = channel(1024, 512, storage), channel(900, 400, storage, k_s=1e6)
    print(f"[case] eviction under passes {storage}", flush=True)
    with _lib.simulation_from_workload(good) as sim:
        sim.step(96)
        ref = (sim.populations(), *sim.beads())
    with _lib.Batch(hbm_budget=1 << 33, max_slots=4, storage=storage) as b:
        b.set_launch(dict(graph_chunk=8))
        ids = [b.add(_lib.params_from_mapping(w.params(), storage=storage), w.beads(), 96)
               for w in (good, bad)]
        while b.run(32):
            pass
        status = dict(b.poll())
        assert status == {ids[0]: _lib.FPD_SIM_DONE, ids[1]: _lib.FPD_SIM_FAILED}
        assert b.info(ids[1])[2] != 0
        for x, y in zip((b.populations(ids[0]), *b.beads(ids[0])), ref):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("boundary", [0, 1])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_unstable_run_on_a_large_lattice_is_reported(storage, boundary):
    over = dict(boundary=1, u_wall=0.0, init_flow=0) if boundary else {}
    w = channel(2048, 520, storage, k_s=1e6, **over)
    print(f"[case] unstable pass {storage} boundary={boundary}", flush=True)
    with _lib.simulation_from_workload(w) as sim:
        sim.set_launch(dict(graph_chunk=8))
        sim.step(45)
        with pytest.raises(_lib.FpdError) as err:
            sim.sync()
        assert err.value.code == _lib.FPD_EUNSTABLE
        assert sim.health()[0] != 0
        assert sim.populations().shape == (9, 520, 2048)  # (still readable)
