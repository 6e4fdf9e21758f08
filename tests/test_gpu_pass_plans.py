"""Passes whose patches meet the edges of a plan: as wide as the lattice, as tall as a periodic box,
taller than one run of plan rows; and binary16 passes against whole steps of every launch shape.
The bits of whole steps, no tolerance."""
import math

import numpy as np
import pytest

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu


def channel(nx, ny, storage, boundary=0, **over):
    kw = dict(name="plan", nx=nx, ny=ny, u_wall=0.02, nu_f=0.05, eta_ratio=20.0, xi=0.8,
              n_beads=8, radius=1.5, l0=3.0, k_s=0.45, k_b=2e-3, theta0=0.3, cx=nx / 2,
              cy=ny / 2, steps=0, storage=storage, boundary=boundary)
    if boundary:
        kw.update(u_wall=0.0, init_flow=0, f_ext=(2e-4, 1e-4))
    kw.update(over)
    return workloads.Workload(**kw)


def alone(w, flags, counts, **launch):
    with _lib.simulation_from_workload(w, flags=flags) as sim:
        f = sim.populations()
        sim.write_populations(f + workloads.perturbation(f.shape, 1e-3, seed=w.nx + w.ny))
        sim.set_launch(dict(graph_chunk=8, **launch))
        for n in counts:
            sim.step(n)
        return (sim.populations(), *sim.beads())


def same(got, ref):
    for x, y in zip(got, ref):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
def test_patches_that_span_small_lattices(storage):
    """A batch of 110 lattices of 64 to 110 nodes a side, fibers about as long as these: patches as
    wide as the lattice and as tall as the box, some of them only in one direction."""
    rng = np.random.default_rng(3)
    odd = storage in ("f64", "f32")
    ws = []
    while sum(w.nx * w.ny for w in ws) < 800_000:
        nx, ny = int(rng.integers(64, 111)), int(rng.integers(64, 111))
        if not odd:
            nx -= nx % 2
        per, n = int(rng.integers(0, 2)), int(rng.integers(1, 13))
        ws.append(channel(nx, ny, storage, per, n_beads=n, l0=4.0,
                          theta0=float(rng.uniform(0.0, math.pi)), cx=float(rng.uniform(0, nx)),
                          cy=float(rng.uniform(0, ny)) if per else ny / 2))
    print(f"[case] spanning patches {storage}, {len(ws)} lattices", flush=True)
    out = []
    for flags in (_lib.FPD_FLAG_NO_SPLIT, 0):
        with _lib.Batch(1 << 33, len(ws), storage=storage) as b:
            b.set_launch(dict(graph_chunk=8))
            ids = [b.add(_lib.params_from_mapping(w.params(), storage=storage, flags=flags,
                                              cutoff=6.0), w.beads(), 1 << 20) for w in ws]
            b.run(30)
            out.append([x for sid in ids for x in (b.populations(sid), *b.beads(sid))])
    same(*out)


@pytest.mark.parametrize("boundary,cy", [(0, 550.0), (1, 1000.0)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_a_patch_of_two_runs_of_plan_rows(storage, boundary, cy):
    """A steep fiber of 640 nodes, between walls and across the periodic edge."""
    w = channel(4096, 1100, storage, boundary, n_beads=40, radius=4.0, l0=16.0,
                theta0=math.pi / 2 - 0.1, cy=cy)
    print(f"[case] tall patch {storage} boundary={boundary}", flush=True)
    same(alone(w, 0, (19,)), alone(w, _lib.FPD_FLAG_NO_SPLIT, (19,)))


@pytest.mark.parametrize("g_body", [(0.0, 0.0), (1e-6, 0.0)])
def test_binary16_passes_against_every_shape_of_whole_steps(g_body):
    w = channel(2048, 512, "f16dev", g_body=g_body)
    print(f"[case] f16dev shapes g={g_body}", flush=True)
    got = alone(w, 0, (16,))
    for rows in (1, 2, 4):
        same(got, alone(w, _lib.FPD_FLAG_NO_SPLIT, (16,), rows_per_thread=rows))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
def test_passes_of_the_smallest_lattices(storage):
    """One to nine nodes a side, with and without walls, in a batch that takes passes: a wave's
    columns go round the lattice many times, a row is its own neighbour."""
    ws = [channel(nx, ny, storage, per, n_beads=0, f_ext=(0.0, 0.0))
          for nx in ((1, 2, 3, 5, 8, 9) if storage in ("f64", "f32") else (2, 4, 6, 8))
          for ny in (1, 2, 3, 4, 5, 9) for per in (0, 1)]
    ws.append(channel(1024, 768, storage, n_beads=0))
    print(f"[case] smallest lattices {storage}", flush=True)
    out = []
    for flags in (_lib.FPD_FLAG_NO_SPLIT, 0):
        with _lib.Batch(1 << 33, len(ws), storage=storage) as b:
            b.set_launch(dict(graph_chunk=8))
            ids = [b.add(_lib.params_from_mapping(w.params(), storage=storage, flags=flags,
                                                  g_body=(1e-5, -2e-5)), None, 1 << 20)
                   for w in ws]
            b.run(21)
            out.append([b.populations(sid) for sid in ids])
    same(*out)
