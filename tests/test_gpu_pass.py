"""Passes of several steps against whole steps.  A large lattice advances four steps per pass:
the fluid away from the fiber in one kernel that marches the steps up the rows in registers,
the nodes around the fiber step by step in patch buffers.  Every node gets the arithmetic of a
whole step in the same order, so populations and beads must be the same bits: no tolerance."""
import math

import numpy as np
import pytest

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu


def channel(nx, ny, storage, cx, cy, theta, boundary=0, beads=8, **over):
    kw = dict(name="pass", nx=nx, ny=ny, u_wall=0.02, nu_f=0.05, eta_ratio=20.0, xi=0.8,
              n_beads=beads, radius=1.5, l0=3.0, k_s=0.45, k_b=2e-3, theta0=theta, cx=cx,
              cy=cy, steps=0, storage=storage, boundary=boundary)
    if boundary == 1:
        kw.update(u_wall=0.0, init_flow=0, f_ext=(2e-4, 1e-4))
    kw.update(over)
    return workloads.Workload(**kw)


def run(w, flags, chunk, counts):
    with _lib.simulation_from_workload(w, storage=w.storage, flags=flags) as sim:
        f = sim.populations()
        f = f + workloads.perturbation(f.shape, 1e-3, seed=w.nx + w.ny)
        sim.write_populations(f)
        sim.set_launch(dict(graph_chunk=chunk))
        for n in counts:
            sim.step(n)
        sim.sync()
        return sim.populations(), sim.beads(), sim.steps


def same(w, chunk=8, counts=(3, 19, 6)):
    print(f"[case] pass {w.nx}x{w.ny} {w.storage} boundary={w.boundary} beads={w.n_beads} "
          f"chunk={chunk} counts={counts}", flush=True)
    f0, b0, n0 = run(w, _lib.FPD_FLAG_NO_SPLIT, chunk, counts)
    for flags in (0, _lib.FPD_FLAG_NO_GRAPH):
        f, b, n = run(w, flags, chunk, counts)
        assert n == n0
        assert np.array_equal(f, f0)
        for x, y in zip(b, b0):
            assert np.array_equal(x, y)


STORAGE = ["f64", "f32", "f16dev", "bf16dev"]


@pytest.mark.parametrize("storage", STORAGE)
def test_passes_are_bitwise_whole_steps(storage):
    same(channel(2050, 513, storage, cx=700.0, cy=250.0, theta=0.7))


@pytest.mark.parametrize("storage", STORAGE)
def test_passes_at_the_walls_and_the_periodic_edge(storage):
    """The partition wraps along x and is clipped at the lower wall."""
    same(channel(2048, 512, storage, cx=1.0, cy=14.0, theta=0.0))


@pytest.mark.parametrize("storage", STORAGE)
def test_passes_in_a_periodic_box_corner(storage):
    """No walls: the partition wraps along both axes; a body force on every node."""
    same(channel(1036, 1030, storage, cx=2.0, cy=1028.0, theta=0.9, boundary=1,
                 g_body=(1e-6, -2e-6)))


@pytest.mark.parametrize("nx,ny,storage", [
    (1049, 1003, "f32"),        # odd columns: one column per lane
    (1049, 1003, "f64"), (1049, 1003, "f16dev"),   # two-byte formats: no passes for odd nx
    (65600, 16, "f32"), (65600, 17, "bf16dev"),    # few rows: every row near a wall
    (64, 16500, "f32"), (130, 8200, "f64")])       # one or two strips, many rows
def test_pass_shapes(nx, ny, storage):
    """Lattices whose strips and row runs end in remainders, without a fiber."""
    same(channel(nx, ny, storage, cx=0.0, cy=0.0, theta=0.0, beads=0), counts=(9, 4, 2))


@pytest.mark.parametrize("chunk", [2, 4, 6, 64])
def test_passes_in_graph_chunks(chunk):
    """Chunks of an even and an odd number of passes, with and without single steps."""
    same(channel(2048, 520, "f32", cx=1000.0, cy=260.0, theta=1.2), chunk=chunk,
         counts=(1, 2 * chunk + 7, 3))


@pytest.mark.parametrize("chunk", [10, 22, 50])
def test_chunks_are_rounded_to_whole_passes(chunk):
    """Odd and even numbers of passes a chunk, calls just below and at the chunk's length."""
    same(channel(2048, 520, "f32", cx=1000.0, cy=260.0, theta=1.2), chunk=chunk,
         counts=(chunk - 3, chunk, 3 * chunk + 1, chunk - 1))


def test_recording_and_checkpoint_between_passes(tmp_path):
    w = channel(2048, 512, "f32", cx=900.0, cy=256.0, theta=math.pi / 3)
    path = str(tmp_path / "pass.ckpt")
    out = []
    for flags in (_lib.FPD_FLAG_NO_SPLIT, 0):
        with _lib.simulation_from_workload(w, storage="f32", flags=flags) as sim:
            sim.record_start(every=3, capacity=8)
            sim.step(13)
            sim.save(path)
            sim.step(9)
            sim.load(path)
            sim.step(9)
            sim.sync()
            out.append((sim.populations(), *sim.beads(), sim.record()))
    for x, y in zip(*out):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("storage", STORAGE)
def test_passes_of_several_fibers(storage):
    """One patch per fiber: apart, close enough that their partitions share nodes, and across
    the periodic edge; with the excluded volume on."""
    w = workloads.fiber_suspension(n_fibers=3, beads=6, nx=2048, ny=512, radius=3.0,
                                   storage=storage, seed=11)
    centres = ((300.0, 200.0, 0.4), (322.0, 215.0, 1.9), (2046.0, 300.0, 0.1))
    same(w.with_(centres=centres, ev_k=1e-3, ev_range=9.0))


@pytest.mark.parametrize("nx,ny,storage", [(2048, 1024, "f32"), (2049, 1100, "f64"),
                                           (8192, 300, "bf16dev")])
def test_passes_of_many_fibers(nx, ny, storage):
    """From 12 fibers on the march takes shorter runs of rows."""
    same(workloads.fiber_suspension(n_fibers=13, beads=5, nx=nx, ny=ny, radius=2.5,
                                    storage=storage, seed=3), counts=(3, 9))


@pytest.mark.parametrize("storage", STORAGE)
def test_passes_of_a_batch(storage):
    """Walls, a periodic box under a body force (odd columns where passes take them), no fiber and
    two fibers in one batch, against single steps; members leave at different times, the rest is
    then too small for passes, and one records its fiber's ends."""
    odd = storage in ("f64", "f32")
    two = workloads.fiber_suspension(n_fibers=2, beads=6, nx=800, ny=400, radius=3.0,
                                     storage=storage, seed=5)
    ws = [channel(702, 257, storage, cx=350.0, cy=120.0, theta=0.7),
          channel(601 if odd else 602, 420, storage, cx=2.0, cy=418.0, theta=0.9, boundary=1,
                  g_body=(1e-6, -2e-6)),
          channel(1000, 301, storage, cx=0.0, cy=0.0, theta=0.0, beads=0),
          two.with_(centres=((200.0, 200.0, 0.4), (222.0, 215.0, 1.9)))]
    targets = [41, 29, 41, 36]
    print(f"[case] batch passes {storage} {[(w.nx, w.ny, w.n_beads) for w in ws]}", flush=True)
    out = []
    for flags, chunk in ((_lib.FPD_FLAG_NO_SPLIT, 64), (0, 8), (0, 64), (0, 2)):
        with _lib.Batch(hbm_budget=1 << 33, max_slots=8, storage=storage) as b:
            b.set_launch(dict(graph_chunk=chunk))
            ids = [b.add(_lib.params_from_mapping(w.params(), storage=storage, flags=flags),
                         w.beads(), t) for w, t in zip(ws, targets)]
            b.record_start(ids[0], every=3, capacity=16)
            while b.run(17):
                pass
            got = [b.record(ids[0])]
            for sid in ids:
                got += [b.populations(sid), *b.beads(sid)]
            out.append(got)
    for got in out[1:]:
        for x, y in zip(got, out[0]):
            assert np.array_equal(x, y)
