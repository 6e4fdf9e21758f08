"""Fibers longer than a pass's patches hold (more than 1.5 times their contour): the passes then take
the whole lattice, step by step, with the bits of whole steps."""
import math

import numpy as np
import pytest

import workloads
from paper_2212_14153_amd import _lib

pytestmark = pytest.mark.gpu

BEADS, L0 = 6, 3.0


def two_fibers(nx, ny, storage, boundary=0, **over):
    kw = dict(name="long", nx=nx, ny=ny, u_wall=0.05, nu_f=0.05, eta_ratio=20.0, xi=0.8,
              n_beads=2 * BEADS, radius=1.5, l0=L0, k_s=0.0, k_b=2e-3, theta0=0.0, cx=nx / 2,
              cy=ny / 2, steps=0, storage=storage, boundary=boundary)
    if boundary:
        kw.update(u_wall=0.0, init_flow=0, f_ext=(2e-4, 1e-4), g_body=(1e-5, 0.0))
    kw.update(over)
    return workloads.Workload(**kw)


def positions(w, bond, theta, c0, c1):
    out = []
    for cx, cy in (c0, c1):
        for i in range(BEADS):
            t = (i - (BEADS - 1) / 2) * bond
            out.append((cx + t * math.cos(theta), cy + t * math.sin(theta)))
    return np.array(out)


def params(w, storage, flags):
    return _lib.params_from_mapping(w.params(), storage=storage, flags=flags, n_chains=2)


def alone(w, R, flags, chunk, counts):
    with _lib.Simulation(params(w, w.storage, flags)) as sim:
        sim.init_fiber(R)
        sim.set_launch(dict(graph_chunk=chunk))
        for n in counts:
            sim.step(n)
        return (sim.populations(), *sim.beads())


@pytest.mark.parametrize("boundary", [0, 1])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
def test_a_fiber_longer_than_its_patch(storage, boundary):
    """From the start, one of two fibers, near the edge: passes of both parities, single steps
    behind them."""
    w = two_fibers(2050, 513, storage, boundary)
    R = positions(w, 2.4 * L0, 0.6, (30.0, 260.0), (900.0, 200.0))
    R[BEADS:] = positions(w, L0, 0.3, (900.0, 200.0), (900.0, 200.0))[BEADS:]
    print(f"[case] long fiber {storage} boundary={boundary}", flush=True)
    counts = (5, 22, 9)
    ref = alone(w, R, _lib.FPD_FLAG_NO_SPLIT, 8, counts)
    for flags in (0, _lib.FPD_FLAG_NO_GRAPH):
        for x, y in zip(alone(w, R, flags, 8, counts), ref):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("start", [0.0, 0.6, 1.2, 1.8])
def test_a_fiber_grows_past_its_patch(start):
    """The shear draws a fiber without springs out, 0.03 nodes a step, across the limit."""
    w = two_fibers(2048, 512, "f32", u_wall=0.09)
    span = 1.5 * (BEADS - 1) * L0 + 5.5 + start
    R = positions(w, span * math.sqrt(2.0) / (BEADS - 1), math.pi / 4, (700.3, 256.0),
                  (1500.7, 250.0))
    R[:, 1] = (R[:, 1] - 253.0) * 4.0 + 253.0   # (steep: the upper beads run ahead)
    print(f"[case] growing fiber {start}", flush=True)
    ref = alone(w, R, _lib.FPD_FLAG_NO_SPLIT, 8, (150,))
    for x, y in zip(alone(w, R, 0, 8, (150,)), ref):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
def test_a_long_fiber_in_a_batch(storage):
    """One member's passes are whole, the others' are not."""
    ws = [two_fibers(900, 500, storage), two_fibers(640, 400, storage, 1),
          two_fibers(701 if storage in ("f64", "f32") else 702, 300, storage)]
    Rs = [positions(w, b * L0, 0.6, (30.0, 140.0), (400.0, 160.0))
          for w, b in zip(ws, (1.0, 2.3, 2.3))]
    print(f"[case] long fibers in a batch {storage}", flush=True)
    out = []
    for flags in (_lib.FPD_FLAG_NO_SPLIT, 0):
        got = []
        with _lib.Batch(hbm_budget=1 << 33, max_slots=4, storage=storage) as b:
            b.set_launch(dict(graph_chunk=8))
            ids = [b.add(params(w, storage, flags), R, 1 << 20) for w, R in zip(ws, Rs)]
            b.run(29)                       # (then the long ones' strain evicts them)
            for sid in ids:
                got += [b.populations(sid), *b.beads(sid)]
        out.append(got)
    for x, y in zip(*out):
        assert np.array_equal(x, y)
