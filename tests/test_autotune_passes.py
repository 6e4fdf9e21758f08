"""The autotuner times launch shapes on steps that use them: a workload large enough for passes of
four steps (which do not) is timed in graphs of two steps, a smaller one as it runs."""
import types

import pytest

from paper_2212_14153_amd import autotune


class Clock:
    t = 0.0

    def perf_counter(self):
        self.t += 1e-3
        return self.t


class Sim:
    def __init__(self):
        self.cfg, self.timed = dict(graph_chunk=64), set()

    def get_launch(self):
        return types.SimpleNamespace(graph_chunk=self.cfg["graph_chunk"])

    def set_launch(self, cfg):
        self.cfg = dict(self.cfg, **cfg)

    def step(self, n):
        self.timed.add(self.cfg["graph_chunk"])

    def run(self, n):
        self.step(n)

    def sync(self):
        pass

    def close(self):
        pass


@pytest.fixture(autouse=True)
def no_clock_no_cache(tmp_path, monkeypatch):
    monkeypatch.setattr(autotune, "time",
                        types.SimpleNamespace(perf_counter=Clock().perf_counter))
    monkeypatch.setenv("FPD_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))


@pytest.mark.parametrize("nodes,chunk", [((1 << 20) - 1, 64), (1 << 20, 2), (1 << 24, 2)])
def test_simulations(nodes, chunk):
    sim = Sim()
    autotune.tune_simulation(sim, "f32", nodes, restore=False)
    assert sim.timed == {chunk} and sim.cfg["graph_chunk"] == 64


@pytest.mark.parametrize("nodes,chunk", [((3 << 18) - 1, 8), (3 << 18, 2), (1 << 24, 2)])
def test_batches(nodes, chunk):
    b = Sim()
    autotune.tune_batch(lambda: b, "f32", nodes)
    assert b.timed == {chunk}
