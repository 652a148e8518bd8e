"""The autotuner ranks pushes, not blocks: blocks from which the library takes
the same work-group share the best of their times, and the first of them
listed is returned."""
import types

from paper_1906_06306_amd import autotune


class FakeSim:
    threads = {(8, 64): 64, (8, 128): 256, (8, 256): 256, (16, 64): 768, (16, 128): 768, (16, 256): 512}

    def __init__(self, plasma, tile, precision, block, capacity_factor):
        self.key, self.stepped = (tile[0], block), False

    def push_threads(self):
        assert self.stepped            # known from the first push on
        return self.threads[self.key]

    def close(self):
        pass


def test_equal_pushes_share_their_best_time(monkeypatch):
    times = {(8, 64): 5.0, (8, 128): 3.5, (8, 256): 3.0, (16, 64): 2.6, (16, 128): 2.0, (16, 256): 2.5}

    def time_step(sim, steps):
        sim.stepped = True
        return times[sim.key]

    monkeypatch.setattr(autotune, "PicSim", FakeSim)
    monkeypatch.setattr(autotune, "time_step", time_step)
    lines = []
    best, res = autotune.tune(types.SimpleNamespace(D=2, n=(16, 16, 1)), "fp32", blocks=(64, 128, 256),
                              log=lines.append)
    assert res == {(8, 64): 5.0, (8, 128): 3.0, (8, 256): 3.0, (16, 64): 2.0, (16, 128): 2.0, (16, 256): 2.5}
    assert best == (16, 64)
    assert len(lines) == 6 and "block=128 (push 768): 2000.000 ms" in lines[4]
