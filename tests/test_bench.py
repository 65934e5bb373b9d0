"""What the benchmark times (no GPU: a recording context in place of the estimator)."""
import types

import pytest
import torch

import bench


class Recorder:
    """Context and event calls in order; `timing` tells the launch timing's state at each."""

    def __init__(self):
        self.log, self.timing = [], False

    def event(self, **kw):
        return types.SimpleNamespace(record=lambda: self.log.append(("event", self.timing)),
                                     elapsed_time=lambda other: 12.0)

    def set_tuning(self, *t):
        self.log.append(("tuning", t))

    def new_accumulators(self):
        return torch.zeros(3, dtype=torch.int64), torch.ones(3, dtype=torch.int32)

    def estimate_grad(self, th, views, tg, seed, t, n_pairs, eps, Q, K):
        self.log.append(("estimate", self.timing, t, th.item()))

    def step(self, th, m, v, t, *a, **kw):
        self.log.append(("step", self.timing, t))
        th += 1.0

    def timing_enable(self, on):
        self.timing = on

    def timing_read(self, reset):
        return {"tile_ms": 1.0, "tile_launches": 2}


@pytest.mark.parametrize("steps,warmup", [(1, 0), (4, 2)])
def test_context_modes_are_timed_as_a_program_runs_them(steps, warmup):
    """The timed steps run without launch timing, which keeps an estimate's
    launches on one stream; the kernels are timed in a second pass over the same
    steps."""
    rec = Recorder()
    fake = types.SimpleNamespace(int64=torch.int64, cuda=types.SimpleNamespace(
        synchronize=lambda: rec.log.append(("sync", rec.timing)), Event=rec.event))
    sc = types.SimpleNamespace(n_pairs=2, views=[], seed=1, lr=[1e-3])
    api = types.SimpleNamespace(ADAM=0, AVG_COUNT=0)
    th = torch.zeros(1)
    r = bench.run_mode(rec, sc, th, torch.zeros(1), torch.zeros(1), None, [1e-3], steps, warmup, (16, 256, 1), api, fake)
    assert r["ms_per_step"] == 12.0 / steps and r["timing"]["tile_launches"] == 2
    a, b = [i for i, e in enumerate(rec.log) if e[0] == "event"]
    timed = rec.log[a + 1: b]
    assert [e[0] for e in timed] == ["estimate", "step"] * steps
    assert not any(e[1] for e in timed)
    assert [e[2] for e in timed if e[0] == "estimate"] == list(range(warmup + 1, warmup + steps + 1))
    kernels = [e for e in rec.log[b:] if e[0] in ("estimate", "step") and e[1]]
    assert [(e[0],) + e[2:] for e in kernels] == [(e[0],) + e[2:] for e in timed]
