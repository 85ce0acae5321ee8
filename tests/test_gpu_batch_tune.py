"""The batch autotuner: its pick is no slower than a default configuration,
also where the tasks are few and short."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


def _tasks(ctx, specs):
    tasks = []
    for k, (gen, n) in enumerate(specs):
        sin = torch.from_numpy(ctx.seed(gen, 1000 + k)).cuda()
        tasks.append((gen, P.F32, n, sin, torch.empty_like(sin), torch.empty(n, dtype=torch.float32, device="cuda")))
    return tasks


def _time(ctx, tasks, cfg):
    """The fastest of 30 launches, in ms."""
    b = P.Batch(ctx, tasks, cfg)
    best = 1e9
    for _ in range(30):
        a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        b.launch()
        z.record()
        z.synchronize()
        best = min(best, a.elapsed_time(z))
    b.close()
    return best


def test_pick_is_no_slower_than_the_default(ctx, monkeypatch):
    monkeypatch.delenv("PRAND_TUNE_CACHE", raising=False)
    r = np.random.default_rng(3)
    tasks = _tasks(ctx, [(P.MRG32K3A + k % 2, int(n)) for k, n in enumerate(np.exp(r.uniform(7, 13.8, 16)))])
    best = P.autotune(ctx, tasks)
    default = _time(ctx, tasks, P.BatchConfig(use_graph=1))
    # a section length of 2048 takes three times the default's here
    assert _time(ctx, tasks, best) <= 1.5 * default

