"""How long batches take.  The autotuner's pick is no slower than a default
configuration, also where the tasks are few and short, and a cache file of a
library with other plans is not taken; a batch's tiles cost little by
themselves, however many there are."""
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


def test_cache_of_other_plans_is_not_taken(ctx, tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("PRAND_TUNE_CACHE", str(path))
    tasks = _tasks(ctx, [(P.GM29, 5000), (P.MRG32K3A, 7000)])
    P.autotune(ctx, tasks)
    key = path.read_text().split("\t")[0]
    old = key[key.index("gfx950"):]   # the key as it was before plans had a version
    path.write_text(f"{old}\t1 32 64 16 1\n")
    best = P.autotune(ctx, tasks)
    assert (best.waves_per_block, best.reg_section, best.gm_section) != (1, 32, 64)
    assert path.read_text().count("\n") == 2
    # what this library wrote is taken
    path.write_text(f"{key}\t2 64 128 16 2\n")
    best = P.autotune(ctx, tasks)
    assert (best.waves_per_block, best.reg_section, best.gm_section, best.overlap) == (2, 64, 128, 2)


def test_many_tiles_cost_little(ctx):
    n = 10**7
    tasks = _tasks(ctx, [(P.GM19, n)])
    state, out = ctx.seed(P.GM19, 1), torch.empty(n, dtype=torch.float32, device="cuda")
    single = 1e9
    for _ in range(30):
        a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        ctx.generate(P.GM19, state, P.F32, out, n)
        z.record()
        z.synchronize()
        single = min(single, a.elapsed_time(z))
    # 10^4 tiles: 67 us and 57 by the single call; 203 with a counter they are taken from
    assert _time(ctx, tasks, P.BatchConfig(use_graph=1)) <= 2.5 * single
