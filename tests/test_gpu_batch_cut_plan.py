"""Which MT19937 tasks of a batch are cut into sections: those of more than
three sections whose workgroup would outlast the rest of the batch, and only
where the context has its jump tables; the caller sees one tile each."""
import ctypes

import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

SECTION = 624 << 10


def _cut(ctx, specs):
    fn = ctx.lib.prand_internal_batch_cut
    fn.restype, fn.argtypes = ctypes.c_uint32, [ctypes.c_void_p]
    tasks = []
    for gen, n in specs:
        sin = torch.from_numpy(ctx.seed(gen, 5)).cuda()
        tasks.append((gen, P.U32, n, sin, torch.empty_like(sin), torch.empty(n, dtype=torch.int32, device="cuda")))
    b = P.Batch(ctx, tasks)
    cut = fn(b.handle)
    if all(gen == P.MT19937 for gen, _ in specs):
        assert b.tiles() == len(specs)
    b.close()
    return cut


def test_cut_sections():
    ctx = P.Context(0)
    long = [(P.MT19937, 3 * SECTION + 1), (P.MT19937, 5 * SECTION), (P.MT19937, 7 * SECTION + 625)]
    assert _cut(ctx, long) == 0                        # no tables yet
    ctx.init_stream(P.MT19937, P.SEQ_DEFAULT, 1)       # builds them
    assert _cut(ctx, long) == 3 + 4 + 7
    assert _cut(ctx, [(P.MT19937, 3 * SECTION)]) == 0
    # beside GM61 outputs that take the chip longer (8.9 ms per 2^30) than the
    # task's workgroup takes (0.45 ns per output)
    n = 3 * SECTION + 1
    rest = int(n * 0.45e-6 / 8.9 * 2**30)
    assert _cut(ctx, [(P.MT19937, n), (P.GM61, rest + rest // 10)]) == 0
    assert _cut(ctx, [(P.MT19937, n), (P.GM61, rest - rest // 10)]) == 3
    ctx.close()
