"""MT19937 tasks that would outlast the rest of their batch are cut into
sections (the caller still sees one tile each): outputs and final states
against the single-stream call, from states inside a block and at its ends,
with the jump tables built before the batch and not."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

SECTION = 624 << 10
TDT = {P.U32: torch.int32, P.F32: torch.float32, P.F64: torch.float64}


@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("tables", [True, False])
def test_long_tasks_of_short_batches(oracle, tables, graph):
    ctx = P.Context(0)
    if tables:
        ctx.init_stream(P.MT19937, P.SEQ_DEFAULT, 1)
    specs = [(0, P.U32, 3 * SECTION), (0, P.U32, 3 * SECTION + 1), (1, P.F32, 4 * SECTION), (300, P.F64, 5 * SECTION - 7),
             (623, P.U32, 7 * SECTION + 625), (624, P.U32, 4 * SECTION + 1), (5, P.U32, 1000), (0, P.U32, 0)]
    tasks, want = [], []
    for k, (used, dt, n) in enumerate(specs):
        st = oracle.seed(P.MT19937, 50 + k)
        oracle.generate(P.MT19937, st, used, P.U32)
        sin = torch.from_numpy(st.copy()).cuda()
        sout = torch.full_like(sin, 0xA5)
        out = torch.zeros(max(n, 1), dtype=TDT[dt], device="cuda")
        ref, end = torch.zeros_like(out), st.copy()
        if n:
            ctx2 = ctx if tables else None
            if ctx2:
                ctx2.generate(P.MT19937, end, dt, ref, n)
            else:
                ref[:n] = torch.from_numpy(oracle.generate(P.MT19937, end, n, dt).view(
                    {P.U32: np.int32, P.F32: np.float32, P.F64: np.float64}[dt])).cuda()
        tasks.append((P.MT19937, dt, n, sin, sout, out))
        want.append((ref, end))
    b = P.Batch(ctx, tasks, P.BatchConfig(use_graph=graph))
    assert b.tiles() == len(specs)
    for _ in range(3):
        for (_, _, _, _, sout, out) in tasks:
            out.zero_()
            sout.fill_(0x5A)
        b.launch()
        torch.cuda.synchronize()
        for (_, _, _, _, sout, out), (ref, end) in zip(tasks, want):
            assert torch.equal(out, ref)
            np.testing.assert_array_equal(sout.cpu().numpy(), end)
    b.close()
    ctx.close()
