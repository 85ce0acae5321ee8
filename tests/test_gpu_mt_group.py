"""MT19937 by a workgroup per stream: lengths around its turns of 227 words,
four turns and blocks, states left inside a block, the stream counts on both
sides of the rule, outputs at any address; values and states against the
oracle."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

NPDT = {P.U32: np.uint32, P.F32: np.float32, P.F64: np.float64}
MAX_COUNT = 1024   # streams up to which a workgroup runs each


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("used", [0, 1, 300, 623, 624])
@pytest.mark.parametrize("n", [1, 226, 227, 228, 623, 624, 625, 907, 908, 909, 1248, 1816, 2500, 9999])
def test_lengths(ctx, oracle, n, used):
    st = oracle.seed(P.MT19937, 99)
    oracle.generate(P.MT19937, st, 624 + used, P.U32)   # `used` words into a block
    for dtype in (P.U32, P.F32, P.F64):
        es = 8 if dtype == P.F64 else 4
        ref = st.copy()
        want = oracle.generate(P.MT19937, ref, n, dtype)
        d = torch.from_numpy(st.copy()).cuda()
        buf = torch.full(((n + 64) * es,), 0x77, dtype=torch.uint8, device="cuda")
        at = 5 * es
        ctx.generate_streams(P.MT19937, d, 1, n, dtype, buf.data_ptr() + at)
        raw = buf.cpu().numpy()
        np.testing.assert_array_equal(raw[at:at + n * es].view(NPDT[dtype]), want)
        assert (raw[:at] == 0x77).all() and (raw[at + n * es:] == 0x77).all()
        np.testing.assert_array_equal(d.cpu().numpy(), ref)


@pytest.mark.parametrize("count", [2, MAX_COUNT - 1, MAX_COUNT, MAX_COUNT + 1])
def test_counts(ctx, oracle, count):
    n = 1999
    sb = P.state_bytes(P.MT19937)
    seeds = torch.arange(1, count + 1, dtype=torch.int64, device="cuda")
    d = torch.empty(count * sb, dtype=torch.uint8, device="cuda")
    ctx.seed_dev(P.MT19937, seeds, count, d)
    out = torch.empty(count * n, dtype=torch.int32, device="cuda")
    ctx.generate_streams(P.MT19937, d, count, n, P.U32, out)
    got, end = out.cpu().numpy().view(np.uint32).reshape(count, n), d.cpu().numpy().reshape(count, sb)
    for s in {0, 1, count // 2, count - 1}:
        st = oracle.seed(P.MT19937, s + 1)
        np.testing.assert_array_equal(got[s], oracle.generate(P.MT19937, st, n, P.U32))
        np.testing.assert_array_equal(end[s], st)
