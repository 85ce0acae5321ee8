"""One host state at the sizes where the plan of a call changes: the ends of
its sections, the counts from which they grow, GM/GQ wavefronts up to and past
those that read the state in host memory, the ballot kernel's first size, one
MT19937 section and two, the array call's direct, pieced and chunked copies.
Long outputs against the many-stream path on the same state, short ones
against the oracle; the state after each, and the bytes around each output."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

NPDT = {P.U32: np.uint32, P.F32: np.float32, P.F64: np.float64}
SEED = 4711
GUARD = 256
SIZES = [(g, n) for g in (P.MRG32K3A, P.LFSR113) for n in (1, 31, 32, 33, 8191, 8193, (1 << 23) - 1, (1 << 23) + 1)]
SIZES += [(g, n) for g in range(P.GM19, P.NUM_GENERATORS) for n in (1, 255, 257, 289, 4097, 65537, 300007, 4200001)]
SIZES += [(g, (1 << 26) + d) for g in (P.GM19, P.GM61) for d in (-1, 0)]
SIZES += [(P.MT19937, n) for n in (1, 623, 625, 1 << 18, (1 << 18) + 1, 624 * 513 - 1, 624 * 512, 624 * 512 + 1, 1000003)]


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


def expected(ctx, oracle, gen, dtype, n):
    """(values, state after them)"""
    st = oracle.seed(gen, SEED)
    if n <= 10000:
        return oracle.generate(gen, st, n, dtype), st
    d = torch.from_numpy(st.copy()).cuda()
    out = torch.empty(n * (8 if dtype == P.F64 else 4), dtype=torch.uint8, device="cuda")
    ctx.generate_streams(gen, d, 1, n, dtype, out)
    return out.cpu().numpy().view(NPDT[dtype]), d.cpu().numpy()


@pytest.mark.parametrize("gen,n", SIZES)
def test_device_output(ctx, oracle, gen, n):
    for dtype in (P.U32, P.F64):
        es = 8 if dtype == P.F64 else 4
        ref, end = expected(ctx, oracle, gen, dtype, n)
        for call in (ctx.generate, ctx.generate_noalloc):
            st = oracle.seed(gen, SEED)
            buf = torch.full((n * es + 2 * GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
            call(gen, st, dtype, buf.data_ptr() + GUARD - 3 * es, n)
            raw = buf.cpu().numpy()
            at = GUARD - 3 * es
            np.testing.assert_array_equal(raw[at:at + n * es].view(NPDT[dtype]), ref)
            assert (raw[:at] == 0x5A).all() and (raw[at + n * es:] == 0x5A).all()
            np.testing.assert_array_equal(st, end)


@pytest.mark.parametrize("used", [1, 300, 623])
def test_mt_sections_from_inside_a_block(ctx, oracle, used):
    """the first section ends on the state's own block grid, wherever in its
    block the state is"""
    st = oracle.seed(P.MT19937, SEED)
    oracle.generate(P.MT19937, st, used, P.U32)
    for n in (624 * 256 + 624 - used, 300007, 624 * 512 + 624 - used, 624 * 512 + 625 - used):
        ref = st.copy()
        want = oracle.generate(P.MT19937, ref, n, P.U32)
        for call in (ctx.generate, ctx.generate_noalloc):
            s = st.copy()
            out = torch.empty(n, dtype=torch.int32, device="cuda")
            call(P.MT19937, s, P.U32, out, n)
            np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)
            np.testing.assert_array_equal(s, ref)


@pytest.mark.parametrize("size", [1, 65535, 65536, 65537, 3 << 19, (3 << 19) + 1, (1 << 24) - 1, (1 << 24) + 5])
@pytest.mark.parametrize("gen", [P.MT19937, P.LFSR113, P.GM31])
def test_array(ctx, oracle, gen, size):
    ref, end = expected(ctx, oracle, gen, P.F32, size)
    for _ in range(2):
        st = oracle.seed(gen, SEED)
        np.testing.assert_array_equal(ctx.generate_array(gen, st, P.F32, size), ref)
        np.testing.assert_array_equal(st, end)


def test_threads_share_a_context(ctx, oracle):
    """array calls, device calls and jumps of one context at the same time"""
    import threading
    want = {g: expected(ctx, oracle, g, P.U32, 70001) for g in (P.MRG32K3A, P.GM55, P.GQ58X3)}
    bad = []

    def work(gen):
        ref, end = want[gen]
        for i in range(20):
            st = oracle.seed(gen, SEED)
            if i % 2:
                got = ctx.generate_array(gen, st, P.U32, ref.size)
            else:
                out = torch.empty(ref.size, dtype=torch.int32, device="cuda")
                (ctx.generate if i % 4 else ctx.generate_noalloc)(gen, st, P.U32, out, ref.size)
                got = out.cpu().numpy().view(np.uint32)
            a = oracle.seed(gen, SEED)
            ctx.skipahead(gen, a, ref.size)
            if not (np.array_equal(got, ref) and np.array_equal(st, end) and np.array_equal(a, end)):
                bad.append((gen, i))

    ts = [threading.Thread(target=work, args=(g,)) for g in want]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
