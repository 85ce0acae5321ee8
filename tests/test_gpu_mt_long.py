"""MT19937 where other tests compare a plan with itself or do not reach: one
state cut into sections of twice and four times the shortest length (more than
512 of those), against the many-stream call, which has no sections; and whole-
section jumps in each launch shape (16, 8 and 4 wavefronts per stream) against
the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

SHORTEST = 624 << 8    # outputs of a section
MOST = 512             # sections


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    c.init_stream(P.MT19937, P.SEQ_DEFAULT, 1)   # builds the jump tables
    yield c
    c.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("used", [0, 300])   # words of the state's block already used (624 - used are left)
@pytest.mark.parametrize("sections,more", [(MOST, 0), (MOST, 1), (2 * MOST, 1)])
def test_longer_sections(ctx, oracle, used, sections, more):
    st = oracle.seed(P.MT19937, 31)
    oracle.generate(P.MT19937, st, 624 + used, P.U32)
    n = (624 - used) % 624 + sections * SHORTEST + more
    d = torch.from_numpy(st.copy()).cuda()
    ref, out = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.generate_streams(P.MT19937, d, 1, n, P.U32, ref)
    end = d.cpu().numpy()
    for call in (ctx.generate, ctx.generate_noalloc):
        mine = st.copy()
        out.fill_(0)
        call(P.MT19937, mine, P.U32, out, n)
        assert torch.equal(out, ref)
        np.testing.assert_array_equal(mine, end)


@pytest.mark.parametrize("count", [512, 4096, 4097])
def test_whole_section_jumps(ctx, oracle, count):
    fn = ctx.lib.prand_internal_mt_jump_sections
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]
    sb, section = P.state_bytes(P.MT19937), 624 << 10
    starts, dists = [], []
    for k, used in enumerate([0, 1, 300, 624]):
        st = oracle.seed(P.MT19937, 900 + k)
        oracle.generate(P.MT19937, st, used, P.U32)
        for d in [0, 1, 17, 255, 2**22 - 1, 2**22]:
            starts.append(st.copy())
            dists.append(d)
    refs = [oracle.skipahead(P.MT19937, s.copy(), d * section) for s, d in zip(starts, dists)]
    m = len(starts)
    # a few kinds repeated over the launch
    states = torch.from_numpy(np.concatenate([starts[k % m] for k in range(count)])).cuda()
    secs = torch.tensor([dists[k % m] for k in range(count)], dtype=torch.int64, device="cuda")
    assert fn(ctx.handle, states.data_ptr(), count, secs.data_ptr(), None) == P.OK
    torch.cuda.synchronize()
    got = states.cpu().numpy().reshape(count, sb)
    for k in range(count):
        assert np.array_equal(got[k], refs[k % m]), (k, dists[k % m])
