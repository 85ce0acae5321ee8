"""Calls of so many streams that one dispatch does not hold them (2^32
work-items; what is beyond wraps, and those streams are left out): MT19937
skip-ahead of 2^24 streams and more, GM/GQ generation of 2^26 (v = 1), 2^27
(GQ58.3) and 2^28 (GM55, GQ58.4) and more, LFSR113 of the largest count.
Streams at both ends and around the seam of the two ranges against the oracle."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    c = P.Context(0)
    yield c
    c.close()
    torch.cuda.empty_cache()


def _room(nbytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < nbytes + (4 << 30):
        pytest.skip("not enough free device memory")


@pytest.mark.parametrize("per_stream", [True, False])
def test_mt19937_skip(ctx, per_stream):
    count, words = 2**24 + 3, P.state_bytes(P.MT19937) // 4
    _room(4 * count * words)
    st = torch.zeros(count * words, dtype=torch.int32, device="cuda")
    i = torch.arange(count, dtype=torch.int64, device="cuda")
    # within the block the distance moves the index alone
    dist = i % 600 if per_stream else torch.tensor([77], dtype=torch.int64, device="cuda")
    rows = st.view(count, words)
    rows[:, 1] = i.to(torch.int32)
    ctx.skipahead_dev(P.MT19937, st, count, dist, 1, per_stream)
    torch.cuda.synchronize()
    assert torch.equal(rows[:, 624].to(torch.int64), dist if per_stream else dist.expand(count))
    assert torch.equal(rows[:, 1], i.to(torch.int32))


@pytest.mark.parametrize("gen,count,per_block,n", [
    (P.GM29, 2**26 + 5, 4, 128), (P.GQ58X3, 2**27 + 5, 8, 3), (P.GM55, 2**28 + 5, 16, 2), (P.LFSR113, 2**32 - 1, 256, 1)])
def test_streams(ctx, oracle, gen, count, per_block, n):
    sb = P.state_bytes(gen)
    _room(count * (sb + 4 * n + 8))
    ids = torch.empty(count, dtype=torch.int64, device="cuda")
    for at in range(0, count, 2**28):   # torch's own launches have limits too
        part = ids[at:at + 2**28]
        part.copy_(torch.arange(3 * at, 3 * (at + len(part)), 3, dtype=torch.int64, device="cuda"))
    st = torch.empty(count * sb, dtype=torch.uint8, device="cuda")
    ctx.init_streams_dev(gen, P.SEQ_DEFAULT, None, ids, count, st)
    out = torch.empty(count * n, dtype=torch.int32, device="cuda")
    ctx.generate_streams(gen, st, count, n, P.U32, out)
    torch.cuda.synchronize()
    seam = (2**24 - 1) * per_block
    for s in [0, 1, seam - 1, seam, seam + 1, count - 2, count - 1]:
        o = oracle.init_stream(gen, 0, 3 * s)
        ref = oracle.generate(gen, o, n, P.U32)
        assert np.array_equal(out[s * n:(s + 1) * n].cpu().numpy().view(np.uint32), ref), s
        assert np.array_equal(st[s * sb:(s + 1) * sb].cpu().numpy(), o), s
