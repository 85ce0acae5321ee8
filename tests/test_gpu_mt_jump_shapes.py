"""MT19937 jumps in launches of more than 4096 streams (four wavefronts per
stream) against the same streams jumped in smaller launches (eight and
sixteen), by block splitting and by per-stream distances, and sampled streams
against the oracle."""
import numpy as np
import torch
import pytest

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu


def test_launch_shapes_agree(oracle):
    ctx = P.Context(0)
    sb = P.state_bytes(P.MT19937)
    r = np.random.default_rng(5)
    total = 4097
    ids = r.integers(0, 10**19, size=total, dtype=np.uint64)
    ids[:4] = [0, 1, 1 << 48, (1 << 63) + 5]
    dist = r.integers(0, 1 << 62, size=total, dtype=np.uint64)
    dist[:3] = [0, 1, 624]
    t_ids = torch.from_numpy(ids.view(np.int64)).cuda()
    t_dist = torch.from_numpy(dist.view(np.int64)).cuda()
    split, moved = {}, {}
    for count in (512, 513, 4096, total):
        st = torch.empty(count * sb, dtype=torch.uint8, device="cuda")
        ctx.init_streams_dev(P.MT19937, P.SEQ_DEFAULT, None, t_ids, count, st)
        split[count] = st.cpu().numpy().copy()
        if count in (513, total):
            ctx.skipahead_dev(P.MT19937, st, count, t_dist, 1, True)
            moved[count] = st.cpu().numpy()
    for count in (512, 513, 4096):
        assert np.array_equal(split[count], split[total][:count * sb])
    assert np.array_equal(moved[513], moved[total][:513 * sb])
    for i in [0, 1, 2, 3, 511, 4096]:
        st = oracle.init_stream(P.MT19937, 0, int(ids[i]))
        assert np.array_equal(split[total][i * sb:(i + 1) * sb], st), i
        oracle.skipahead(P.MT19937, st, int(dist[i]))
        assert np.array_equal(moved[total][i * sb:(i + 1) * sb], st), i
    ctx.close()
