"""MRG32K3A/LFSR113 many-stream outputs at addresses off the 128-byte chunks
in which a run is stored: output pointers at every kind of offset, lengths
around a chunk and a section, nothing written outside the output; values and
final states against the oracle."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

NPDT = {P.U32: np.uint32, P.F32: np.float32, P.F64: np.float64}
GUARD = 64


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("count,n", [(1, 1), (3, 31), (2, 33), (65, 5), (5, 255), (4, 257), (3, 999), (2, 4999), (1, 20003),
                                     (300, 60), (107, 123), (64, 128), (33, 820), (9, 2080), (129, 513)])
@pytest.mark.parametrize("dtype", [P.U32, P.F32, P.F64])
@pytest.mark.parametrize("gen", [P.MRG32K3A, P.LFSR113])
def test_any_address(ctx, oracle, gen, dtype, count, n):
    es = 8 if dtype == P.F64 else 4
    start = [oracle.seed(gen, 1000 + 77 * i) for i in range(count)]
    ref, end = [], []
    for st in start:
        s = st.copy()
        ref.append(oracle.generate(gen, s, n, dtype))
        end.append(s)
    for offset in (0, 1, 3, 13, 31):
        d = torch.from_numpy(np.concatenate(start)).cuda()
        buf = torch.full(((count * n + 2 * GUARD) * es,), 0xA5, dtype=torch.uint8, device="cuda")
        at = (GUARD + offset) * es
        ctx.generate_streams(gen, d, count, n, dtype, buf.data_ptr() + at)
        torch.cuda.synchronize()
        raw = buf.cpu().numpy()
        got = raw[at:at + count * n * es].view(NPDT[dtype]).reshape(count, n)
        for i in range(count):
            np.testing.assert_array_equal(got[i], ref[i], err_msg=f"stream {i} offset {offset}")
        assert (raw[:at] == 0xA5).all() and (raw[at + count * n * es:] == 0xA5).all()
        assert np.array_equal(d.cpu().numpy(), np.concatenate(end))
