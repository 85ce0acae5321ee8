"""GM/GQ generation by matrix instructions against the oracle where it can go
wrong: lengths around the 32-, 64- and 256-step blocks and the cut into
sections, stream counts around the wavefront's share, states that have not
collapsed, states whose values reach the digit boundaries at every step of a
block, and every dtype; outputs and final states."""
import numpy as np
import pytest
import torch

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu

TDT = {P.U32: torch.int32, P.F32: torch.float32, P.F64: torch.float64}
NPDT = {P.U32: np.uint32, P.F32: np.float32, P.F64: np.float64}
GENS = list(range(P.GM19, P.GQ58X4 + 1))
# (k, q, e, c, v, s, t): modulus (2^e - c) 2^t
PARAMS = {P.GM19: (15, 28, 19, 1, 1, 32, 0), P.GM29: (4, 2, 29, 3, 1, 32, 0), P.GM31: (11, 14, 31, 1, 1, 32, 0),
          P.GM55: (256, 176, 51, 129, 4, 8, 4), P.GM61: (24, 74, 61, 1, 1, 32, 0),
          P.GQ58X1: (8, 48, 29, 3, 1, 32, 29), P.GQ58X3: (8, 48, 29, 3, 3, 12, 29), P.GQ58X4: (8, 48, 29, 3, 4, 8, 29)}


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


def check(ctx, oracle, gen, states, n, dtype):
    count = len(states)
    d = torch.from_numpy(np.concatenate(states)).cuda()
    out = torch.empty(count * n, dtype=TDT[dtype], device="cuda")
    ctx.generate_streams(gen, d, count, n, dtype, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(NPDT[dtype]).reshape(count, n)
    got_st = d.cpu().numpy().reshape(count, -1)
    for i, st in enumerate(states):
        ref = oracle.generate(gen, st, n, dtype)
        np.testing.assert_array_equal(got[i], ref, err_msg=f"{P.NAMES[gen]} stream {i} of {count}, n {n}")
        assert np.array_equal(got_st[i], st), f"{P.NAMES[gen]} state {i} of {count}, n {n}"


@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 127, 128, 255, 256, 257, 511, 513, 767, 768, 863, 864, 1025, 2881, 4607, 4608, 5000,
                               9216, 20011])
@pytest.mark.parametrize("gen", GENS)
def test_lengths(ctx, oracle, gen, n):
    count = 5 if n < 1000 else 2
    fresh = [oracle.seed(gen, 50 + i) for i in range(count)]
    moved = [oracle.init_stream(gen, 0, 10**17 + 3 * i) for i in range(count)]
    for st in moved:
        oracle.generate(gen, st, 5)      # GQ58.3: inside a block
    for dtype in (P.U32, P.F32, P.F64) if n in (33, 4608, 5000) else (P.U32,):
        check(ctx, oracle, gen, [s.copy() for s in fresh], n, dtype)
        check(ctx, oracle, gen, [s.copy() for s in moved], n, dtype)


@pytest.mark.parametrize("count", [1, 2, 3, 4, 7, 9, 33])
@pytest.mark.parametrize("gen", GENS)
def test_counts(ctx, oracle, gen, count):
    # one state that has not collapsed among collapsed ones
    states = [oracle.init_stream(gen, 0, 7 * i + 1) for i in range(count)]
    states[count // 2] = oracle.seed(gen, 99)
    check(ctx, oracle, gen, states, 300, P.U32)


@pytest.mark.parametrize("gen", GENS)
def test_digit_boundaries(ctx, oracle, gen):
    """Element e of stream i takes a value at a digit boundary at step j(e, i)."""
    k, q, e, c, v, s, t = PARAMS[gen]
    p = 2**e - c
    edges = [x % p for b in range(2**v + 1) for x in range(-(-b * p // 2**v) - 2, -(-b * p // 2**v) + 2)]
    rows = [((1, 0), (0, 1))]
    for _ in range(256):
        (a, b), prev = rows[-1]
        rows.append((((k * a - q * prev[0]) % p, (k * b - q * prev[1]) % p), (a, b)))
    r = np.random.default_rng(gen)
    states = []
    for i in range(64):
        st = oracle.init_stream(gen, 0, i)
        w = st.view(np.uint64)
        for el in range(s):
            j = 1 + (el + 4 * s * i + 5 * i) % 256
            (a, b), (cc, d) = rows[j]
            target, other = edges[(el + i) % len(edges)], int(r.integers(p))
            inv = pow(a * d - b * cc, -1, p)
            w[32 + el] = (d * target - b * other) * inv % p << t
            w[el] = (a * other - cc * target) * inv % p << t
        states.append(st)
    check(ctx, oracle, gen, [s_.copy() for s_ in states], 290, P.U32)
    if gen in (P.GM19, P.GM61):   # the matrix form of these: streams cut into sections
        check(ctx, oracle, gen, [s_.copy() for s_ in states[:8]], 4700, P.U32)
