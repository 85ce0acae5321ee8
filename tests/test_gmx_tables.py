"""The coefficient tables of the GM/GQ matrix-instruction kernels, on the CPU:
the digits of every step represent the step's coefficients mod p, lose less
than the result's offset allows (the bound that makes every digit exact), keep
the sums within the 22 bits that the accumulators hold exactly, and the
kernels' arithmetic, emulated in integers on states whose later values sit at
the digit boundaries, gives the exact digits."""
import ctypes
import random

import numpy as np
import pytest

from paper_1307_5869_amd import prand as P

# (k, q, e, c, v) with p = 2^e - c, table order
GENS = [(15, 28, 19, 1, 1), (4, 2, 29, 3, 1), (11, 14, 31, 1, 1), (256, 176, 51, 129, 4), (24, 74, 61, 1, 1),
        (8, 48, 29, 3, 1), (8, 48, 29, 3, 3), (8, 48, 29, 3, 4)]
NAMES = ["GM19", "GM29", "GM31", "GM55", "GM61", "GQ58.1", "GQ58.3", "GQ58.4"]


@pytest.fixture(scope="module")
def tables():
    fn = P.load().prand_internal_gmx_table
    res = []
    for g in range(8):
        mat = np.zeros((257, 4), dtype=np.uint64)
        dig = np.zeros((256, 2, 8), dtype=np.int16)
        dims = (ctypes.c_int * 7)()
        assert fn(g, ctypes.c_void_p(mat.ctypes.data), ctypes.c_void_p(dig.ctypes.data), dims) == 0
        assert dims[0] == 256
        res.append((mat, dig, *dims[1:]))
    return res


@pytest.mark.parametrize("g", range(8), ids=NAMES)
def test_digits_represent_the_steps_and_keep_the_bound(tables, g):
    k, q, e, c, v = GENS[g]
    p = 2**e - c
    mat, dig, D, L, bits, delta, b, top = tables[g]
    tb = bits * (L - 1) + (bits if top else 8)
    row, prev = (1, 0), (0, 1)
    for j in range(257):
        assert tuple(int(x) for x in mat[j]) == row + prev
        if j:
            lost = gained = low = high = 0
            for h in range(2):
                d = [int(x) for x in dig[j - 1, h]]
                assert all(-2**(b - 1) <= x < 2**(b - 1) for x in d) and not any(d[D:])
                assert (sum(x * 2**(b * m) for m, x in enumerate(d)) - row[h]) % p == 0
                low -= sum(x for x in d if x < 0)
                high += sum(x for x in d if x > 0)
                # a fraction cut i digits above the last loses [0, 1) and
                # 2^(-b i) more for the rounding of x / p (itself a little
                # over one unit)
                w = [1 + 1.01 * 2.0 ** (-b * (D - 1 - m)) for m in range(D)]
                lost += sum(x * w[m] for m, x in enumerate(d[:D]) if x > 0)
                gained -= sum(x * w[m] for m, x in enumerate(d[:D]) if x < 0)
            assert lost <= delta
            assert delta + gained < 2**tb / (p * 2**v)
            # a position's sum with the carry into it (a sum over 2^10 or 2^11)
            assert (1 + top) * max(low, high) * (2**bits - 1) + 2**13 < 2**22
        row, prev = tuple((k * a - q * b) % p for a, b in zip(row, prev)), row


WF = [43, 65, 69, 114, 130, 65, 69, 69]


def fraction(g, x):
    """The kernels' form of floor(2^WF x / p), WF = TB + b (D - 1)."""
    if g == 0:
        return (x << 24) | (x << 5) | (x >> 14)
    if g == 2:
        return (x << 38) | (x << 7) | (x >> 24)
    if g == 3:
        return (x << 63) + ((129 * x) << 12) + ((16641 * x) >> 39)
    if g == 4:
        return (x << 69) | (x << 8) | (x >> 53)
    sh = WF[g] - 29
    return (x << sh) + ((3 * x) << (sh - 29)) + ((9 * x) >> (58 - sh))


def kernel_digit(g, dig, D, L, bits, delta, b, top, v, j, xc, xp):
    """The accumulator chain of one step of one element."""
    acc = delta
    f = (fraction(g, xc), fraction(g, xp))
    for s in range(L):
        double = top and s == L - 1
        if s:
            acc >>= bits - double
        for h in range(2):
            for m in range(D):
                acc += int(dig[j - 1, h, m]) * (((f[h] >> (bits * s + b * (D - 1 - m))) & (2**bits - 1)) << double)
        assert -2**22 <= acc < 2**22
    return (acc >> (bits + top if top else 8) - v) & (2**v - 1)


@pytest.mark.parametrize("g", range(8), ids=NAMES)
def test_fraction_error(g):
    _, _, e, c, _ = GENS[g]
    p = 2**e - c
    wf = WF[g]
    r = random.Random(7 + g)
    for x in [0, 1, 2, p - 1, p - 2, p // 2, p // 2 + 1] + [r.randrange(p) for _ in range(3000)]:
        err = (x << wf) - fraction(g, x) * p     # in [0, 1.01) units of 2^-WF x p
        assert 0 <= err < 1.01 * p


@pytest.mark.parametrize("g", range(8), ids=NAMES)
def test_digits_at_the_boundaries(tables, g):
    k, q, e, c, v = GENS[g]
    p = 2**e - c
    mat, dig, D, L, bits, delta, bd, top = tables[g]
    assert bits * (L - 1) + (bits if top else 8) + bd * (D - 1) == WF[g]
    r = random.Random(11 + g)
    edges = []
    for i in range(2**v + 1):
        b = -(-i * p // 2**v)        # the least value with digit i
        edges += [x % p for x in (b - 2, b - 1, b, b + 1)]
    for j in list(range(1, 9)) + [31, 32, 33, 64, 100, 200, 255, 256]:
        a, b, cc, d = (int(x) for x in mat[j])
        inv = pow(a * d - b * cc, -1, p)
        for target in edges if j in (1, 32, 255, 256) else r.sample(edges, min(len(edges), 8)):
            # (xc, xp) whose step j is `target`
            o = r.randrange(p)
            xc, xp = (d * target - b * o) * inv % p, (a * o - cc * target) * inv % p
            assert (a * xc + b * xp) % p == target
            assert kernel_digit(g, dig, D, L, bits, delta, bd, top, v, j, xc, xp) == (target << v) // p
    for _ in range(300):
        xc, xp, j = r.randrange(p), r.randrange(p), r.randrange(1, 257)
        a, b = int(mat[j][0]), int(mat[j][1])
        assert kernel_digit(g, dig, D, L, bits, delta, bd, top, v, j, xc, xp) == ((a * xc + b * xp) % p << v) // p
