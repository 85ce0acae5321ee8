"""Host arrays filled by several threads of one context: a short call does not
wait for the end of a long one, and all of them continue their own states."""
import threading
import time

import numpy as np
import pytest
import torch  # noqa: F401 (its HIP runtime, before the library loads one)

from paper_1307_5869_amd import prand as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    c.close()


def test_short_calls_beside_a_long_one(ctx):
    a, b = ctx.seed(P.MRG32K3A, 1), ctx.seed(P.LFSR113, 1000)
    ctx.generate_array(P.MRG32K3A, a, P.F64, 1 << 20)
    ctx.generate_array(P.LFSR113, b, P.U32, 1000)
    span, short, stop = [], [], threading.Event()

    def long_call():
        t = time.perf_counter()
        ctx.generate_array(P.MRG32K3A, a, P.F64, 1 << 28)   # 2 GB
        span.extend([t, time.perf_counter()])
        stop.set()

    def short_calls():
        while not stop.is_set():
            t = time.perf_counter()
            ctx.generate_array(P.LFSR113, b, P.U32, 1000)
            short.append((t, time.perf_counter()))

    threads = [threading.Thread(target=f) for f in (short_calls, long_call)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    inside = [1 for s, e in short if s >= span[0] and e <= span[1]]
    # while calls excluded one another, at most the one that came first
    assert len(inside) >= 10


def test_many_threads(ctx, oracle):
    """more calls at once than buffers are kept, of several sizes"""
    jobs = [(g, dt, n) for k, n in enumerate([1000, 70000, 300001, 9000001]) for g, dt in
            [(P.MRG32K3A, P.F64), (P.LFSR113, P.U32), (P.GM29 + k % 2, P.F32)]]
    got = {}

    def run(j, job):
        g, dt, n = job
        st = ctx.seed(g, 500 + j)
        got[j] = [ctx.generate_array(g, st, dt, m) for m in (n, 777)], st

    threads = [threading.Thread(target=run, args=(j, job)) for j, job in enumerate(jobs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for j, (g, dt, n) in enumerate(jobs):
        (first, second), st = got[j]
        o = ctx.seed(g, 500 + j)
        if n <= 300001:
            np.testing.assert_array_equal(first, oracle.generate(g, o, n, dt))
        else:
            np.testing.assert_array_equal(first, ctx.generate_array(g, o, dt, n))
        np.testing.assert_array_equal(second, oracle.generate(g, o, 777, dt))
        np.testing.assert_array_equal(st, o)
