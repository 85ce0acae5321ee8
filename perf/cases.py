"""Performance cases: what programs that use this library have it do, through
the public entry points of ``paper_1307_5869_amd.prand``.

A case is a dict of plain values.  Its ``kind`` names the call pattern:

  step     every generator in turn: block-splitting start of `count` streams,
           then n words of each (the library's benchmark step)
  streams  one generator: `count` streams of n numbers each, started by block
           splitting in the pass itself (init) or by the program beforehand
  skip     `count` states moved 2^k outputs ahead, k drawn per stream over the
           range that the generator's stream table supports
  spaced   `count` MRG32K3A streams k * 2^76 apart: skip-ahead, then n words
           and n float64 numbers of each
  single   one host state continued by n numbers into device memory
  array    one host state continued by n numbers into host memory
  batch    a planned batched launch: `count` tasks of mixed generators and
           lengths log-uniform in [lo, hi], replayed
  serve    the serving loop: `count` requests of mixed generators, dtypes and
           lengths log-uniform in [lo, hi], submitted at once, their outputs
           copied into the program's own buffers as they complete
"""
import math

import numpy as np
import torch

from paper_1307_5869_amd import prand as P
from paper_1307_5869_amd import workloads as W

DEV = "cuda:0"
TORCH_DT = {P.U32: torch.int32, P.F32: torch.float32, P.F64: torch.float64}
SIZE = {P.U32: 4, P.F32: 4, P.F64: 8}
ID_BOUND = W.ID_BOUND

# ensemble elements, and element steps per 32-bit word, of the GM/GQ generators
ELEMENTS = {P.GM19: 32, P.GM29: 32, P.GM31: 32, P.GM55: 8, P.GM61: 32, P.GQ58X1: 32, P.GQ58X3: 12, P.GQ58X4: 8}

_ctx = None


def context():
    """The library context a program creates once and keeps."""
    global _ctx
    if _ctx is None:
        _ctx = P.Context(0)
    return _ctx


def listed():
    return [
        # The benchmark step of bench.py: all eleven generators, 65536
        # block-split streams of 16384 words each.
        {"name": "step-65536x16384", "kind": "step", "count": 65536, "n": 16384},
        # A simulation on a thousand Mersenne-twister streams in double
        # precision: stream starts and one refill of 100000 numbers each.
        {"name": "mt19937-start-1000x100000", "kind": "streams", "gen": P.MT19937, "count": 1000, "n": 100000,
         "dtype": P.F64, "init": True},
        # 4096 MRG32K3A streams at a spacing of 2^76, the usual substream
        # length of this generator: words and doubles.
        {"name": "mrg32k3a-spaced-4096x4096", "kind": "spaced", "gen": P.MRG32K3A, "count": 4096, "n": 4096},
        # Odd sizes: rows that end off every alignment.
        {"name": "lfsr113-odd-10007x4999", "kind": "streams", "gen": P.LFSR113, "count": 10007, "n": 4999,
         "dtype": P.F32, "init": False},
        # A medium number of long streams of a torus-map ensemble, refilled.
        {"name": "gm29-1000x100003", "kind": "streams", "gen": P.GM29, "count": 1000, "n": 100003, "dtype": P.F32,
         "init": False},
        # Many short refills in double precision.
        {"name": "gq58.3-65536x1000", "kind": "streams", "gen": P.GQ58X3, "count": 65536, "n": 1000, "dtype": P.F64,
         "init": False},
        # 2^20 stream states placed by skip-ahead.
        {"name": "gm55-skip-1048576", "kind": "skip", "gen": P.GM55, "count": 1 << 20},
        # The smallest call: a program that draws a thousand numbers from its
        # one state at a time.
        {"name": "mrg32k3a-single-1000", "kind": "single", "gen": P.MRG32K3A, "n": 1000, "dtype": P.F64},
        # One long stream filled by sections.
        {"name": "gm61-single-100000000", "kind": "single", "gen": P.GM61, "n": 100000000, "dtype": P.F32},
        # Numbers wanted in host memory.
        {"name": "lfsr113-array-1000000", "kind": "array", "gen": P.LFSR113, "n": 1000000, "dtype": P.F64},
        # A tenth of the benchmark's batched workload.
        {"name": "batch-2000", "kind": "batch", "count": 2000, "lo": 1000, "hi": 10000000, "dtype": P.F32},
        # A burst of requests to the serving loop.
        {"name": "serve-128", "kind": "serve", "count": 128, "lo": 1000, "hi": 1000000},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["streams"] * 6 + ["single"] * 3 + ["skip"] * 2 + ["spaced", "array", "batch", "serve"])
    gen = rng.randrange(P.NUM_GENERATORS)
    dtype = rng.randrange(3)
    if kind == "streams":
        count = _log_uniform(rng, 1, 65536)
        n = _log_uniform(rng, 100, max(101, min(1 << 20, (1 << 29) // count)))
        # one stream of MT19937 is one chain: its longest rows stay short
        if gen == P.MT19937 and count < 256:
            n = min(n, 100000)
        return {"kind": kind, "gen": gen, "count": count, "n": n, "dtype": dtype, "init": rng.random() < 0.5}
    if kind == "single":
        return {"kind": kind, "gen": gen, "n": _log_uniform(rng, 1, 100000000), "dtype": dtype}
    if kind == "skip":
        return {"kind": kind, "gen": gen, "count": _log_uniform(rng, 1, 1 << 16 if gen == P.MT19937 else 1 << 20)}
    if kind == "spaced":
        return {"kind": kind, "gen": P.MRG32K3A, "count": _log_uniform(rng, 64, 8192),
                "n": _log_uniform(rng, 64, 8192)}
    if kind == "array":
        return {"kind": kind, "gen": gen, "n": _log_uniform(rng, 1000, 10000000), "dtype": dtype}
    if kind == "batch":
        return {"kind": kind, "count": _log_uniform(rng, 20, 2000), "lo": 1000, "hi": 10000000, "dtype": dtype}
    return {"kind": kind, "count": _log_uniform(rng, 16, 256), "lo": 1000, "hi": 1000000}


# ------------------------------------------------------------------- inputs
def _ids(r, count):
    return torch.from_numpy(r.integers(0, ID_BOUND, size=count, dtype=np.uint64).view(np.int64)).to(DEV)


def _started(ctx, gen, r, count):
    st = torch.empty(count * P.state_bytes(gen), dtype=torch.uint8, device=DEV)
    ctx.init_streams_dev(gen, P.SEQ_DEFAULT, None, _ids(r, count), count, st)
    return st


def _mixed(case):
    """Generators, lengths and dtypes of a batch or a burst of requests: the
    shape of the workload, which belongs to the case; its stream ids are the
    seed's."""
    c = case["count"]
    r = np.random.default_rng([c, case["lo"], case["hi"]])
    gens = r.integers(0, P.NUM_GENERATORS, size=c)
    lens = np.rint(np.exp(r.uniform(np.log(case["lo"]), np.log(case["hi"]), size=c))).astype(np.int64)
    return gens, lens, r.integers(0, 3, size=c)


def _state_seed(seed):
    """The seed of a host state: below MRG32K3A's moduli, above LFSR113's
    least seed, different in its upper bits from one seed to the next."""
    return int(np.random.default_rng(seed).integers(1 << 10, 1 << 31))


def prepare(case, seed):
    ctx = context()
    r = np.random.default_rng(seed)
    kind = case["kind"]
    s = {"case": case, "ctx": ctx}
    if kind == "step":
        c, n = case["count"], case["n"]
        # the MT19937 jump tables, built once per program
        _started(ctx, P.MT19937, r, 1)
        s["ids"] = [_ids(r, c) for _ in range(P.NUM_GENERATORS)]
        s["states"] = [torch.empty(c * P.state_bytes(g), dtype=torch.uint8, device=DEV)
                       for g in range(P.NUM_GENERATORS)]
        s["out"] = [torch.empty(c * n, dtype=torch.int32, device=DEV) for _ in range(P.NUM_GENERATORS)]
    elif kind == "streams":
        g, c = case["gen"], case["count"]
        s["states"] = _started(ctx, g, r, c)
        s["ids"] = _ids(r, c) if case["init"] else None
        s["out"] = torch.empty(c * case["n"], dtype=TORCH_DT[case["dtype"]], device=DEV)
    elif kind == "skip":
        g, c = case["gen"], case["count"]
        s["states"] = _started(ctx, g, r, c)
        lo, hi = W.JUMP_EXP_RANGE[g]
        k = r.integers(lo, hi + 1, size=c)
        limbs = np.zeros((c, P.MAX_LIMBS), dtype=np.uint64)
        limbs[np.arange(c), k // 64] = np.left_shift(np.uint64(1), (k % 64).astype(np.uint64))
        s["dist"] = torch.from_numpy(limbs.reshape(-1).view(np.int64)).to(DEV)
    elif kind == "spaced":
        c, n = case["count"], case["n"]
        base = ctx.seed(case["gen"], _state_seed(seed))
        s["base"] = torch.from_numpy(np.tile(base, c)).to(DEV)
        limbs = np.stack([P.limbs(k << 76) for k in range(c)])
        s["dist"] = torch.from_numpy(limbs.reshape(-1).view(np.int64)).to(DEV)
        s["a"], s["b"] = torch.empty_like(s["base"]), torch.empty_like(s["base"])
        s["words"] = torch.empty(c * n, dtype=torch.int32, device=DEV)
        s["reals"] = torch.empty(c * n, dtype=torch.float64, device=DEV)
    elif kind == "single":
        s["state"] = ctx.seed(case["gen"], _state_seed(seed))
        if case["gen"] == P.MT19937:
            _started(ctx, P.MT19937, r, 1)
        s["out"] = torch.empty(case["n"], dtype=TORCH_DT[case["dtype"]], device=DEV)
    elif kind == "array":
        s["state"] = ctx.seed(case["gen"], _state_seed(seed))
        if case["gen"] == P.MT19937:
            _started(ctx, P.MT19937, r, 1)
    elif kind == "batch":
        gens, lens, _ = _mixed(case)
        dt = case["dtype"]
        s["out"] = torch.empty(int(lens.sum()), dtype=TORCH_DT[dt], device=DEV)
        sb = [P.state_bytes(g) for g in range(P.NUM_GENERATORS)]
        s["in"], s["states"], place = {}, {}, {}
        for g in sorted(set(gens.tolist())):
            sel = np.nonzero(gens == g)[0]
            s["in"][g] = _started(ctx, g, r, len(sel))
            s["states"][g] = torch.empty_like(s["in"][g])
            place[g] = {int(k): j for j, k in enumerate(sel)}
        off = np.concatenate([[0], np.cumsum(lens)[:-1]])
        tasks = []
        for k, (g, n) in enumerate(zip(gens.tolist(), lens.tolist())):
            at = place[g][k] * sb[g]
            tasks.append((g, dt, n, s["in"][g].data_ptr() + at, s["states"][g].data_ptr() + at,
                          s["out"].data_ptr() + SIZE[dt] * int(off[k])))
        torch.cuda.synchronize()
        s["batch"] = P.Batch(ctx, tasks, P.BatchConfig(use_graph=1))
    elif kind == "serve":
        gens, lens, dts = _mixed(case)
        ids = r.integers(0, ID_BOUND, size=len(gens), dtype=np.uint64)
        s["out"] = {d: torch.empty(int(lens[dts == d].sum()), dtype=TORCH_DT[d], device=DEV) for d in TORCH_DT}
        used = {d: 0 for d in TORCH_DT}
        s["requests"] = []
        for g, i, n, d in zip(gens.tolist(), ids.tolist(), lens.tolist(), dts.tolist()):
            s["requests"].append((g, i, n, d, s["out"][d][used[d]:used[d] + n]))
            used[d] += n
        _started(ctx, P.MT19937, r, 1)
        s["server"] = P.Server(ctx, P.ServerConfig(hbm_budget=2 << 30))
    else:
        raise ValueError(kind)
    torch.cuda.synchronize()
    return s


class _DeviceArray:
    """Device memory that the serving loop owns, for torch to read."""

    def __init__(self, ptr, n, dtype):
        typestr = {P.U32: "<i4", P.F32: "<f4", P.F64: "<f8"}[dtype]
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": typestr, "data": (ptr, False), "version": 2}


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "step":
        c, n = case["count"], case["n"]
        for g in range(P.NUM_GENERATORS):
            ctx.init_streams_dev(g, P.SEQ_DEFAULT, None, s["ids"][g], c, s["states"][g])
            ctx.generate_streams(g, s["states"][g], c, n, P.U32, s["out"][g])
        return {"out": s["out"], "states": s["states"]}
    if kind == "streams":
        g, c = case["gen"], case["count"]
        if case["init"]:
            ctx.init_streams_dev(g, P.SEQ_DEFAULT, None, s["ids"], c, s["states"])
        ctx.generate_streams(g, s["states"], c, case["n"], case["dtype"], s["out"])
        return {"out": s["out"], "states": s["states"]}
    if kind == "skip":
        ctx.skipahead_dev(case["gen"], s["states"], case["count"], s["dist"], P.MAX_LIMBS, True)
        return s["states"]
    if kind == "spaced":
        g, c, n = case["gen"], case["count"], case["n"]
        s["a"].copy_(s["base"])
        ctx.skipahead_dev(g, s["a"], c, s["dist"], P.MAX_LIMBS, True)
        s["b"].copy_(s["a"])
        ctx.generate_streams(g, s["a"], c, n, P.U32, s["words"])
        ctx.generate_streams(g, s["b"], c, n, P.F64, s["reals"])
        return {"words": s["words"], "reals": s["reals"], "states": s["a"]}
    if kind == "single":
        ctx.generate(case["gen"], s["state"], case["dtype"], s["out"], case["n"])
        return {"out": s["out"], "state": s["state"]}
    if kind == "array":
        return {"out": ctx.generate_array(case["gen"], s["state"], case["dtype"], case["n"]), "state": s["state"]}
    if kind == "batch":
        s["batch"].launch()
        return {"out": s["out"], "states": s["states"]}
    srv = s["server"]
    for k, (g, i, n, d, _) in enumerate(s["requests"]):
        srv.submit(g, i, n, d, tag=k)
    done = 0
    held = []
    while done < len(s["requests"]):
        for c in srv.poll(wait_ms=50):
            s["requests"][c.tag][4].copy_(torch.as_tensor(_DeviceArray(c.out, c.n, c.dtype), device=DEV))
            held.append(c.ticket)
            done += 1
    # the copies have to be over before the loop may reuse the memory
    torch.cuda.current_stream().synchronize()
    for t in held:
        srv.release(t)
    return s["out"]


# --------------------------------------------------------------------- work
def _steps(gen, n):
    """Operations of n outputs: the recurrence itself, without packing."""
    if gen == P.MT19937:
        return 8 * n          # twist and tempering of a word
    if gen == P.MRG32K3A:
        return 9 * n          # four products, three sums, two reductions
    if gen == P.LFSR113:
        return 23 * n         # four components of five operations, three sums
    words = 1.0 if gen != P.GQ58X3 else 8.0 / 9.0
    return 4 * ELEMENTS[gen] * words * n   # two products, a difference, a reduction per element


def _start_ops(gen, count):
    """Operations of `count` block-splitting starts: one dense jump each."""
    if gen == P.MT19937:
        return count * 9968.0 * 624
    if gen == P.MRG32K3A:
        return count * 36.0
    if gen == P.LFSR113:
        return count * 256.0
    return count * 8.0 * ELEMENTS[gen]


def work(case):
    kind = case["kind"]
    sb = [P.state_bytes(g) for g in range(P.NUM_GENERATORS)]
    if kind == "step":
        c, n = case["count"], case["n"]
        gens = range(P.NUM_GENERATORS)
        return {"bytes": sum(c * (n * 4 + sb[g] + 8) for g in gens),
                "flops": sum(_steps(g, c * n) + _start_ops(g, c) for g in gens)}
    if kind == "streams":
        g, c, n = case["gen"], case["count"], case["n"]
        return {"bytes": c * (n * SIZE[case["dtype"]] + sb[g] + (8 if case["init"] else sb[g])),
                "flops": _steps(g, c * n) + (_start_ops(g, c) if case["init"] else 0)}
    if kind == "skip":
        g, c = case["gen"], case["count"]
        return {"bytes": c * (2 * sb[g] + 64), "flops": _start_ops(g, c)}
    if kind == "spaced":
        g, c, n = case["gen"], case["count"], case["n"]
        return {"bytes": c * (n * 12 + 64 + 3 * sb[g]), "flops": 2 * _steps(g, c * n) + _start_ops(g, c)}
    if kind in ("single", "array"):
        return {"bytes": case["n"] * SIZE[case["dtype"]] + 2 * sb[case["gen"]], "flops": _steps(case["gen"], case["n"])}
    # lengths log-uniform in [lo, hi], generators uniform
    mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
    numbers = case["count"] * mean
    ops = sum(_steps(g, numbers / P.NUM_GENERATORS) for g in range(P.NUM_GENERATORS))
    if kind == "batch":
        return {"bytes": numbers * SIZE[case["dtype"]], "flops": ops}
    ops += sum(_start_ops(g, case["count"] / P.NUM_GENERATORS) for g in range(P.NUM_GENERATORS))
    return {"bytes": numbers * 16.0 / 3 * 2, "flops": ops}


# -------------------------------------------------------------------- exact
M1, M2 = 4294967087, 4294944443
A1 = [[0, 1403580, M1 - 810728], [1, 0, 0], [0, 1, 0]]
A2 = [[527612, 0, M2 - 1370589], [1, 0, 0], [0, 1, 0]]


def _matmul(a, b, m):
    return [[sum(a[i][k] * b[k][j] for k in range(3)) % m for j in range(3)] for i in range(3)]


def _matpow(a, e, m):
    r = [[int(i == j) for j in range(3)] for i in range(3)]
    while e:
        if e & 1:
            r = _matmul(r, a, m)
        a = _matmul(a, a, m)
        e >>= 1
    return r


def _mrg_lanes(x, y, spacing, lanes):
    """States x, y (newest value first) of `lanes` streams, `spacing` apart."""
    j1, j2 = _matpow(A1, spacing, M1), _matpow(A2, spacing, M2)
    xs, ys = [], []
    for _ in range(lanes):
        xs.append(x)
        ys.append(y)
        x = [sum(j1[i][k] * x[k] for k in range(3)) % M1 for i in range(3)]
        y = [sum(j2[i][k] * y[k] for k in range(3)) % M2 for i in range(3)]
    return np.array(xs, dtype=np.int64).T.copy(), np.array(ys, dtype=np.int64).T.copy()


def _mrg_reals(x, y, n):
    """[lane][i]: z / (m1 + 1) of n steps of every lane, z in [1, m1]."""
    x, y = [v for v in x], [v for v in y]
    out = np.empty((n, x[0].size), dtype=np.float64)
    for i in range(n):
        nx = (1403580 * x[1] - 810728 * x[2]) % M1
        ny = (527612 * y[0] - 1370589 * y[2]) % M2
        x, y = [nx, x[0], x[1]], [ny, y[0], y[1]]
        z = (nx - ny) % M1
        out[i] = np.where(z == 0, M1, z) / float(M1 + 1)
    return out.T.copy()


def exact(case, seed):
    """The float64 numbers of the MRG32K3A cases and of one MT19937 state, in
    64 bits from the generators' definitions; None elsewhere."""
    kind, gen = case["kind"], case.get("gen")
    if kind == "spaced":
        c, n = case["count"], case["n"]
        s = [_state_seed(seed)] * 3
        x, y = _mrg_lanes(s, s, 1 << 76, c)
        return {"words": None, "reals": _mrg_reals(x, y, n).reshape(-1), "states": None}
    if kind not in ("single", "array") or case["n"] > 1 << 23:
        return None
    n = case["n"]
    if gen == P.MRG32K3A and case["dtype"] == P.F64:
        lanes = min(n, 2048)
        per = -(-n // lanes)
        s = [_state_seed(seed)] * 3
        x, y = _mrg_lanes(s, s, per, lanes)
        return {"out": _mrg_reals(x, y, per).reshape(-1)[:n], "state": None}
    if gen == P.MT19937 and case["dtype"] != P.U32:
        w = np.random.RandomState(_state_seed(seed))._bit_generator.random_raw(n).astype(np.uint64)
        return {"out": w * 2.0 ** -32 if case["dtype"] == P.F64 else (w >> np.uint64(8)) * 2.0 ** -24, "state": None}
    return None
