"""The ranges of streams in which launches go out: they follow one another,
cover every stream, and none is a dispatch of 2^32 work-items or more (the
hardware's count of them)."""
import ctypes

import pytest

from paper_1307_5869_amd import prand as P


@pytest.mark.parametrize("block,per_block", [
    (64, 1),       # MT19937 generation, a wavefront per stream
    (256, 1),      # MT19937 jumps by four wavefronts, MT19937 tiles
    (512, 1),      # by eight; MT19937 section starts of a batch
    (1024, 1),     # by sixteen
    (256, 4),      # v = 1 GM/GQ generation: a wavefront per stream
    (256, 8),      # GQ58.3 generation; v = 1 ballots; v = 1 jumps
    (256, 16),     # GM55, GQ58.4 generation; GQ58.3 jumps
    (256, 32),     # GM55, GQ58.4 jumps
    (256, 256),    # MRG32K3A, LFSR113, seeds: a lane per stream
])
def test_ranges_cover_and_fit(block, per_block):
    fn = P.load().prand_internal_launch_ranges
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_int]
    most = (2**32 - 1) // block * per_block
    for count in [0, 1, per_block, per_block + 1, most - 1, most, most + 1, 2 * most, 2 * most + 1, 2**26 + 3, 2**32 - 1]:
        buf = (ctypes.c_uint64 * (3 * 2048))()
        k = fn(count, block, per_block, buf, 2048)
        assert k == -(-count // most) <= 2048
        at = 0
        for i in range(k):
            first, m, blocks = buf[3 * i:3 * i + 3]
            assert first == at and m > 0
            assert (blocks - 1) * per_block < m <= blocks * per_block
            assert blocks * block < 2**32
            at += m
        assert at == count
