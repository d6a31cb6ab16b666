"""The rules that choose between kernels by size, on the host (no GPU): the library's own functions, compared over all
sizes they accept with what they must hold to."""
import ctypes as C

import pytest

from harness import library_rule


def _stream_parts(M, d, part_rows):
    """k parts of the streaming kernel for the fuse projection: 512 workgroups, at most 16 parts, each at least two
    128-wide ranges, partial sums within the buffer."""
    groups = -(-M // 256) if M > 128 else 1          # 256 rows per workgroup, 128 below
    tiles = (d // 128) * groups
    return max(1, min(-(-512 // tiles), 16, d // 128, part_rows // M))


@pytest.mark.parametrize("nCU", [32, 256])
@pytest.mark.parametrize("wide", [1, 6])             # the layers' partial-sum buffer holds that many times as many rows
def test_fuse_projection_keeps_its_k_parts_on_tiles(nCU, wide):
    fuse_parts = library_rule("_ZN3mrp15fuse_tile_partsEiiiimm", C.c_int, *[C.c_int] * 4, C.c_size_t, C.c_size_t)
    taken = set()
    for M in [*range(1, 20), *range(20, 768, 7), 128, 129, 192, 256, 257, 384, 512, 513]:
        part_rows = 16 * M if M <= 128 else 4096
        for d in range(128, 8193, 128):
            for planes in (1, 2):
                parts = fuse_parts(M, d, planes, nCU, part_rows, wide * part_rows)
                if parts == 0:
                    continue
                taken.add((M, d))
                steps = d // 64 * (planes + 1)
                assert steps % parts == 0 and steps // parts >= 4 and parts * M <= wide * part_rows
                assert parts >= _stream_parts(M, d, part_rows), (M, d, planes)
    if nCU == 256 and wide == 6:                     # the sizes it was measured at, on either side
        assert {(4, 4096), (128, 4096), (384, 4096), (512, 4096), (256, 2048), (384, 2048), (384, 5120)} <= taken
        assert not {(128, 2048), (128, 1024), (512, 1024), (4, 2176), (128, 2176)} & taken


@pytest.mark.parametrize("S,resident", [(3, 8), (5, 8), (9, 4), (17, 2)])      # workgroups that a CU holds (LDS, registers)
def test_residual_workgroups_fill_the_device(S, resident):
    workgroups = library_rule("_ZN3mrp23residual_rms_workgroupsEiili", C.c_int, C.c_int, C.c_int, C.c_long, C.c_int)
    nCU, room = 256, 4096                            # partials the context's buffer holds
    for n in [*range(1, 130), 200, 300, 400, 1000, 4095, 4096]:
        for ntiles in (1, 2, 31, 32, 33, 128, 512, 786, 1571, 2374, 4749):
            w = workgroups(n, S, ntiles, nCU)
            assert 1 <= w <= ntiles and n * w <= room
            if S < 9:
                assert w == min(ntiles, room // n)   # requests in flight: every partial there is room for
                continue
            # tile times until the last workgroup is done, in whole rounds of what is resident: no more than with all
            # the partials' room (a start and a reduction, half a tile each time, included)
            rounds = lambda v: -(-n * v // (resident * nCU))
            cost = lambda v: rounds(v) * (2 * -(-ntiles // v) + 1)
            assert cost(w) <= cost(min(ntiles, room // n)), (n, ntiles, w)
