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


class _TileForm(C.Structure):
    _fields_ = [("nb", C.c_int), ("nv", C.c_int), ("ks", C.c_int)]


@pytest.mark.parametrize("nCU", [32, 256])
def test_two_plane_forms_fit_and_sum_no_longer(nCU):
    form = library_rule("_ZN3mrp14two_plane_formEiiiimi", _TileForm, *[C.c_int] * 4, C.c_size_t, C.c_int)
    ksplit = library_rule("_ZN3mrp12tiled_ksplitEiiimi", C.c_int, *[C.c_int] * 3, C.c_size_t, C.c_int)
    blocks = library_rule("_ZN3mrp16tiled_row_blocksEi", C.c_int, C.c_int)
    for M in [*range(1, 70), 96, 128, 129, 160, 192, 193, 250, 384, 400, 512, 513, 592, 767, 768, 1000, 1024, 4096, 65535]:
        for R, K in [(32, 64), (32, 128), (128, 128), (4096, 4096), (6144, 4096), (24576, 4096), (4096, 12288), (12288, 2048),
                     (2176, 2176), (131072, 128), (2304, 8192)]:
            for cap in (M, 4 * M, 16 * M, max(M, 4096)):
                for wide in (-1, 0, 1, 2, 4, 8):     # in the place of the one-plane tiles, the small-row kernels, the wide kernel's parts
                    f = form(M, R, K, nCU, cap, wide)
                    if f.ks == 0:                    # (another kernel's: never where the tile kernel is the only one)
                        assert wide >= 0
                        continue
                    tiles = -(-M // (32 * f.nb))
                    assert 4 <= f.nb <= 8 and f.nv in (3, 4) and 1 <= f.ks <= 16 and f.ks * M <= cap
                    assert tiles * f.nb <= -(-M // 256) * 8 and tiles * f.nb * 32 >= M  # row blocks that the planes hold
                    assert K // 32 % f.ks == 0 and K // 32 // f.ks >= min(4, K // 32)   # whole parts of four k steps at least
                    apart = f.nv * f.nb <= 18        # a sum of its own for the low plane: as good as twice the parts
                    if wide < 0:
                        own = ksplit(-(-M // (32 * blocks(M))) * -(-R // 256), K // 32, nCU, cap, M)
                        assert f.ks * (2 if apart else 1) >= own
                    else:
                        assert wide < 8 and apart and f.ks >= (2 * wide or 4)
    if nCU == 256:                                   # the sizes it was measured at
        assert [(f.nb, f.nv, f.ks) for f in (form(384, 24576, 4096, 256, 4096, 1), form(128, 12288, 2048, 256, 2048, 2),
                                             form(592, 4096, 4096, 256, 4096, -1), form(1024, 4096, 4096, 256, 4096, -1),
                                             form(4096, 4096, 4096, 256, 4096, -1), form(384, 4096, 4096, 256, 4096, 0))] \
            == [(6, 3, 2), (4, 3, 4), (5, 4, 4), (4, 4, 2), (8, 4, 1), (4, 4, 4)]


def test_first_body_gemm_keeps_its_parts_or_takes_more():
    form = library_rule("_ZN3mrp12partial_formEiiiim", _TileForm, *[C.c_int] * 4, C.c_size_t)
    ksplit = library_rule("_ZN3mrp12tiled_ksplitEiiimi", C.c_int, *[C.c_int] * 3, C.c_size_t, C.c_int)
    blocks = library_rule("_ZN3mrp16tiled_row_blocksEi", C.c_int, C.c_int)
    for nCU in (32, 256):
        for M in [*range(129, 2000, 31), 592, 640, 768, 1024, 4096, 65535]:
            for d in (128, 1024, 2048, 2176, 2560, 4096, 5120):
                for nsteps in (d // 32, d // 64 * 3):
                    f, cap = form(M, d, nsteps, nCU, max(M, 4096)), max(M, 4096)
                    own = ksplit(-(-M // (32 * blocks(M))) * -(-d // 256), nsteps, nCU, cap, M)
                    assert f.nv == 4 and 5 <= f.nb <= 8 and own <= f.ks <= 16 and f.ks * M <= cap and nsteps % f.ks == 0
                    assert own > 1 or (f.nb, f.ks) == (blocks(M), 1)
                    tiles = -(-M // (32 * f.nb))
                    assert tiles * f.nb <= -(-M // 256) * 8 and tiles * f.nb * 32 >= M
    assert [(f.nb, f.ks) for f in (form(592, 4096, 192, 256, 4096), form(768, 2048, 96, 256, 4096))] == [(5, 4), (6, 4)]


def test_mlp_body_kernel_by_rows_and_width():
    on_tiles = library_rule("_ZN3mrp12mlp_on_tilesEiiim", C.c_bool, *[C.c_int] * 3, C.c_size_t)
    ksplit = library_rule("_ZN3mrp12tiled_ksplitEiiimi", C.c_int, *[C.c_int] * 3, C.c_size_t, C.c_int)
    blocks = library_rule("_ZN3mrp16tiled_row_blocksEi", C.c_int, C.c_int)
    rows = lambda M: 16 * M if M <= 128 else 4096
    for M in range(1, 800):
        for d in range(128, 8193, 128):
            if M >= 768 or (d > 2048 and M > 512):
                assert on_tiles(M, d, 256, rows(M))
            elif M <= 128 or d <= 2048:
                assert not on_tiles(M, d, 256, rows(M))
            elif on_tiles(M, d, 256, rows(M)):       # 129 to 512 rows: k parts of the first GEMM, for one and for two planes
                parts = [ksplit(-(-M // (32 * blocks(M))) * -(-d // 256), d // 64 * n, 256, rows(M), M) for n in (2, 3)]
                assert min(parts) >= 8, (M, d)       # (the small-row kernels have eight waves)
    assert all(on_tiles(M, 4096, 256, 4096) for M in (129, 144, 160, 256, 257, 512))
    assert not any(on_tiles(M, 2560, 256, 4096) for M in (129, 192, 384))
    assert not any(on_tiles(M, 3072, 256, 4096) for M in (129, 144, 256)) and all(on_tiles(M, 3072, 256, 4096) for M in (257, 384, 512))


def test_head_body_per_sequence_only_where_it_is_ahead():
    rule = library_rule("_ZN3mrp16mlp_per_sequenceEiii", C.c_bool, *[C.c_int] * 3)
    for d in range(128, 1025, 128):
        for L in range(1, 65):
            for B in (1, 3, 256, 4096, 65535 // L):
                assert not (rule(B, L, d) and (d > 256 or L > 16))
    ahead = {256: [(1, 1), (512, 1), (768, 1), (1024, 1), (256, 2), (1500, 2), (2000, 3), (2000, 4), (2300, 6), (8000, 8), (4000, 16)],
             128: [(1, 1), (1400, 1), (3000, 2), (4000, 3), (4000, 4), (8192, 6), (8000, 8), (4000, 16)]}
    behind = {256: [(513, 1), (767, 1), (1200, 1), (4096, 1), (2600, 2), (4096, 2), (3000, 3), (4000, 4), (8192, 6)],
              128: [(4096, 1), (8000, 3), (8000, 4)]}          # B x L as measured
    assert all(rule(B, L, d) for d in ahead for B, L in ahead[d])
    assert not any(rule(B, L, d) for d in behind for B, L in behind[d])


def test_waiting_gradient_workgroups_leave_the_device_free():
    counters = library_rule("_ZN3mrp11kl_countersEiii", C.c_int, *[C.c_int] * 3)
    for nCU in (1, 8, 32, 64, 127, 128, 256):
        for nT in range(1, 300):
            for M in (1, 16, 100, 1024, 65535):
                nq = counters(M, nT, nCU)
                assert nq in (0, 1, 3, 5, 7) and nq * (nT - 1) <= nCU // 2      # of 4 nCU resident workgroups
                assert nq == 0 or (nCU >= 128 and M * nT * nCU >= 2048 * 256)
    assert counters(1024, 19, 256) == 7 and counters(64, 19, 256) == 0 and counters(1024, 33, 256) == 3
    assert counters(128, 19, 128) == 0 and counters(512, 19, 128) == 3 and counters(1024, 4, 64) == 0   # (where it was measured)


def test_two_pass_gradient_takes_rows_that_the_cache_holds():
    rows = library_rule("_ZN3mrp13kl_group_rowsEii", C.c_int, C.c_int, C.c_int)
    for V in (1, 100, 4096, 50257, 151936, 1100000, 3000000, 3500000, 4000000, 67000000):
        for M in (1, 2, 16, 89, 128, 135, 1024, 32768, 65535):
            r, row = rows(M, V), 4 * V
            assert 1 <= r <= M
            if r < M:                                # two tensors of two groups in 256 MB, no fewer than four rows a group
                assert 4 * r * row <= 256 << 20 and r >= 4 and 2 * r <= 65535
            else:
                assert row > (13 << 20) or M * row < 78 << 20
    assert [rows(128, 1200000), rows(100, 3000000), rows(64, 4000000), rows(1024, 151936), rows(16, 151936)] == [11, 4, 64, 89, 16]
