"""The tile kernel's forms through their own launchers: the SiLU epilogue (with all the CUs of a whole device the library
splits k at the row counts whose tiles are shorter than seven row blocks, so no chain step reaches this epilogue there; on
a partition of the device, with fewer CUs, it does), the partial sums at every tile size, and their error beside that of
the kernels in whose place they stand."""
import ctypes as C

import pytest
import torch

import paper_2605_18817_amd as mrp

pytestmark = pytest.mark.gpu

EPI_SILU = 2


class _Seg(C.Structure):
    _fields_ = [("base", C.c_void_p), ("plane_stride", C.c_long), ("nkq", C.c_int), ("nplanes", C.c_int)]


class _Args(C.Structure):
    _fields_ = ([("Wp", C.c_void_p)] + [(n, C.c_int) for n in ("KBw", "n_rb", "nIb", "M", "R")] + [("seg", _Seg * 2)]
                + [(n, C.c_int) for n in ("nseg", "nMt", "nVt", "nKs")]
                + [("out", C.c_void_p), ("planes", C.c_void_p), ("plane_stride", C.c_long)]
                + [(n, C.c_void_p) for n in ("z", "pm", "ps")])


def _plane_index(rows, cols, nIb):
    """Position of entry (row, col) in an activation plane [k block][row block][lane][8]."""
    r, c = torch.arange(rows, device="cuda").unsqueeze(1), torch.arange(cols, device="cuda").unsqueeze(0)
    return (((c >> 4) * nIb + (r >> 5)) * 64 + (r & 31) + 32 * ((c >> 3) & 1)) * 8 + (c & 7)


@pytest.mark.parametrize("M", [1, 300, 513, 576, 577, 768])     # 5, 5, 6, 6, 7 and 8 row blocks fit the rows
def test_silu_epilogue_at_every_tile_height(M):
    lib = mrp.load_library()
    row_blocks = getattr(lib, "_ZN3mrp16tiled_row_blocksEi")(M)
    launch = getattr(lib, "_ZN3mrp17launch_tiled_gemmERKNS_13TiledGemmArgsEiP12ihipStream_t")
    R, K, nIb = 256, 256, -(-M // 256) * 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    x = torch.empty(M, K, device="cuda").normal_(0, 1, generator=gen)
    w = torch.empty(R, K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=gen)
    planes = torch.zeros(2, K // 16 * nIb * 512, dtype=torch.float16, device="cuda")
    idx = _plane_index(M, K, nIb)
    hi = x.half()
    planes[0, idx], planes[1, idx] = hi, (x - hi.float()).half()
    out = torch.full((2, R // 16 * nIb * 512), 7.0, dtype=torch.float16, device="cuda")
    Wp = mrp.pack_weight(w, body=True)
    a = _Args()
    a.Wp, a.KBw, a.n_rb, a.nIb, a.M, a.R = Wp.data_ptr(), K // 16, R // 32, nIb, M, R
    a.seg[0] = _Seg(planes.data_ptr(), planes.shape[1] // 8, K // 64, 2)
    a.nseg, a.nMt, a.nVt, a.nKs = 1, -(-M // (32 * row_blocks)), 1, 1
    a.planes, a.plane_stride = out.data_ptr(), out.shape[1] // 8
    assert launch(C.byref(a), EPI_SILU, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    xe, we = planes[0, idx].double() + planes[1, idx].double(), w.half().double()
    s = xe @ we.t()
    ref = s * torch.sigmoid(s)
    idx_o = _plane_index(M, R, nIb)
    got = out[0, idx_o].double() + out[1, idx_o].double()
    # fp32 sums: two planes of K / 16 MFMAs of 16 products, each addition within 2^-24 of what was summed so far; SiLU's
    # slope is below 1.1 and its own evaluation a few ulp; hi + lo holds 2^-22 of the value, 2^-25 where lo is subnormal
    bound = 1.1 * (2 * K // 16 + 16) * 2.0 ** -24 * (xe.abs() @ we.abs().t()) + 2.0 ** -20 * ref.abs() + 2.0 ** -24
    assert bool(((got - ref).abs() <= bound).all()), float(((got - ref).abs() / bound).max())
    rest = torch.ones_like(out[0], dtype=torch.bool)
    rest[idx_o] = False
    assert bool((out[:, rest] == 7.0).all())                      # rows past M are not written


# Tiles of 192 and 256 weight rows x every height; 4 to 14 k steps of 32 (each length of the kernel's tail), one part or
# several; rows and outputs that end inside a tile, an output narrower than one
@pytest.mark.parametrize("M,R,K,nb,nv,ks", [
    (1, 32, 128, 4, 4, 1), (128, 256, 192, 4, 4, 1), (129, 288, 320, 4, 3, 2), (250, 192, 1024, 4, 3, 8),
    (160, 416, 576, 5, 3, 3), (75, 224, 320, 5, 4, 2), (192, 384, 448, 6, 3, 2), (190, 320, 512, 6, 4, 4),
    (200, 192, 256, 7, 3, 2), (224, 512, 384, 7, 4, 2), (256, 96, 448, 8, 3, 1), (450, 544, 640, 8, 4, 4),
])
def test_two_plane_forms(M, R, K, nb, nv, ks):
    lib = mrp.load_library()
    launch = getattr(lib, "_ZN3mrp23launch_tiled_two_planesERKNS_13TiledGemmArgsEiiP12ihipStream_t")
    nIb = max(-(-M // 256) * 8, -(-M // (32 * nb)) * nb)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + R)
    x = torch.empty(M, K, device="cuda").normal_(0, 1, generator=gen)
    w = torch.empty(R, K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=gen)
    planes = torch.zeros(2, K // 16 * nIb * 512, dtype=torch.float16, device="cuda")
    idx = _plane_index(M, K, nIb)
    hi = x.half()
    planes[0, idx], planes[1, idx] = hi, (x - hi.float()).half()
    out = torch.full((ks * M * R + 64,), 7.0, device="cuda")
    Wp = mrp.pack_weight(w, body=True)
    a = _Args()
    a.Wp, a.KBw, a.n_rb, a.nIb, a.M, a.R = Wp.data_ptr(), K // 16, R // 32, nIb, M, R
    a.seg[0] = _Seg(planes.data_ptr(), planes.shape[1] // 8, K // 64, 2)
    a.nseg, a.nMt, a.nVt, a.nKs, a.out = 1, -(-M // (32 * nb)), -(-R // (64 * nv)), ks, out.data_ptr()
    assert launch(C.byref(a), nb, nv, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    got = out[:ks * M * R].view(ks, M, R).double()
    xe, we = planes[0, idx].double() + planes[1, idx].double(), w.half().double()
    kp = K // ks
    for n in range(ks):
        xs, ws = xe[:, n * kp:(n + 1) * kp], we[:, n * kp:(n + 1) * kp]
        # two planes of K / 32 MFMAs of twice 16 products (the bits are those of the 16-wide instruction), each addition
        # within 2^-24 of what was summed so far
        bound = (2 * kp // 16 + 32) * 2.0 ** -24 * (xs.abs() @ ws.abs().t())
        err = (got[n] - xs @ ws.t()).abs()
        assert bool((err <= bound).all()), (n, float((err / bound).max()))
    assert bool((out[ks * M * R:] == 7.0).all())                   # nothing past the last part


def test_tile_height_does_not_change_partial_sums():
    """The forms of 256 weight rows and one plane at a time: what a part adds up does not depend on the tile."""
    lib = mrp.load_library()
    launch = getattr(lib, "_ZN3mrp20launch_tiled_partialERKNS_13TiledGemmArgsEiP12ihipStream_t")
    M, R, K, ks, nIb = 592, 288, 320, 3, 24
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.empty(M, 2 * K, device="cuda").normal_(0, 1, generator=gen)
    w = torch.empty(R, 2 * K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=gen)
    planes = torch.zeros(3, K // 16 * nIb * 512, dtype=torch.float16, device="cuda")
    idx = _plane_index(M, K, nIb)
    hi = x[:, :K].half()
    planes[0, idx], planes[1, idx], planes[2, idx] = hi, (x[:, :K] - hi.float()).half(), x[:, K:].half()
    Wp = mrp.pack_weight(w, body=True)
    xe = torch.cat([planes[0, idx].double() + planes[1, idx].double(), planes[2, idx].double()], 1)
    outs = []
    for nb in (5, 6, 7, 8):
        out = torch.full((ks * M * R + 64,), 7.0, device="cuda")
        a = _Args()
        a.Wp, a.KBw, a.n_rb, a.nIb, a.M, a.R = Wp.data_ptr(), 2 * K // 16, R // 32, nIb, M, R
        a.seg[0] = _Seg(planes.data_ptr(), planes.shape[1] // 8, K // 64, 2)
        a.seg[1] = _Seg(planes[2].data_ptr(), 0, K // 64, 1)
        a.nseg, a.nMt, a.nVt, a.nKs, a.out = 2, -(-M // (32 * nb)), -(-R // 256), ks, out.data_ptr()
        assert launch(C.byref(a), nb, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        assert bool((out[ks * M * R:] == 7.0).all())
        outs.append(out[:ks * M * R].view(ks, M, R))
        assert torch.equal(outs[0], outs[-1])
    we = w.half().double()
    # K / 32 MFMAs of twice 16 products for each of three planes, the parts' sums in 64 bits
    bound = (3 * K // 16 + 32) * 2.0 ** -24 * (xe.abs() @ we.abs().t())
    assert bool(((outs[0].double().sum(0) - xe @ we.t()).abs() <= bound).all())


class _Wide(C.Structure):
    _fields_ = ([("Wp", C.c_void_p), ("X", C.c_void_p), ("plane", C.c_long), ("nplanes", C.c_int), ("out", C.c_void_p)]
                + [(n, C.c_int) for n in ("nIb", "M", "R", "Kc", "nKs", "nft", "nrg", "nf")])


class _Small(C.Structure):
    _fields_ = ([("Wp", C.c_void_p), ("X", C.c_void_p), ("plane", C.c_long), ("nplanes", C.c_int), ("out", C.c_void_p)]
                + [(n, C.c_int) for n in ("nIb", "M", "R", "Kc", "nf", "nct", "nrt")])


@pytest.mark.parametrize("K", [1024, 2560, 4096, 12288])
def test_two_planes_are_no_further_from_64_bits(K):
    """A two-plane form that sums as long as the rule allows, and the kernel in whose place it stands, on the same product
    (a root mean square over 256 x 512 sums, of which each kernel's rounding is a fixed property): the wide kernel with
    1, 2 and 4 parts, the small-row kernels, the one-plane tiles with 1 to 8 parts."""
    lib = mrp.load_library()
    two = getattr(lib, "_ZN3mrp23launch_tiled_two_planesERKNS_13TiledGemmArgsEiiP12ihipStream_t")
    one = getattr(lib, "_ZN3mrp20launch_tiled_partialERKNS_13TiledGemmArgsEiP12ihipStream_t")
    wide = getattr(lib, "_ZN3mrp16launch_wide_gemmERKNS_12WideGemmArgsEP12ihipStream_t")
    small = getattr(lib, "_ZN3mrp17launch_small_gemmERKNS_13SmallGemmArgsEP12ihipStream_t")
    M, R, nIb = 256, 512, 8
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    x = torch.empty(M, K, device="cuda").normal_(0, 1, generator=gen)
    w = torch.empty(R, K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=gen)
    planes = torch.zeros(2, K // 16 * nIb * 512, dtype=torch.float16, device="cuda")
    idx = _plane_index(M, K, nIb)
    hi = x.half()
    planes[0, idx], planes[1, idx] = hi, (x - hi.float()).half()
    Wp = mrp.pack_weight(w, body=True)
    exact = (planes[0, idx].double() + planes[1, idx].double()) @ w.half().double().t()
    out = torch.empty(8 * M * R, device="cuda")
    src = (Wp.data_ptr(), planes.data_ptr(), planes.shape[1] // 8, 2, out.data_ptr())

    def tiles(launch, ks, nb, *nv):
        a = _Args()
        a.Wp, a.KBw, a.n_rb, a.nIb, a.M, a.R = Wp.data_ptr(), K // 16, R // 32, nIb, M, R
        a.seg[0] = _Seg(planes.data_ptr(), planes.shape[1] // 8, K // 64, 2)
        a.nseg, a.nMt, a.nVt, a.nKs, a.out = 1, -(-M // (32 * nb)), -(-R // (64 * (nv or (4,))[0])), ks, out.data_ptr()
        return launch(C.byref(a), nb, *nv, st)

    def error(rc, ks):
        assert rc == 0
        torch.cuda.synchronize()
        parts = out[:ks * M * R].view(ks, M, R)
        total = parts[0].clone()
        for p in parts[1:]:                                        # as the consumers add them
            total += p
        return float((total.double() - exact).norm() / exact.norm())

    apart = {ks: error(tiles(two, ks, 4, nv), ks) for ks, nv in ((1, 4), (2, 3), (4, 4), (8, 3)) if K // 32 % ks == 0}
    both = {ks: error(tiles(two, ks, 8, 4), ks) for ks in (1, 2, 4, 8)}
    own = {ks: error(tiles(one, ks, 8), ks) for ks in (1, 2, 4, 8)}
    for ks in (1, 2, 4):
        if K // 16 % (ks * 16) == 0:
            assert apart[2 * ks] <= error(wide(C.byref(_Wide(*src, nIb, M, R, K, ks, R // 64, M // 128, 2)), st), ks), ks
        assert apart[ks] <= own[2 * ks], ks
    assert apart[4] <= error(small(C.byref(_Small(*src, nIb, M, R, K, 1, R // 32, M // 32)), st), 1)
    # (one sum for both planes adds the same products in another order: at most 1 % apart either way)
    assert all(both[ks] <= 1.01 * own[ks] for ks in both), (both, own)
