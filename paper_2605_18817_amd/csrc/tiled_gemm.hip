// Launchers of the tile kernel (tiled_gemm_kernel.h): the partial-sum and SiLU forms here, the LM head's in two files of
// their own (compiled side by side).
#include "tiled_gemm_kernel.h"

namespace mrp {

namespace {

template <int NB>
hipError_t launch_two_planes(const TiledGemmArgs &a, int nv, int rem, hipStream_t st) {
    return nv == 3 ? launch_inst<EPI_PARTIAL, false, NB, 3, true>(a, rem, st) : launch_inst<EPI_PARTIAL, false, NB, 4, true>(a, rem, st);
}

// k steps of a part (0: the arguments do not fit)
int part_steps(const TiledGemmArgs &a, bool split) {
    int nsteps = 0;
    for (int sg = 0; sg < a.nseg; ++sg) nsteps += a.seg[sg].nkq * a.seg[sg].nplanes;
    if (a.nKs < 1 || nsteps % a.nKs != 0 || nsteps / a.nKs < 2 || (!split && a.nKs != 1)) return 0;
    return nsteps / a.nKs;       // (at least two)
}

}  // namespace

// Activation rows per tile: M rows in the fewest tiles of at most 256, each of as few 32-row blocks as that needs.
// A block that no row falls into costs what a full one does (time per tile goes with the blocks: 592 rows in three
// tiles are 21 blocks instead of 24).
int tiled_row_blocks(int M) {
    const int ib = (M + 31) / 32, nMt = (ib + 7) / 8, nb = (ib + nMt - 1) / nMt;
    return nb < 5 ? 5 : nb;
}

// Few output tiles (the head body's GEMMs at 1024 or 2048 rows have 64 or 128) leave most CUs idle: split k
// into up to 16 parts so that tiles x parts comes near the CU count; every part must have an equal number of at
// least MRP_TILED_MIN_STEPS k steps and its partial sums must fit the buffer.
int tiled_ksplit(int tiles, int nsteps, int nCU, size_t cap_rows, int M) {
    int ks = 1;
    while (ks < 16 && tiles * ks * 2 <= nCU && nsteps % (ks * 2) == 0 && nsteps / (ks * 2) >= MRP_TILED_MIN_STEPS &&
           (size_t)(ks * 2) * M <= cap_rows)
        ks *= 2;
    return ks;
}

hipError_t launch_tiled_gemm(const TiledGemmArgs &a, int epi, hipStream_t st) {
    const int nsteps = part_steps(a, false), rem = 2 + (nsteps - 2) % 3;
    if (nsteps == 0 || (epi != EPI_LM && epi != EPI_SILU)) return hipErrorInvalidValue;
    int nb = tiled_row_blocks(a.M);
    // EPI_SILU has instances of 7 and 8 row blocks only: on 256 CUs an unsplit k comes with 768 rows and more, which make
    // no shorter tiles.  With fewer CUs (a partition of the device) it comes with fewer rows, too; those are as many
    // tiles of 7 blocks, which fit the workspace (at most 8 blocks for each tile's 256 rows).
    if (epi == EPI_SILU && nb < 7) nb = 7;
    if (a.nMt != (a.M + 32 * nb - 1) / (32 * nb) || a.nMt * nb > a.nIb) return hipErrorInvalidValue;
    if (epi == EPI_LM) {
        const int left = a.nMt * a.nVt % 256;
        return left > 0 && left <= 128 ? launch_tiled_lm_halves(a, nb, rem, st) : launch_tiled_lm(a, nb, rem, st);
    }
    return nb == 7 ? launch_inst<EPI_SILU, false, 7, 4, false>(a, rem, st) : launch_inst<EPI_SILU, false, 8, 4, false>(a, rem, st);
}

hipError_t launch_tiled_partial(const TiledGemmArgs &a, int nb, hipStream_t st) {
    const int nsteps = part_steps(a, true), rem = 2 + (nsteps - 2) % 3;
    if (nsteps == 0 || nb < 5 || nb > 8 || a.nMt != (a.M + 32 * nb - 1) / (32 * nb) || a.nMt * nb > a.nIb) return hipErrorInvalidValue;
    if (nb == 5) return launch_inst<EPI_PARTIAL, false, 5, 4, false>(a, rem, st);
    if (nb == 6) return launch_inst<EPI_PARTIAL, false, 6, 4, false>(a, rem, st);
    if (nb == 7) return launch_inst<EPI_PARTIAL, false, 7, 4, false>(a, rem, st);
    return launch_inst<EPI_PARTIAL, false, 8, 4, false>(a, rem, st);
}

hipError_t launch_tiled_two_planes(const TiledGemmArgs &a, int nb, int nv, hipStream_t st) {
    const int nsteps = part_steps(a, true), rem = 2 + (nsteps - 2) % 3;
    if (nsteps == 0 || a.nseg != 1 || a.seg[0].nplanes != 2 || nv < 3 || nv > 4 || nb < 4 || nb > 8 || a.R % 4 != 0 ||
        a.nMt != (a.M + 32 * nb - 1) / (32 * nb) || a.nMt * nb > a.nIb || a.nVt != (a.R + 64 * nv - 1) / (64 * nv))
        return hipErrorInvalidValue;
    if (nb == 4) return launch_two_planes<4>(a, nv, rem, st);
    if (nb == 5) return launch_two_planes<5>(a, nv, rem, st);
    if (nb == 6) return launch_two_planes<6>(a, nv, rem, st);
    if (nb == 7) return launch_two_planes<7>(a, nv, rem, st);
    return launch_two_planes<8>(a, nv, rem, st);
}

}  // namespace mrp
