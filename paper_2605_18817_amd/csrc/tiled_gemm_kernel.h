// Tiled MFMA GEMM (bf16 operands for the LM head, fp16 for the head body) for many activation rows (the MFMA-bound regime of the MRP
// chain):  out[i][r] (+)= sum_k W[r][k] * X[i][k]  with output tiles of up to 256 x 256.
//
// A workgroup of four wavefronts computes a tile of 256 weight rows x 160 to 256 activation rows (LM head: as few 32-row
// blocks as M rows need in that many tiles; halved tiles 96 or 128; two planes 192 or 256 x 128 to 256);
// each wave owns 64 (48) weight rows x all activation rows as 4 (3) x 6 to 16 MFMA 16x16x32 tiles (up to
// 256 fp32 accumulators).  The weight fragments go from the packed layout straight into MFMA
// operand registers (the same 1 KiB blocks of 32 rows x 16 k, a fragment of 16 rows x 32 k being four 256-byte
// runs of two of them); no two waves load the same fragment.  The activation operand arrives in LDS by LDS-direct
// loads (three 32 KiB stages) and every wave reads all of it.  As in the streaming kernels the weight fragment is
// the MFMA "A" operand, so a lane's accumulators of a sub-tile are 4 consecutive outputs of one activation row.
//
// What limits this kernel: the chip's power and the memory requests of a k step.  With zero weights the LM head of
// 4096 rows (d = 4096, V = 151936) took 3.71 ms, with random ones 4.28 ms: the clock falls under the load.  So it
// takes the MFMA that costs the least per product: a loop of LDS fragment reads and MFMAs reaches 1.73 PFLOP/s on random
// data with 32x32x16 (which passes its accumulators through the core twice as often) and 1.93 with 16x16x32 (2.45 both
// on zeros).  Without its epilogue that LM head takes 3.64 ms (1.4 PFLOP/s; without the k loop's memory requests
// 2.84 ms, without its LDS reads as well 2.55 ms): the layout is the one with the fewest request bytes (64 KiB per
// step), operands are requested two steps ahead, and the requests are spread between the MFMAs.
// Per head, 32x32x16 / now, epilogue and halved tiles included: 4.69 / 4.23 ms at 4096 rows, 1.23 / 1.11 at 1024, 0.78 / 0.73 at
// 592 (d = 4096); of that the MFMA shape 4 %, one wait for the LDS reads per phase 1.5 %, the place of the barrier 1.5 %, the order of
// the MFMAs 0.7 %.
//
// The head body's activations are two fp16 planes.  Where all of an operand is (P2), a k step is 32 k of both planes,
// so that a weight fragment is requested once for both (48 KiB of requests per step instead of 64), and the tiles
// come in more sizes (192 or 256 weight rows, 128 to 256 activation rows): with few tiles what counts is how many CUs
// they leave idle.  At 384 rows, d = 4096 (us, the wide GEMM kernel / 256 x 192 tiles with the planes one after the other /
// in the parts that keep the wide kernel's rounding): 24576 x 4096 187 / 146 / 121, 6144 x 4096 52 / 45 / 36, 4096 x 12288 78 /
// 62 / 69.
//
// Workgroups are ordered so that the 32 CUs of one XCD work at the same time on a
// block of 4 (activation) x 8 (weight) tiles and share its operand slices in that
// XCD's L2.
//
// Epilogues: EPI_PARTIAL (fp32 tile to out[i][r]; part ks of a k split to out[ks][i][r]), EPI_SILU (SiLU of the
// tile as the two fp16 activation planes of the next GEMM; no k split) and EPI_LM (the tile is added to the
// logit state, which is stored back, and the per-row (max, sum-exp) partial of
// the tile's 256 vocabulary entries is written: the merge looks up which entry the maximum is; paper Section 3.2 / Algorithm 2
// l <- l + delta).
#pragma once
#include "mrp_kernels.h"

#include <type_traits>

namespace mrp {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));   // native vector: arrays of it stay in registers
// One 16x16x32 matrix multiply-accumulate on 16-byte operand fragments: the partial-sum GEMMs of the
// head body take fp16 operands (weights converted at pack time, activations as fp16 planes), the LM
// head bf16 ones.  The accumulator stays where it is (with the builtin the compiler gives sources and result
// different registers and moves accumulators about), and volatile statements keep their order against the memory
// requests.  Nothing here waits: operands must come from loads, and accumulators may be read after
// acc_ready() only.
template <int EPI, bool VREG = false>      // VREG: the accumulator is among the ordinary registers
__device__ __forceinline__ void mma_frag(f32x4 &c, const u32x4 &w, const u32x4 &x) {
    if constexpr (VREG)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(x));
    else if constexpr (EPI != EPI_LM)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}

constexpr int TG_KB = 4;                    // 16-wide k blocks per step (64 k)
constexpr int TG_B = TG_KB * 8 * 64;        // u32x4 of an activation stage (up to 256 rows x 64 k)
constexpr int TG_STAGE = TG_B;              // 32 KiB
constexpr int TG_DEPTH = 3;                 // operand sets: steps s, s + 1, s + 2

// One array per activation stage: the stage arrives by LDS-direct loads, and with separate
// arrays the compiler's wait before reading one stage does not cover the loads into the others.
__shared__ u32x4 tg_stage0[TG_STAGE];
__shared__ u32x4 tg_stage1[TG_STAGE];
__shared__ u32x4 tg_stage2[TG_STAGE];

typedef const __attribute__((address_space(1))) void *gas_ptr;
typedef __attribute__((address_space(3))) void *las_ptr;

// Workgroup barrier after this wave's LDS accesses have completed; no fence, so the loads in
// flight for later steps are not drained.
__device__ __forceinline__ void tg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Maximum without the instruction per operand that the compiler puts ahead of fmaxf to quieten signalling NaNs
__device__ __forceinline__ float max3(float x, float y, float z) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
}
// The four lanes of a row of a 16 x 16 tile lie 16 apart.  The exchanges swap every other 16 lanes / the two halves of two
// registers, here of two copies of the same one.
template <class F>
__device__ __forceinline__ float row_combine(float x, F f) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    x = f(__int_as_float(a[0]), __int_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
    return f(__int_as_float(b[0]), __int_as_float(b[1]));
}

// REM = 2 + (k steps - 2) % 3: the k steps left for the straight-line tail after the unrolled loop (one form each: where
// the tails of one form meet again, accumulators are moved about)
// RAG: R is not a multiple of 4 (EPI_LM), so a row of the logit state starts on any 4-byte boundary and ends inside a
// 16-byte piece
// NB: 32-row blocks of activation rows per tile (4 to 8)
// NV: 16-row blocks of weight rows per wave (3 or 4: tiles of 192 or 256 weight rows)
// P2: the activation is one segment of two planes; a step is 32 k of both, whose weight fragments are fetched once
// vt, ib0, ks: weight tile, first row block and k part; row_lim: the rows from there on are not the tile's
template <int EPI, int REM, bool RAG, int NB, int NV, bool P2>
__device__ __forceinline__ void tile_body(const TiledGemmArgs &a, int vt, int ib0, int ks, int row_lim) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 15, lq = lane >> 4;

    const int rw0 = (vt * 4 + wave) * 16 * NV;      // this wave's first weight row
    const u32x4 *Wp = reinterpret_cast<const u32x4 *>(a.Wp);

    // A fragment of 16 rows x 32 k is four runs of 16 chunks (256 bytes) of two packed blocks: the lane's chunk in it
    // (for activations, whose next k block lies NB blocks on, frag_x)
    const int frag_w = ln + 32 * (lq & 1) + 64 * (lq >> 1), frag_x = ln + 32 * (lq & 1) + 64 * NB * (lq >> 1);

    // this wave's NV blocks of 16 weight rows, two of which share a packed block (rows past the padded matrix re-read
    // the last one)
    constexpr int NPTR = NV % 2 ? NV : NV / 2;
    const u32x4 *asrc[NPTR];
#pragma unroll
    for (int n = 0; n < NPTR; ++n) {
        const int r16 = rw0 / 16 + n * (NV / NPTR);
        const int rb = r16 / 2 < a.n_rb ? r16 / 2 : a.n_rb - 1;
        asrc[n] = Wp + (size_t)rb * a.KBw * 64 + 16 * (r16 & 1) + frag_w;
    }
    auto wfrag = [&](int q, int kb) __attribute__((always_inline)) -> u32x4 {      // rows 16 q .., k blocks kb and kb + 1
        return NV % 2 ? asrc[q % NPTR][(size_t)kb * 64] : asrc[q / 2 % NPTR][(size_t)kb * 64 + 16 * (q & 1)];
    };

    // k-step sequence: segments x (k quads) x planes
    const int seg0_steps = a.seg[0].nkq * a.seg[0].nplanes;
    const int nsteps_all = seg0_steps + (a.nseg > 1 ? a.seg[1].nkq * a.seg[1].nplanes : 0);
    const int nsteps = nsteps_all / a.nKs;          // this k part's steps (the host makes the split even)
    const int st_begin = ks * nsteps, st_end = st_begin + nsteps;
    // Cursor over the k steps (segment, k quad, plane), advanced one step at a time without
    // divisions; it stops on the last step, which the padded tail re-fetches.  The segment
    // descriptions are copied out of the kernel arguments once (and made opaque, so that they
    // are not re-read from memory in every step).
    long seg_base0 = (long)a.seg[0].base, seg_base1 = (long)a.seg[1].base;
    long seg_ps0 = a.seg[0].plane_stride, seg_ps1 = a.seg[1].plane_stride;
    int seg_np0 = a.seg[0].nplanes, seg_np1 = a.seg[1].nplanes;
    int seg_nkq0 = a.seg[0].nkq;
    asm volatile("" : "+s"(seg_base0), "+s"(seg_base1), "+s"(seg_ps0), "+s"(seg_ps1), "+s"(seg_np0), "+s"(seg_np1),
                 "+s"(seg_nkq0));
    const long kq_stride = (long)TG_KB * a.nIb * 64;   // u32x4 per k quad of a plane
    int cu_st = st_begin, cu_seg = 0, cu_kq = 0, cu_p = 0;
    if (st_begin > 0) {      // where this k part starts: steps run over (segment, k quad, plane)
        cu_seg = st_begin >= seg0_steps ? 1 : 0;
        const int sl = cu_seg ? st_begin - seg0_steps : st_begin, np = cu_seg ? seg_np1 : seg_np0;
        cu_kq = sl / np;
        cu_p = sl % np;
    }
    auto cursor_get = [&](int &kbw, const u32x4 *&bptr) __attribute__((always_inline)) {
        if constexpr (P2) {
            kbw = 2 * cu_st;
            bptr = reinterpret_cast<const u32x4 *>(seg_base0) + ((long)kbw * a.nIb + ib0) * 64;
            return;
        }
        kbw = ((cu_seg ? seg_nkq0 : 0) + cu_kq) * TG_KB;
        const long base = cu_seg ? seg_base1 : seg_base0;
        const long ps = cu_seg ? seg_ps1 : seg_ps0;
        bptr = reinterpret_cast<const u32x4 *>(base) + (cu_p * ps + cu_kq * kq_stride + (long)ib0 * 64);
    };
    auto cursor_next = [&]() __attribute__((always_inline)) {
        if (cu_st + 1 < st_end) {
            ++cu_st;
            if constexpr (!P2) {
                if (++cu_p == (cu_seg ? seg_np1 : seg_np0)) {
                    cu_p = 0;
                    if (++cu_kq == seg_nkq0 && cu_seg == 0) { cu_kq = 0; cu_seg = 1; }
                }
            }
        }
    };
    // activation chunk c of a step (c = 0 .. 4 NB - 1: row block c % NB of k block c / NB; P2: of plane c / (2 NB))
    const long chunk_hi = P2 ? seg_ps0 : 2 * (long)a.nIb * 64;
    auto chunk_at = [&](const u32x4 *b, int c) __attribute__((always_inline)) -> const u32x4 * {
        const int ib = NB > 4 || EPI != EPI_LM || ib0 + c % NB < a.nIb ? c % NB : 0;      // (the second half of a tile of 5 or 7 blocks)
        return b + ((c / NB >> 1) * chunk_hi + ((long)(c / NB & 1) * a.nIb + ib) * 64 + lane);
    };

    // Operands are requested two steps ahead.  Per step and wave: NB LDS-direct loads (this wave's
    // quarter of the activation stage, [k block][row block]) and NWL weight-fragment loads into the register set
    // of that step, in turn; requests complete in issue order.
    constexpr int NWK = P2 ? 1 : 2, NWL = NWK * NV, NREQ = NB + NWL;
    u32x4 areg[TG_DEPTH][NWK][NV];    // [step % 3][32 k][16 weight rows]
    auto request = [&](u32x4 (&set)[NWK][NV], u32x4 *stage, int kbw, const u32x4 *bp, int r) __attribute__((always_inline)) {
        const int wl = r * NWL / NREQ;
        if ((r + 1) * NWL / NREQ > wl) {
            set[wl / NV][wl % NV] = wfrag(wl % NV, kbw + 2 * (wl / NV));
        } else {
            const int c = wave + 4 * (r - wl);
            __builtin_amdgcn_global_load_lds((gas_ptr)chunk_at(bp, c), (las_ptr)(stage + c * 64), 16, 0, 0);
        }
    };
    int kbw_n;
    const u32x4 *bp_n;
    auto request_step = [&](u32x4 (&set)[NWK][NV], u32x4 *stage) __attribute__((always_inline)) {
        cursor_get(kbw_n, bp_n);
        cursor_next();
#pragma unroll
        for (int r = 0; r < NREQ; ++r) request(set, stage, kbw_n, bp_n, r);
        __builtin_amdgcn_sched_barrier(0);
    };
    request_step(areg[0], tg_stage0);
    request_step(areg[1], tg_stage1);

    f32x4 acc[NV][NB][2];             // [16 weight rows][32-row block][its 16 rows]
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                acc[q][ib][hi] = f32x4{0.f, 0.f, 0.f, 0.f};
                asm volatile("" : "+a"(acc[q][ib][hi]));      // (opaque: zeros made anew on two paths end in copies where they meet)
            }
    // Two planes on short tiles leave registers for a sum of its own for the low plane: its products (2^-11 of the high
    // plane's) would round the high plane's sum as often again.
    constexpr bool LO = P2 && tiled_low_apart(NV, NB);
    f32x4 low[LO ? NV : 1][LO ? NB : 1][2];
    if constexpr (LO) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int ib = 0; ib < NB; ++ib)
#pragma unroll
                for (int hi = 0; hi < 2; ++hi) {
                    low[q][ib][hi] = f32x4{0.f, 0.f, 0.f, 0.f};
                    asm volatile("" : "+v"(low[q][ib][hi]));
                }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70 | (NREQ & 15) | (NREQ >> 4 << 14));   // vmcnt(NREQ): the first step's operands
    tg_barrier();

    // activation fragments are double-buffered: the LDS reads of the next phase (half the rows of every row block,
    // 32 k) are issued among the MFMAs of the current one (one wave per SIMD: nothing else hides them)
    u32x4 bf[2][NB];
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) bf[0][ib] = tg_stage0[ib * 64 + frag_x];
    constexpr int NBQ = (NB + 2) / 3;           // LDS reads in each of a phase's first three quarters

    // Logit tile of the epilogue (EPI_LM): NB slices of 32 activation rows x this wave's 64 vocabulary
    // entries, 8 16-byte pieces per lane each.  A piece is always fetched (addresses clamped into
    // the matrix; what lies outside is never used), so the number of requests per step is fixed.
    // The first two slices are requested during the last two k steps, in place of the operand
    // requests those steps no longer need (more would not fit the registers next to the k loop's; RAG with eight row
    // blocks has room for the first only: with the second it spills ten registers, 108 -> 111 us at 512 rows, d = 1024,
    // V = 50257).
    constexpr int ZD = RAG ? 2 : (NB < 5 ? NB + 1 : 6);     // slice buffers: five (one) slices in flight ahead of the one added
    constexpr int ZE = RAG && NB == 8 ? 1 : 2;  // slices requested in the k loop
    f32x4 zc[ZD][8];
    // Every 16 rows of the tile as a buffer of their own, with as many of them as lie inside row_lim: a piece past those, or
    // (zoff) past the end of its row, reads zero and is not stored, without a branch for each piece.  The rows stand in the
    // buffer's base and its size: a scalar offset is no part of what a raw buffer's bounds check compares.
    const int zv_lane = rw0 + 4 * lq;           // + 16 q
    float *const ztile = a.z + (size_t)ib0 * 32 * a.R;
    const size_t zgroup = (size_t)16 * a.R;
    auto zbuf = [&](int ib, int hi) __attribute__((always_inline)) -> __amdgpu_buffer_rsrc_t {
        const int g = 2 * ib + hi, left = row_lim - ib0 * 32 - 16 * g, rows = left < 16 ? left : 16;
        return __builtin_amdgcn_make_buffer_rsrc(ztile + g * zgroup, 0, left > 0 ? (unsigned)rows * (unsigned)a.R * 4u : 0u, 0x00020000);
    };
    unsigned zoff[4];
    if constexpr (EPI == EPI_LM && !RAG) {
#pragma unroll
        for (int q = 0; q < 4; ++q) zoff[q] = zv_lane + 16 * q < a.R ? (unsigned)(ln * a.R + zv_lane + 16 * q) * 4u : 0xffffff00u;
    }
    auto zpiece = [&](int ib, int pc) __attribute__((always_inline)) -> f32x4 {   // pc: 4 hi + q
        if constexpr (RAG) {
            int i = (ib0 + ib) * 32 + 16 * (pc >> 2) + ln;
            int v = zv_lane + 16 * (pc & 3);
            i = i < a.M ? i : a.M - 1;
            // (a piece that crosses the end of its row takes in the start of the next one, or starts early where that
            //  would pass the end of the matrix: the epilogue does not use it)
            const int to_end = a.M - i < 4 ? (a.M - i) * a.R - 4 : a.R, v_max = to_end < a.R - 1 ? to_end : a.R - 1;
            v = v < v_max ? v : v_max;
            const float4 x = load4(a.z + ((long)i * a.R + v));
            return f32x4{x.x, x.y, x.z, x.w};
        } else {
            return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(zbuf(ib, pc >> 2), zoff[pc & 3], 0, 0));
        }
    };

    // One k step.  A wave issues in order, and a memory request that finds the request queue full
    // holds up the MFMAs behind it, so the step's NREQ requests are spread between its 4 NV NB MFMAs
    // (ahead of every sixteenth of them but the first) instead of being issued in a burst.
    constexpr auto group_of = [](int r) { return 1 + r * 15 / NREQ; };
    constexpr int NEARLY = [] { int n = 0; for (int r = 0; r < NREQ; ++r) n += 1 + r * 15 / NREQ < 12; return n; }();
    // The workgroup meets three quarters into the step: the next step's operands (requested a step ago) are there by
    // then, every wave has read its last fragments of this step, and the last quarter reads the next step's first ones
    // behind its MFMAs (meeting at the end of a step, these reads are in nobody's shadow: four waves fetch 8 KiB each).
    auto step = [&](auto par_c, auto role_c, const u32x4 *cur, const u32x4 *next, u32x4 *after) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_c)::value;   // st % 3: activation stage and weight register set
        constexpr int NS = (PAR + 2) % TG_DEPTH;      // set and stage (`after`) of step st + 2
        // 0: the operands of the step after next are still to request, 1: second to last step,
        // 2: last step
        constexpr int role = decltype(role_c)::value;
        // (`after` was last read one step ago and every wave has met the others since;
        //  past the end the last step is re-fetched, never used)
#pragma unroll
        for (int ph = 0; ph < 4; ++ph) {               // phase: 32 k (ph / 2), rows 16 (ph % 2) .. of every row block
            // (all of this phase's fragments are there, the last of them requested a quarter of a phase ago; without this
            //  wait the compiler waits for every LDS read, the youngest among them, ahead of each use)
            __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0)
            if (ph == 3) {
                // the next step's operands are there once at most the requests of this step's groups 1..11 are pending
                // (8 logit pieces in the second to last step, none there in the partial-sum kernel)
                constexpr int NP = role == 0 ? NEARLY : (EPI == EPI_LM ? 8 : 0);
                static_assert(NP < 16);
                if constexpr (role < 2) __builtin_amdgcn_s_waitcnt(0x0F70 | NP);       // vmcnt(NP)
                tg_barrier();
            }
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int c = ph * 4 + g4;             // group 0..15
                if constexpr (role == 0) {
#pragma unroll
                    for (int r = 0; r < NREQ; ++r)
                        if (group_of(r) == c) request(areg[NS], after, kbw_n, bp_n, r);
                } else if constexpr (EPI == EPI_LM) {
                    if (c >= 1 && c <= 8) {            // second to last step: slice 0; last step: slice 1
                        if constexpr (role == 1) zc[0][c - 1] = zpiece(0, c - 1);
                        else if constexpr (ZE == 2) zc[1][c - 1] = zpiece(1, c - 1);
                    }
                }
#pragma unroll
                for (int ib = NBQ * g4; ib < NBQ * (g4 + 1); ++ib)
                    if (ib < NB) {
                        if (ph < 3) bf[(ph + 1) & 1][ib] = cur[(((ph + 1) >> 1) * 2 * NB + ib) * 64 + 16 * ((ph + 1) & 1) + frag_x];
                        else if (role < 2) bf[0][ib] = next[ib * 64 + frag_x];
                    }
                __builtin_amdgcn_sched_barrier(0);
                // this group's share of the phase's NV NB, in an order in which successive ones share an operand (the
                // matrix cores run against the power limit: 1.90 PFLOP/s in a loop of LDS reads and MFMAs, 1.86 with the
                // weight fragments in the same order every time)
#pragma unroll
                for (int m = g4 * NV * NB / 4; m < (g4 + 1) * NV * NB / 4; ++m) {
                    const int ib = m / NV, q = ib & 1 ? NV - 1 - m % NV : m % NV;
                    if constexpr (LO) {
                        if (ph >= 2) mma_frag<EPI, true>(low[q][ib][ph & 1], areg[PAR][0][q], bf[ph & 1][ib]);
                        else mma_frag<EPI>(acc[q][ib][ph & 1], areg[PAR][0][q], bf[ph & 1][ib]);
                    } else {
                        mma_frag<EPI>(acc[q][ib][ph & 1], areg[PAR][P2 ? 0 : ph >> 1][q], bf[ph & 1][ib]);
                    }
                }
                if (c == 0 && role == 0) {   // behind the first MFMAs: where the operands of the step after next are
                    cursor_get(kbw_n, bp_n);
                    cursor_next();
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    {
        using P0 = std::integral_constant<int, 0>;
        using P1 = std::integral_constant<int, 1>;
        using P2_ = std::integral_constant<int, 2>;
        for (int left = nsteps; left >= TG_DEPTH + 2; left -= TG_DEPTH) {
            step(P0{}, P0{}, tg_stage0, tg_stage1, tg_stage2);
            step(P1{}, P0{}, tg_stage1, tg_stage2, tg_stage0);
            step(P2_{}, P0{}, tg_stage2, tg_stage0, tg_stage1);
        }
        // the last REM steps (second argument: 0 ordinary, 1 second to last, 2 last)
        if constexpr (REM == 2) {
            step(P0{}, P1{}, tg_stage0, tg_stage1, tg_stage2);
            step(P1{}, P2_{}, tg_stage1, tg_stage2, tg_stage0);
        } else if constexpr (REM == 3) {
            step(P0{}, P0{}, tg_stage0, tg_stage1, tg_stage2);
            step(P1{}, P1{}, tg_stage1, tg_stage2, tg_stage0);
            step(P2_{}, P2_{}, tg_stage2, tg_stage0, tg_stage1);
        } else {
            step(P0{}, P0{}, tg_stage0, tg_stage1, tg_stage2);
            step(P1{}, P0{}, tg_stage1, tg_stage2, tg_stage0);
            step(P2_{}, P1{}, tg_stage2, tg_stage0, tg_stage1);
            step(P0{}, P2_{}, tg_stage0, tg_stage1, tg_stage2);
        }
    }

    // ---- epilogue ----
    // (an MFMA's result may be read 18 cycles after it was issued at the earliest; the compiler does not see the MFMAs)
    asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                asm volatile("" : "+a"(acc[q][ib][hi]));
                if constexpr (LO) {
                    asm volatile("" : "+v"(low[q][ib][hi]));
                    acc[q][ib][hi] += low[q][ib][hi];
                }
            }
    // (an opaque zero keeps the compiler from sharing the prologue's 64 tile addresses with
    // the epilogue, which would hold them in registers across the whole k loop)
    int opq = 0;
    asm volatile("" : "+v"(opq));
    const int lne = ln + opq;
    if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int i = (ib0 + ib) * 32 + 16 * hi + lne;
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const int r = rw0 + 16 * q + 4 * lq;
                    if (i < row_lim && r < a.R)
                        *reinterpret_cast<f32x4 *>(a.out + ((size_t)ks * a.M + i) * a.R + r) = acc[q][ib][hi];
                }
            }
    } else if constexpr (EPI == EPI_SILU) {
        // s = SiLU(tile) written as the two fp16 planes of the next GEMM's activation: a lane holds 4 of the
        // 8 features of a 16-byte chunk (the lane ^ 16 holds the other 4), so it stores 8 bytes per plane;
        // the 64 lanes' pieces of one (q, ib, hi) are two runs of 256 contiguous bytes
        uint2 *planes = reinterpret_cast<uint2 *>(a.planes);
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int i = (ib0 + ib) * 32 + 16 * hi + lne;
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const int c8 = rw0 / 8 + 2 * q + (lq >> 1);
                    if (i < row_lim && c8 * 8 < a.R) {
                        uint16_t h[4], l[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float x = acc[q][ib][hi][e];
                            split2(x / (1.0f + expf(-x)), h[e], l[e]);
                        }
                        const size_t o = 2 * act_chunk_index(i, c8, a.nIb) + (lq & 1);
                        planes[o] = make_uint2(pack2(h[0], h[1]), pack2(h[2], h[3]));
                        planes[o + 2 * a.plane_stride] = make_uint2(pack2(l[0], l[1]), pack2(l[2], l[3]));
                    }
                }
            }
    } else {
        // per wave: 32 NB activation rows x 64 vocabulary entries.  The logit tile is added here, one
        // 32-row slice (32 registers) at a time; the row reduction over v runs in registers: the maximum of a row's 64
        // entries first (they lie in four lanes), then the sum of exponentials against it.
        // (A lane's 256 entries cost 9.5 vector instructions each, an exponential counted as four, and a tile 5 of its
        // 115 us. Before, with a branch for every piece and the index of the maximum kept: LM head of 4096 rows, d = 4096, 4250 us, now
        // 4205; of 1024 rows 1125 / 1112; of 192 rows, V = 50257, d = 2048, 60.8 / 59.1. Non-temporal pieces: 4330.)
        float *red_m = reinterpret_cast<float *>(tg_stage0);       // [4 waves][256 rows] (the stages are dead)
        float *red_s = red_m + 1024;
        const bool row_end = !RAG && rw0 + 64 > a.R;       // (uniform over the wave) the rows end among its entries
        // The first ZE slices were requested during the last two k steps; ZD - 1 slices are kept in flight
        // ahead of the one being added; the sum is formed in place in the fetched registers.
        auto zfetch = [&](int ib, f32x4 (&dst)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int pc = 0; pc < 8; ++pc) dst[pc] = zpiece(ib, pc);
        };
#pragma unroll
        for (int n = ZE; n < ZD - 1; ++n) zfetch(n, zc[n]);
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {
            if (ib + ZD - 1 >= ZE && ib + ZD - 1 < NB) zfetch(ib + ZD - 1, zc[(ib + ZD - 1) % ZD]);
            f32x4(&xs)[8] = zc[ib % ZD];
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int i = (ib0 + ib) * 32 + 16 * hi + lne;
                float m = -INFINITY;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int v = rw0 + 16 * q + 4 * lq;
                    f32x4 &x4 = xs[4 * hi + q];
                    if constexpr (RAG) {
                        if (v + 4 > a.R) {      // the piece with the end of the row (or past it): entry by entry
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                x4[e] = 0.f;
                                if (i < row_lim && v + e < a.R) x4[e] = a.z[(size_t)i * a.R + v + e];
                            }
                        }
                    }
                    x4 += acc[q][ib][hi];
                    if constexpr (RAG) {
                        if (v + 4 <= a.R) {
                            if (i < row_lim) store4(a.z + (size_t)i * a.R + v, make_float4(x4[0], x4[1], x4[2], x4[3]));
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                if (i < row_lim && v + e < a.R) a.z[(size_t)i * a.R + v + e] = x4[e];
                                if (v + e >= a.R) x4[e] = -INFINITY;      // no part of the row
                            }
                        }
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x4), zbuf(ib, hi), zoff[q], 0, 0);
                    }
                }
                if (row_end) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        asm volatile("" : "+v"(xs[4 * hi + q]));      // (kept a branch: as selects this would cost every tile)
                        if (zv_lane + 16 * q >= a.R) xs[4 * hi + q] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 x4 = xs[4 * hi + q];
                    m = max3(max3(m, x4[0], x4[1]), x4[2], x4[3]);
                }
                m = row_combine(m, [](float x, float y) { return max3(x, y, y); });
                float sum = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 x4 = xs[4 * hi + q];
                    sum += (__expf(x4[0] - m) + __expf(x4[1] - m)) + (__expf(x4[2] - m) + __expf(x4[3] - m));
                }
                sum = row_combine(sum, [](float x, float y) { return x + y; });
                if (lq == 0) {
                    const int row = 32 * ib + 16 * hi + lne;
                    red_m[wave * 256 + row] = m;
                    red_s[wave * 256 + row] = sum;
                }
            }
        }
        __syncthreads();
        if (tid < 32 * NB) {
            Part pt = {red_m[tid], red_s[tid], 0};
#pragma unroll
            for (int w = 1; w < 4; ++w) pt = part_merge(pt, Part{red_m[w * 256 + tid], red_s[w * 256 + tid], 0});
            const int i = ib0 * 32 + tid;
            if (i < row_lim) {
                a.pm[(size_t)vt * a.M + i] = pt.m;
                a.ps[(size_t)vt * a.M + i] = pt.s;
            }
        }
    }
}

// The tiles in an order where 32 consecutive ones are a block of up to 4 (activation) x 8 (weight) tiles go to
// the XCDs 32 at a time in turn; what is left after the last whole turn of all eight is dealt out evenly.  (The
// k parts of a split follow each other, so that few tiles still spread over all XCDs.)
// HALVES: left-over tiles that fill at most half a turn are dealt out as halves of their rows, so that the last round
// takes half as long (a form of its own: with both bodies in one kernel the whole tiles are up to 2.7 % slower). LM head,
// whole / halved, us: d = 4096, V = 151936: 338 / 326 at 192 rows, 378 / 357 at 256, 1128 / 1112 at 1024 (9.3 turns),
// 4261 / 4232 at 4096 (37.1); d = 2048: 222 / 210 at 256; V = 8192, d = 4096: 94 / 65 at 512 (64 tiles); V = 32000, d = 1024: 27.4 / 22
// at 144 (125 tiles).
template <int EPI, int REM, bool RAG, int NB, int NV, bool P2, bool HALVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void tiled_gemm_kernel(
    const TiledGemmArgs a) {
    const int x = blockIdx.x & 7, s = blockIdx.x >> 3, T = a.nMt * a.nVt, total = T * a.nKs;
    const int turns = total >> 8, left = total & 255, s_left = s - 32 * turns;
    const int units = HALVES ? 2 * left : left, per = (units + 7) >> 3, unit = x * per + s_left;
    if (s_left >= 0 && (s_left >= per || unit >= units)) return;
    const int id = s_left < 0 ? ((s >> 5) * 8 + x) * 32 + (s & 31) : 256 * turns + (HALVES ? unit >> 1 : unit);
    const int ks = id / T, tl = id - ks * T;
    const int vchunk = tl / (8 * a.nMt), in_chunk = tl - vchunk * 8 * a.nMt;
    const int v_cnt = a.nVt - 8 * vchunk < 8 ? a.nVt - 8 * vchunk : 8;
    const int mgrp = in_chunk / (4 * v_cnt), in_grp = in_chunk - mgrp * 4 * v_cnt;
    const int m_cnt = a.nMt - 4 * mgrp < 4 ? a.nMt - 4 * mgrp : 4;
    const int vt = vchunk * 8 + in_grp / m_cnt, mt = mgrp * 4 + in_grp % m_cnt;
    if constexpr (HALVES) {
        if (s_left >= 0) {
            constexpr int H = (NB + 1) / 2;
            const int ib0 = mt * NB + (unit & 1) * H, end = 32 * (mt * NB + NB), row_lim = end < a.M ? end : a.M;
            if (32 * ib0 < row_lim) tile_body<EPI, REM, RAG, H, NV, P2>(a, vt, ib0, ks, row_lim);
            return;
        }
    }
    tile_body<EPI, REM, RAG, NB, NV, P2>(a, vt, mt * NB, ks, a.M);
}

template <int EPI, bool RAG, int NB, int NV, bool P2, bool HALVES = false>
hipError_t launch_inst(const TiledGemmArgs &a, int rem, hipStream_t st) {
    const int total = a.nMt * a.nVt * a.nKs, units = total % 256 * (HALVES ? 2 : 1);
    const dim3 grid(8 * (total / 256 * 32 + (units + 7) / 8)), block(256);
    if (rem == 2) hipLaunchKernelGGL((tiled_gemm_kernel<EPI, 2, RAG, NB, NV, P2, HALVES>), grid, block, 0, st, a);
    else if (rem == 3) hipLaunchKernelGGL((tiled_gemm_kernel<EPI, 3, RAG, NB, NV, P2, HALVES>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((tiled_gemm_kernel<EPI, 4, RAG, NB, NV, P2, HALVES>), grid, block, 0, st, a);
    return hipGetLastError();
}

// EPI_LM: a row that is no whole number of pieces has its own form (the handling of its end costs registers, and with
// them four of the five logit slices in flight; the other one's byte offsets inside 16 rows are 32 bits)
template <int NB, bool HALVES>
hipError_t launch_lm_nb(const TiledGemmArgs &a, int rem, hipStream_t st) {
    return a.R % 4 || a.R > (1 << 26) - 64 ? launch_inst<EPI_LM, true, NB, 4, false, HALVES>(a, rem, st)
                                    : launch_inst<EPI_LM, false, NB, 4, false, HALVES>(a, rem, st);
}
template <bool HALVES>
hipError_t launch_lm(const TiledGemmArgs &a, int nb, int rem, hipStream_t st) {
    if (nb == 5) return launch_lm_nb<5, HALVES>(a, rem, st);
    if (nb == 6) return launch_lm_nb<6, HALVES>(a, rem, st);
    if (nb == 7) return launch_lm_nb<7, HALVES>(a, rem, st);
    return launch_lm_nb<8, HALVES>(a, rem, st);
}

}  // namespace

}  // namespace mrp
