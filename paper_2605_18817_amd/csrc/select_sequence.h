// The decision of one sequence at one state, by a whole workgroup: merge of its rows' partials into (token,
// confidence, log-sum-exp), reveal / draft / remask (see select.hip).
#pragma once
#include "mrp_kernels.h"

#include <type_traits>

namespace mrp {

namespace {

__device__ __forceinline__ Part wave_merge(Part p) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Part o;
        o.m = __shfl_xor(p.m, off);
        o.s = __shfl_xor(p.s, off);
        o.i = __shfl_xor(p.i, off);
        p = part_merge(p, o);
    }
    return p;
}

constexpr int TILE_V = 256;      // vocabulary entries per tile of the tile kernel

// All NT threads call.  Returns the token that conditions the next head (as it stands: it may be the caller's and out of
// range).
// MERGE_BATCH: most strides of 64 partials fetched together.
template <int NT, int MERGE_BATCH>
__device__ __forceinline__ int merge_select_sequence(const SelectArgs &a, int b) {
    constexpr int NW = NT / 64;
    __shared__ float s_conf[MAX_L], s_lse[MAX_L];
    __shared__ int s_tok[MAX_L], s_xtok[MAX_L];
    __shared__ uint8_t s_mk[MAX_L];
    __shared__ int8_t s_ra[MAX_L];
    __shared__ int s_gather;
    const int L = a.L;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    // state of the sequence: fetched up front so that its latency hides behind the merge
    int in_cond = 0, in_prot = -1;
    if (threadIdx.x < L) {
        s_mk[threadIdx.x] = a.fresh ? (uint8_t)1 : a.masked[b * L + threadIdx.x];
        s_ra[threadIdx.x] = a.fresh ? (int8_t)-1 : a.revealed_at[b * L + threadIdx.x];
        s_xtok[threadIdx.x] = (a.x_tok && !a.fresh) ? a.x_tok[b * L + threadIdx.x] : -1;
    }
    if (threadIdx.x == 0) {
        in_cond = a.cond_tok[b];
        in_prot = a.write_protect ? -1 : a.protect_pos[b];
    }

    if (a.row_stride == 1 && a.slot_stride > 1) {
        // Layout [tile][row] (the GEMM kernel that owns whole row tiles writes it, without indices): the sequence's L
        // rows of one tile are contiguous.  Thread (row p, group grp) merges tiles grp, grp + NG, ...
        // in order, so a load instruction fetches whole 4 L-byte runs; the groups' results are then
        // merged per row, first inside each wavefront, then over the wavefronts in order.
        __shared__ Part g_part[NW][MAX_L];
        __shared__ float s_max[MAX_L];
        int Lp = 1;
        while (Lp < L) Lp <<= 1;
        const int NG = NT / Lp, p = threadIdx.x % Lp, grp = threadIdx.x / Lp;
        Part pt = part_identity();
        if (p < L) {
            const size_t i = (size_t)b * L + p;
            for (int t0 = grp; t0 < a.nT; t0 += NG * 8) {
                float m[8], sx[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {   // eight tiles in flight
                    const int t = t0 + u * NG;
                    const bool ok = t < a.nT;
                    const size_t o = (size_t)(ok ? t : 0) * a.slot_stride + i;
                    m[u] = ok ? a.pm[o] : -INFINITY;
                    sx[u] = ok ? a.ps[o] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) pt = part_merge(pt, Part{m[u], sx[u], t0 + u * NG});
            }
        }
        for (int o = Lp; o < 64; o <<= 1) {      // (lanes o apart hold the same row)
            Part other;
            other.m = __shfl_xor(pt.m, o);
            other.s = __shfl_xor(pt.s, o);
            other.i = __shfl_xor(pt.i, o);
            pt = part_merge(pt, other);
        }
        if (lane < Lp) g_part[wave][p] = pt;
        __syncthreads();
        if (threadIdx.x < L) {
            const int q = threadIdx.x;
            Part r = part_identity();
#pragma unroll
            for (int w = 0; w < NW; ++w) r = part_merge(r, g_part[w][q]);
            const int i = b * L + q;
            const float conf = 1.0f / r.s;
            const float lse = r.m + logf(r.s);
            a.conf[i] = conf; a.lse[i] = lse;
            s_lse[q] = lse; s_conf[q] = conf; s_tok[q] = r.i; s_max[q] = r.m;
        }
        __syncthreads();
        // the lowest entry of the winning tile that is the maximum: one wavefront per row, 4 of the tile's 256 entries per
        // lane (a row of a single wavefront's lanes each; the tile kernel would spend 2 of its 11 vector instructions per
        // entry on keeping it)
        for (int q = wave; q < L; q += NW) {
            const float mx = s_max[q];
            const int i = b * L + q, v = s_tok[q] * TILE_V + 4 * lane;
            int at = 0x7fffffff;
            if (mx > -INFINITY) {
                const float4 x = load4_row(a.z + (size_t)i * a.V, v, a.V, -INFINITY);
                at = x.x == mx ? v : (x.y == mx ? v + 1 : (x.z == mx ? v + 2 : (x.w == mx ? v + 3 : at)));
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const int other = __shfl_xor(at, off);
                at = other < at ? other : at;
            }
            if (lane == 0) { a.tok[i] = at; s_tok[q] = at; }
        }
    } else {
    // one wavefront per row: merge the row's nT partials in a fixed order, as many strides of 64 together as there are (the
    // loads and merges of strides that hold none are not free: 256 partials in batches of 16 strides make a launch of one
    // sequence 5.2 us, in batches of 4 3.9; of 32 sequences 7.4 and 6.1)
    for (int p = wave; p < L; p += NW) {
        const int i = b * L + p;
        Part pt = part_identity();
        auto batch = [&](auto strides, int t0) __attribute__((always_inline)) {
            constexpr int N = decltype(strides)::value;
            float m[N], sx[N];
            int ix[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {  // issue every load of the batch before merging any
                const int t = t0 + u * 64 + lane;
                const bool ok = t < a.nT;
                const size_t o = (size_t)(ok ? t : 0) * a.slot_stride + (size_t)i * a.row_stride;
                m[u] = ok ? a.pm[o] : -INFINITY;
                sx[u] = ok ? a.ps[o] : 0.f;
                ix[u] = ok ? a.pi[o] : 0x7fffffff;
            }
#pragma unroll
            for (int u = 0; u < N; ++u) pt = part_merge(pt, Part{m[u], sx[u], ix[u]});
        };
        if constexpr (MERGE_BATCH > 4) {
            if (a.nT <= 64) batch(std::integral_constant<int, 1>{}, 0);
            else if (a.nT <= 256) batch(std::integral_constant<int, 4>{}, 0);
            else
                for (int t0 = 0; t0 < a.nT; t0 += 64 * MERGE_BATCH) batch(std::integral_constant<int, MERGE_BATCH>{}, t0);
        } else {
            for (int t0 = 0; t0 < a.nT; t0 += 64 * MERGE_BATCH) batch(std::integral_constant<int, MERGE_BATCH>{}, t0);
        }
        pt = wave_merge(pt);
        if (lane == 0) {
            const float conf = 1.0f / pt.s;
            a.tok[i] = pt.i;
            a.conf[i] = conf;
            const float lse = pt.m + logf(pt.s);
            a.lse[i] = lse;
            s_lse[p] = lse;
            s_conf[p] = conf;
            s_tok[p] = pt.i;
        }
    }
    }
    __syncthreads();

    // The decision of the state, one lane per position (L <= 64: the first wavefront).  A still-masked
    // position's rank is the number of still-masked positions that are more confident (ties: lower
    // position first), so "the ns most confident" are the positions of rank < ns; the number above the
    // threshold, the cap and the forced minimum are counted with ballots.  Same outcome as sorting the
    // candidates and walking the sorted list, without a serial part.
    if (wave == 0) {
        const int p = lane;
        const bool in = p < L;
        bool mk = in && s_mk[in ? p : 0] != 0;
        const float cf = in ? s_conf[p] : 0.f;
        int ra = in ? (int)s_ra[p] : -1;
        int xt = in ? s_xtok[p] : -1;
        in_cond = __shfl(in_cond, 0);
        in_prot = __shfl(in_prot, 0);
        int dpos = -1, dtok = -1, cond = in_cond, prot = in_prot;
        if (a.do_reveal) {
            int rank = 0;
            for (int q = 0; q < L; ++q) {
                const float cq = s_conf[q];
                if (s_mk[q] && (cq > cf || (cq == cf && q < p))) ++rank;
            }
            const int nc = __popcll(__ballot(mk));
            int ns = __popcll(__ballot(mk && cf > a.tau));
            if (a.max_accept) {
                int m = (7 * nc) / 10;
                if (m < 5) m = 5;
                if (m > L) m = L;
                if (ns > m) ns = m;
            }
            if (ns < a.r_min) ns = a.r_min < nc ? a.r_min : nc;
            const unsigned long long top = __ballot(mk && rank == 0);
            if (ns > 0) {
                dpos = __ffsll((long long)top) - 1;
                dtok = s_tok[dpos];
                cond = dtok;
                if (lane == 0) a.cond_tok[b] = dtok;
            }
            if (mk && rank < ns) { mk = false; ra = a.state; xt = s_tok[p]; }
            if (a.write_protect) {
                prot = dpos;
                if (lane == 0) a.protect_pos[b] = dpos;
            }
        }
        if (lane == 0) {
            a.draft_pos[(size_t)b * a.draft_stride] = dpos;
            a.draft_tok[(size_t)b * a.draft_stride] = dtok;
            s_gather = cond;
        }
        uint8_t rem = 0;
        if (in && a.tau_remask >= 0.f) {
            float cr = cf;
            if (a.remask_mode == 1 && ra >= 0 && ra <= a.state - 1) {
                // probability of the token that was revealed here under the updated logits
                int t = xt;
                if (t >= a.V && a.err_flag) atomicOr(a.err_flag, ERR_X_TOK);
                t = t < 0 ? 0 : (t >= a.V ? a.V - 1 : t);
                cr = (xt >= 0) ? expf(a.z[(size_t)(b * L + p) * a.V + t] - s_lse[p]) : 0.f;
            }
            if (ra >= 0 && ra <= a.state - 1 && p != prot && cr < a.tau_remask) {
                mk = true; ra = -1; rem = 1;
            }
        }
        if (in) {
            a.masked[b * L + p] = mk ? 1 : 0;
            a.revealed_at[b * L + p] = (int8_t)ra;
            if (a.remasked) a.remasked[b * L + p] = rem;
            if (a.x_tok) a.x_tok[b * L + p] = xt;
        }
    }
    __syncthreads();
    return s_gather;
}

}  // namespace

}  // namespace mrp
