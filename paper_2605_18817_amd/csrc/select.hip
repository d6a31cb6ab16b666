// Vocabulary reductions and the per-sequence decision logic of the MRP chain:
//   reduce_rows    state 0: split-vocabulary (max, sum-exp, argmax) partials of z
//   merge_select   merge a row's partials into (token, confidence, log-sum-exp)
//                  — confidence is the top-1 softmax probability (paper
//                  Section 2) — then, one workgroup per sequence, apply the
//                  reveal rule (threshold with a forced minimum, Section 4.1;
//                  optional max-accept cap, Section 4.4), record the draft
//                  (Algorithm 3: most confident new reveal), optionally remask
//                  (Algorithm 4) and gather the embedding row that conditions
//                  the next head
//   remask         Algorithm 4's remask rule on its own
//   verify         Algorithm 3's accept test: argmax of the verifier's logits at
//                  the drafted positions, longest matching prefix
#include "select_sequence.h"

namespace mrp {

namespace {

constexpr int RT = 8192;  // vocabulary entries per workgroup in the plain row reductions

// all 256 threads call; result valid in thread 0
__device__ __forceinline__ Part block_merge(Part p, float *sm, float *ss, int *si) {
    p = wave_merge(p);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sm[wave] = p.m; ss[wave] = p.s; si[wave] = p.i; }
    __syncthreads();
    if (threadIdx.x == 0) {
        p = Part{sm[0], ss[0], si[0]};
        for (int w = 1; w < 4; ++w) p = part_merge(p, Part{sm[w], ss[w], si[w]});
    }
    return p;
}

// Grid: the row tiles of z; past its M rows the units of `init` (its M is 0: none), which need nothing of z and would
// otherwise be a launch of their own (5 us at 4 to 200 rows).
__global__ __launch_bounds__(256) void reduce_rows_kernel(const float *__restrict__ z, int M, int V,
                                                          float *__restrict__ pm, float *__restrict__ ps,
                                                          int *__restrict__ pi, const InitHiddenArgs init) {
    __shared__ float sm[4], ss[4];
    __shared__ int si[4];
    const int t = blockIdx.x, i = blockIdx.y;
    if (i >= M) {
        init_hidden_unit(init, ((size_t)(i - M) * gridDim.x + t) * 4 + (threadIdx.x >> 6));
        return;
    }
    const float *row = z + (size_t)i * V;
    const int v0 = t * RT;
    float x[32];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const float4 q = load4_row(row, v0 + 4 * (threadIdx.x + 256 * n), V, -INFINITY);
        x[4 * n] = q.x; x[4 * n + 1] = q.y; x[4 * n + 2] = q.z; x[4 * n + 3] = q.w;
    }
    Part p = part_identity();
#pragma unroll
    for (int n = 0; n < 32; ++n) {
        const int v = v0 + 4 * (threadIdx.x + 256 * (n >> 2)) + (n & 3);
        if (x[n] > p.m) { p.m = x[n]; p.i = v; }
    }
    float s = 0.f;
    if (p.m > -INFINITY) {
#pragma unroll
        for (int n = 0; n < 32; ++n) s += __expf(x[n] - p.m);  // exp(-inf) = 0 for padding
    }
    p.s = s;
    p = block_merge(p, sm, ss, si);
    if (threadIdx.x == 0) {
        // a row's partials are contiguous, so that the merge reads them coalesced
        const size_t o = (size_t)i * gridDim.x + t;
        pm[o] = p.m;
        ps[o] = p.s;
        pi[o] = p.i;
    }
}

// One workgroup per sequence.  What bounds it is latency (partials, decision and gather follow each other), so the
// workgroup is wide enough that the merge is one round of loads: 1024 threads, or 256 where four wavefronts already
// hold a row each.
template <int NT>
__global__ __launch_bounds__(NT) void merge_select_kernel(const SelectArgs a) {
    const int b = blockIdx.x, L = a.L;
    const int cond = merge_select_sequence<NT, 16>(a, b);
    if (a.E != nullptr) {  // embedding row that conditions the next head
        const int C8 = a.d >> 3;
        int tokc = cond;  // caller contract: 0 <= cond_tok < V; a bad value is clamped and reported
        if ((tokc < 0 || tokc >= a.V) && threadIdx.x == 0 && a.err_flag) atomicOr(a.err_flag, ERR_COND_TOK);
        tokc = tokc < 0 ? 0 : (tokc >= a.V ? a.V - 1 : tokc);
        const uint4 *erow = reinterpret_cast<const uint4 *>(a.E + (size_t)tokc * a.d);
        for (int n = threadIdx.x; n < C8 * L; n += NT) {   // a plane's rows of one chunk are contiguous
            const int c8 = n / L, p = n - c8 * L;
            a.xe[act_chunk_index(b * L + p, c8, a.nIb)] = bf16x8_to_f16x8(erow[c8]);   // the head body's operands are fp16
        }
    }
}

// End of a denoising step: commit this step's reveals (one workgroup per sequence, one lane per row).
__global__ __launch_bounds__(64) void commit_kernel(int L, const int32_t *__restrict__ x_tok,
                                                    int8_t *__restrict__ revealed_at,
                                                    const uint8_t *__restrict__ masked, int32_t *__restrict__ x_out,
                                                    int32_t *__restrict__ n_masked) {
    const int b = blockIdx.x, p = threadIdx.x;
    int m = 0;
    if (p < L) {
        const int i = b * L + p;
        if (revealed_at[i] >= 0) {
            x_out[i] = x_tok[i];
            revealed_at[i] = -2;
        }
        m = masked[i] ? 1 : 0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m += __shfl_xor(m, off);
    if (p == 0) n_masked[b] = m;
}

__global__ __launch_bounds__(64) void remask_kernel(int B, int L, int state, const float *__restrict__ conf,
                                                    float tau_remask, const int32_t *__restrict__ protect_pos,
                                                    int8_t *__restrict__ revealed_at, uint8_t *__restrict__ masked,
                                                    uint8_t *__restrict__ remasked) {
    const int b = blockIdx.x, p = threadIdx.x;
    if (p >= L) return;
    const int i = b * L + p;
    const int prot = protect_pos ? protect_pos[b] : -1;
    const int r = revealed_at[i];
    uint8_t rem = 0;
    if (r >= 0 && r <= state - 1 && p != prot && conf[i] < tau_remask) {
        masked[i] = 1;
        revealed_at[i] = -1;
        rem = 1;
    }
    remasked[i] = rem;
}

// argmax partial of one RT-wide chunk of the verifier row of draft (b, j)
__global__ __launch_bounds__(256) void verify_argmax_kernel(int L, int V, int K, int joint,
                                                            const float *__restrict__ verify,
                                                            const int32_t *__restrict__ draft_pos, int draft_stride,
                                                            int nC, float *__restrict__ wm, int *__restrict__ wi,
                                                            int *err_flag) {
    __shared__ float sm[4], ss[4];
    __shared__ int si[4];
    const int c = blockIdx.x, bk = blockIdx.y;
    const int b = bk / K, j = bk % K;
    int pos = draft_pos[(size_t)b * draft_stride + j];
    if (pos >= L) {  // caller contract: pos < L; an invalid position counts as a missing draft and is reported
        if (threadIdx.x == 0 && c == 0 && err_flag) atomicOr(err_flag, ERR_DRAFT_POS);
        pos = -1;
    }
    Part p = part_identity();
    if (pos >= 0) {  // uniform over the workgroup
        // joint: [B][K+1][L][V], draft j reads candidate j; else one [B][L][V] tensor
        const size_t blk = joint ? (size_t)b * (K + 1) + j : (size_t)b;
        const float *row = verify + (blk * L + pos) * V;
        const int v0 = c * RT;
        float4 q[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) q[n] = load4_row(row, v0 + 4 * (threadIdx.x + 256 * n), V, -INFINITY);
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int v = v0 + 4 * (threadIdx.x + 256 * n);
            if (q[n].x > p.m) { p.m = q[n].x; p.i = v; }
            if (q[n].y > p.m) { p.m = q[n].y; p.i = v + 1; }
            if (q[n].z > p.m) { p.m = q[n].z; p.i = v + 2; }
            if (q[n].w > p.m) { p.m = q[n].w; p.i = v + 3; }
        }
    }
    p = block_merge(p, sm, ss, si);
    if (threadIdx.x == 0) {
        wm[(size_t)bk * nC + c] = p.m;
        wi[(size_t)bk * nC + c] = (pos >= 0) ? p.i : -1;
    }
}

// Accept test of one sequence, one wavefront each.  What bounds it is latency: the nC partials of a draft are
// contiguous, so the lanes fetch them (and those of VB drafts) in one round trip and merge them across lanes; equal
// maxima keep the lower index, as in a walk over the chunks.  One thread per sequence, walking drafts and chunks
// serially, took 15.6 us for 128 sequences x 3 drafts x 19 chunks; this form takes 4.
constexpr int VB = 4;   // drafts fetched together
__global__ __launch_bounds__(256) void verify_accept_kernel(int B, int K, int nC, const float *__restrict__ wm,
                                                            const int *__restrict__ wi,
                                                            const int32_t *__restrict__ draft_tok, int draft_stride,
                                                            uint8_t *__restrict__ match, int32_t *__restrict__ accept_len,
                                                            int32_t *__restrict__ correction_tok) {
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= B) return;   // (uniform over the wave)
    const int tok = lane < K ? draft_tok[(size_t)b * draft_stride + lane] : 0;   // (K <= 16)
    int alen = 0, corr = -1;
    bool open = true;
    for (int j0 = 0; j0 < K; j0 += VB) {
        float m[VB];
        int v[VB];
#pragma unroll
        for (int u = 0; u < VB; ++u) { m[u] = -INFINITY; v[u] = 0x7fffffff; }
        for (int c = lane; c < nC; c += 64) {
            float mc[VB];
            int vc[VB];
#pragma unroll
            for (int u = 0; u < VB; ++u) {   // (a draft past the last one repeats it and is not used)
                const size_t o = ((size_t)b * K + (j0 + u < K ? j0 + u : K - 1)) * nC + c;
                mc[u] = wm[o];
                vc[u] = wi[o];
            }
#pragma unroll
            for (int u = 0; u < VB; ++u)
                if (mc[u] > m[u] || (mc[u] == m[u] && vc[u] < v[u])) { m[u] = mc[u]; v[u] = vc[u]; }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                const float mo = __shfl_xor(m[u], off);
                const int vo = __shfl_xor(v[u], off);
                if (mo > m[u] || (mo == m[u] && vo < v[u])) { m[u] = mo; v[u] = vo; }
            }
#pragma unroll
        for (int u = 0; u < VB; ++u) {
            const int j = j0 + u;
            if (j < K) {
                const bool ok = v[u] >= 0 && v[u] == __shfl(tok, j);
                if (lane == 0) match[(size_t)b * K + j] = ok ? 1 : 0;
                if (open) {
                    if (ok) ++alen;
                    else { open = false; corr = v[u]; }
                }
            }
        }
    }
    if (lane == 0) {
        accept_len[b] = alen;
        correction_tok[b] = corr;
    }
}

// Candidate blocks of the joint verification (paper Figure 1 (d)): candidate k of a sequence is its
// block x_t with the first k drafts written in.  One workgroup per sequence, one lane per position.
__global__ __launch_bounds__(64) void build_candidates_kernel(int L, int K, const int32_t *__restrict__ x_t,
                                                              const uint8_t *__restrict__ masked_t,
                                                              const int32_t *__restrict__ draft_pos,
                                                              const int32_t *__restrict__ draft_tok, int draft_stride,
                                                              int32_t mask_token, int32_t *__restrict__ cand_tok,
                                                              uint8_t *__restrict__ cand_masked, int *err_flag) {
    const int b = blockIdx.x, p = threadIdx.x;
    if (p >= L) return;
    const uint8_t m0 = masked_t[(size_t)b * L + p] ? 1 : 0;
    int32_t tok = m0 ? mask_token : x_t[(size_t)b * L + p];
    uint8_t m = m0;
    for (int k = 0; k <= K; ++k) {
        if (k > 0) {   // candidate k adds draft k - 1
            const int pos = draft_pos[(size_t)b * draft_stride + k - 1];
            if (pos >= L && p == 0 && err_flag) atomicOr(err_flag, ERR_DRAFT_POS);
            if (pos == p) { tok = draft_tok[(size_t)b * draft_stride + k - 1]; m = 0; }
        }
        const size_t o = ((size_t)b * (K + 1) + k) * L + p;
        cand_tok[o] = tok;
        cand_masked[o] = m;
    }
}

}  // namespace

hipError_t launch_build_candidates(int B, int L, int K, const int32_t *x_t, const uint8_t *masked_t,
                                   const int32_t *draft_pos, const int32_t *draft_tok, int draft_stride,
                                   int32_t mask_token, int32_t *cand_tok, uint8_t *cand_masked, int *err_flag,
                                   hipStream_t st) {
    hipLaunchKernelGGL(build_candidates_kernel, dim3(B), dim3(64), 0, st, L, K, x_t, masked_t, draft_pos, draft_tok,
                       draft_stride, mask_token, cand_tok, cand_masked, err_flag);
    return hipGetLastError();
}

int reduce_rows_tiles(int V) { return (V + RT - 1) / RT; }
int verify_chunks(int V) { return (V + RT - 1) / RT; }

hipError_t launch_reduce_rows(const float *z, int M, int V, float *pm, float *ps, int *pi, int *nT_out,
                              const InitHiddenArgs *init, hipStream_t st) {
    const int nT = reduce_rows_tiles(V);
    *nT_out = nT;
    InitHiddenArgs ia = {};
    unsigned more = 0;      // grid rows for the hidden state
    if (init) {
        const unsigned rows = (plane_blocks(init->M, init->d) + nT - 1) / nT;
        if (M + rows <= 65535) { more = rows; ia = *init; }
        else {
            const hipError_t e = launch_init_hidden(*init, st);
            if (e != hipSuccess) return e;
        }
    }
    hipLaunchKernelGGL(reduce_rows_kernel, dim3(nT, M + more), dim3(256), 0, st, z, M, V, pm, ps, pi, ia);
    return hipGetLastError();
}

hipError_t launch_merge_select(const SelectArgs &a, hipStream_t st) {
    if (a.L <= 4 && a.slot_stride == 1) hipLaunchKernelGGL(merge_select_kernel<256>, dim3(a.B), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(merge_select_kernel<1024>, dim3(a.B), dim3(1024), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_commit(int B, int L, const int32_t *x_tok, int8_t *revealed_at, const uint8_t *masked,
                         int32_t *x_out, int32_t *n_masked, hipStream_t st) {
    hipLaunchKernelGGL(commit_kernel, dim3(B), dim3(64), 0, st, L, x_tok, revealed_at, masked, x_out, n_masked);
    return hipGetLastError();
}

hipError_t launch_remask(int B, int L, int state, const float *conf, float tau_remask,
                         const int32_t *protect_pos, int8_t *revealed_at, uint8_t *masked, uint8_t *remasked,
                         hipStream_t st) {
    hipLaunchKernelGGL(remask_kernel, dim3(B), dim3(64), 0, st, B, L, state, conf, tau_remask, protect_pos,
                       revealed_at, masked, remasked);
    return hipGetLastError();
}

hipError_t launch_verify(int B, int L, int V, int K, int joint, const float *verify, const int32_t *draft_pos,
                         const int32_t *draft_tok, int draft_stride, float *wm, int *wi, uint8_t *match,
                         int32_t *accept_len, int32_t *correction_tok, int *err_flag, hipStream_t st) {
    const int nC = verify_chunks(V);
    hipLaunchKernelGGL(verify_argmax_kernel, dim3(nC, B * K), dim3(256), 0, st, L, V, K, joint, verify, draft_pos,
                       draft_stride, nC, wm, wi, err_flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(verify_accept_kernel, dim3((B + 3) / 4), dim3(256), 0, st, B, K, nC, wm, wi,
                       draft_tok, draft_stride, match, accept_len, correction_tok);
    return hipGetLastError();
}

}  // namespace mrp
