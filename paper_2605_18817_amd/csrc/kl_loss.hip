// Training-side loss of the MRP head (paper Section 3.3, Equation 3): per masked row
//     L_i = KL( softmax(l_{t-1}[i]) || softmax(l_t[i] + delta_t[i]) )
// and its gradient with respect to the student logits (hence to delta_t),
//     dL_i / ds[i][v] = softmax(s[i])[v] - softmax(l_{t-1}[i])[v],
// with teacher T = l_{t-1} and student S = l_t + delta_t given as fp32 [M][V].
//
// All of it is a memory stream.  Every (row, 8192-wide vocabulary tile) keeps the online partial
//     (m_T, s_T = sum e^{T - m_T}, a_T = sum e^{T - m_T} (T - S),  m_S, s_S = sum e^{S - m_S})
// of the forward pass, and a row's partials merge to
//     L_i = a_T / s_T - (m_T + log s_T) + (m_S + log s_S).
// No softmax is written.  Algorithmic bytes: 8 M V forward, 4 M V for the gradient, which is the difference of the two
// softmaxes: taken from the entries that the forward pass left in registers (kl_grad_kernel; 1024 rows of 151936: 1.87 GB in
// 383 us, 4.9 TB/s, where a large copy moves 4.7), or from a second read: at few rows, and where a row's tiles are too many
// for the places that may wait.
#include "mrp_kernels.h"

namespace mrp {

namespace {

constexpr int KT = 8192;   // vocabulary entries per workgroup

struct KlPart {
    float mT, sT, aT, mS, sS;
};

__device__ __forceinline__ KlPart kl_identity() { return {-INFINITY, 0.f, 0.f, -INFINITY, 0.f}; }

__device__ __forceinline__ KlPart kl_merge(const KlPart &x, const KlPart &y) {
    KlPart r;
    r.mT = fmaxf(x.mT, y.mT);
    const float fx = (x.mT == -INFINITY) ? 0.f : __expf(x.mT - r.mT);
    const float fy = (y.mT == -INFINITY) ? 0.f : __expf(y.mT - r.mT);
    r.sT = x.sT * fx + y.sT * fy;
    r.aT = x.aT * fx + y.aT * fy;
    r.mS = fmaxf(x.mS, y.mS);
    const float gx = (x.mS == -INFINITY) ? 0.f : __expf(x.mS - r.mS);
    const float gy = (y.mS == -INFINITY) ? 0.f : __expf(y.mS - r.mS);
    r.sS = x.sS * gx + y.sS * gy;
    return r;
}

__device__ __forceinline__ KlPart kl_shfl_xor(const KlPart &p, int off) {
    return {__shfl_xor(p.mT, off), __shfl_xor(p.sT, off), __shfl_xor(p.aT, off), __shfl_xor(p.mS, off),
            __shfl_xor(p.sS, off)};
}

__device__ __forceinline__ KlPart kl_wave_merge(KlPart p) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) p = kl_merge(p, kl_shfl_xor(p, off));
    return p;
}

// Partials of row i, all its nT tiles: lane l merges tiles l, l + 64, ...; the result is in every lane.
// Partial (t, i) of array a lives at a[i * nT + t].
__device__ __forceinline__ KlPart kl_row(const float *__restrict__ part, size_t stride, int nT, int i) {
    KlPart p = kl_identity();
    for (int t = threadIdx.x & 63; t < nT; t += 64) {
        const size_t o = (size_t)i * nT + t;
        p = kl_merge(p, KlPart{part[o], part[stride + o], part[2 * stride + o], part[3 * stride + o], part[4 * stride + o]});
    }
    return kl_wave_merge(p);
}

struct KlArgs {
    const float *T, *S;
    const uint8_t *mask;
    int V, nT;
    float scale;
    float *part;                  // without a gradient: five arrays, `stride` apart
    unsigned long long *words;    // with one: the same as 64-bit words, mark and value
    size_t stride;
    float *loss, *grad;
    int M;
    int nq;                       // counters that the one-pass form draws from (0: two passes)
    int spin;                     // looks at a word before its tile is taken as one that nobody has room for
    int p0, nP;                   // two passes: rows p0 .. p0 + nP - 1: partials
    int g0, nG;                   // rows g0 .. g0 + nG - 1: loss and gradient (their partials are complete)
};

constexpr int MAX_Q = 7;

// The 32 entries of a tensor's row that a thread handles in tile t: eight 16-byte pieces, -inf past the row's end
__device__ __forceinline__ void kl_fetch(const float *row, int v0, int V, float4 (&x)[8]) {
#pragma unroll
    for (int n = 0; n < 8; ++n) x[n] = load4_row(row, v0 + 4 * (threadIdx.x + 256 * n), V, -INFINITY);
}
__device__ __forceinline__ float kl_at(const float4 (&x)[8], int n) {
    const float4 &q = x[n >> 2];
    return (n & 3) == 0 ? q.x : ((n & 3) == 1 ? q.y : ((n & 3) == 2 ? q.z : q.w));
}

__device__ __forceinline__ void kl_max(KlPart &p, float vt, float vs) { p.mT = fmaxf(p.mT, vt); p.mS = fmaxf(p.mS, vs); }
__device__ __forceinline__ void kl_add(KlPart &p, float vt, float vs) {
    if (vt > -INFINITY) {       // (padding past V is -inf in both tensors: skip, T - S would be NaN)
        const float e = __expf(vt - p.mT);
        p.sT += e;
        p.aT += e * (vt - vs);
        p.sS += __expf(vs - p.mS);
    }
}

// The workgroup's partial from its threads'; valid in thread 0.  sw: one slot per wavefront
__device__ __forceinline__ KlPart kl_join(KlPart p, KlPart *sw) {
    p = kl_wave_merge(p);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sw[wave] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        p = sw[0];
        for (int w = 1; w < 4; ++w) p = kl_merge(p, sw[w]);
    }
    return p;
}

// Partial of one KT-wide tile from its entries; valid in thread 0
__device__ __forceinline__ KlPart kl_tile(const float4 (&xt)[8], const float4 (&xs)[8], KlPart *sw) {
    KlPart p = kl_identity();
#pragma unroll
    for (int n = 0; n < 32; ++n) kl_max(p, kl_at(xt, n), kl_at(xs, n));
    if (p.mT > -INFINITY) {
#pragma unroll
        for (int n = 0; n < 32; ++n) kl_add(p, kl_at(xt, n), kl_at(xs, n));
    }
    return kl_join(p, sw);
}

// The same from memory, four entries at a time in the same order (few registers: the caller holds another tile)
__device__ __forceinline__ KlPart kl_tile_again(const float *T, const float *S, int v0, int V, KlPart *sw) {
    KlPart p = kl_identity();
#pragma clang loop unroll(disable)
    for (int n = 0; n < 16; ++n) {
        const int v = v0 + 4 * (threadIdx.x + 256 * (n & 7));
        const float4 x = load4_row(T, v, V, -INFINITY), y = load4_row(S, v, V, -INFINITY);
        if (n < 8) {
            kl_max(p, x.x, y.x); kl_max(p, x.y, y.y); kl_max(p, x.z, y.z); kl_max(p, x.w, y.w);
        } else if (p.mT > -INFINITY) {
            kl_add(p, x.x, y.x); kl_add(p, x.y, y.y); kl_add(p, x.z, y.z); kl_add(p, x.w, y.w);
        }
    }
    return kl_join(p, sw);
}

// partials of one KT-wide tile of one row
__device__ __forceinline__ void kl_partial(const KlArgs &a, int t, int i, KlPart *sw) {
    if (a.mask && !a.mask[i]) return;   // (uniform over the workgroup)
    float4 xt[8], xs[8];
    kl_fetch(a.T + (size_t)i * a.V, t * KT, a.V, xt);
    kl_fetch(a.S + (size_t)i * a.V, t * KT, a.V, xs);
    const KlPart p = kl_tile(xt, xs, sw);
    if (threadIdx.x == 0) {
        const size_t o = (size_t)i * a.nT + t;
        a.part[o] = p.mT; a.part[a.stride + o] = p.sT; a.part[2 * a.stride + o] = p.aT;
        a.part[3 * a.stride + o] = p.mS; a.part[4 * a.stride + o] = p.sS;
    }
}
__global__ __launch_bounds__(256) void kl_partial_kernel(const KlArgs a) {      // loss alone
    __shared__ KlPart sw[4];
    kl_partial(a, blockIdx.x, blockIdx.y, sw);
}

// Gradient of one KT-wide tile of one row from its entries; zero where the row is not in the mask
__device__ __forceinline__ void kl_write(const KlArgs &a, int t, int i, bool on, const float4 (&xt)[8], const float4 (&xs)[8],
                                         float lT, float lS) {
    float *gr = a.grad + (size_t)i * a.V;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int v = t * KT + 4 * (threadIdx.x + 256 * n);
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) {
            g.x = a.scale * (__expf(xs[n].x - lS) - __expf(xt[n].x - lT));
            g.y = a.scale * (__expf(xs[n].y - lS) - __expf(xt[n].y - lT));
            g.z = a.scale * (__expf(xs[n].z - lS) - __expf(xt[n].z - lT));
            g.w = a.scale * (__expf(xs[n].w - lS) - __expf(xt[n].w - lT));
        }
        if (v + 4 <= a.V) {
            const f32x4_any gv = {g.x, g.y, g.z, g.w};
            __builtin_nontemporal_store(gv, reinterpret_cast<f32x4_any *>(gr + v));
        } else if (v < a.V) {
            gr[v] = g.x;
            if (v + 1 < a.V) gr[v + 1] = g.y;
            if (v + 2 < a.V) gr[v + 2] = g.z;
        }
    }
}

// Loss and gradient in one pass over the tensors: a workgroup keeps its tile's entries in registers (64 per thread, four
// workgroups per CU), publishes the tile's partial, waits for the other tiles of its row and writes the gradient from
// what it holds.  A value and its mark travel in one 64-bit word, so nothing else has to be ordered; words and counters are
// cleared by a launch before.
//
// Which tile a workgroup takes is drawn from one of nq counters as it starts, so of the rows of a counter at most one has tiles
// that nobody has drawn yet.  Rows that are all drawn need nobody else and leave; the others hold at most nq (nT - 1) places, an
// eighth of the device (kl_counters).  The wait ends with fewer places, too (a device shared with kernels that stay, a
// graph replayed on a stream of fewer CUs): after `spin` looks the workgroup takes the missing partial itself, with the same
// bits, and from then on does not wait for others of the row.  (512 rows of 151936 on a device that has 32 places left: 16 ms with
// 128 looks, 24 with 512; 1050 with 8192 for each partial that is missing.  Two passes, which a stream of 8 CUs takes, 2.9.)
// It offers what it found only in words that are still empty: a tile may be overwritten with its gradient (a gradient in the
// place of the logits) once all its words are there, so what was read too late is not taken.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void kl_grad_kernel(const KlArgs a) {
    __shared__ KlPart sw[4];
    __shared__ float s_lse[2];
    __shared__ int s_draw, s_missing;
    const int lane = threadIdx.x & 63, q = blockIdx.x % a.nq;
    if (threadIdx.x == 0)
        s_draw = (int)__hip_atomic_fetch_add(a.words + 5 * a.stride + 16 * q, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int draw = __builtin_amdgcn_readfirstlane(s_draw), t = draw % a.nT, i = draw / a.nT * a.nq + q;
    if (i >= a.M) return;                     // (uniform over the workgroup, as is what follows)
    const bool on = !a.mask || a.mask[i];
    float4 xt[8], xs[8];
    float lT = 0.f, lS = 0.f;
    if (on) {
        kl_fetch(a.T + (size_t)i * a.V, t * KT, a.V, xt);
        kl_fetch(a.S + (size_t)i * a.V, t * KT, a.V, xs);
        unsigned long long *words = a.words + (size_t)i * a.nT;
        const KlPart p = kl_tile(xt, xs, sw);
        if (threadIdx.x == 0) {
            const float v[5] = {p.mT, p.sT, p.aT, p.mS, p.sS};
#pragma unroll
            for (int n = 0; n < 5; ++n)
                __hip_atomic_store(words + n * a.stride + t, (1ull << 32) | __float_as_uint(v[n]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int patience = a.spin;; patience = 0) {
            if (threadIdx.x < 64) {      // the order of kl_row
                KlPart r = kl_identity();
                int missing = -1;
                for (int u = lane; u < a.nT; u += 64) {
                    unsigned long long w[5];
                    bool all;
                    int looks = 0;
                    do {
                        all = true;
#pragma unroll
                        for (int n = 0; n < 5; ++n) {
                            w[n] = __hip_atomic_load(words + n * a.stride + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            all = all && (w[n] >> 32) != 0;
                        }
                        if (!all) __builtin_amdgcn_s_sleep(4);
                    } while (!all && ++looks < patience);
                    if (!all) missing = u;
                    float v[5];
#pragma unroll
                    for (int n = 0; n < 5; ++n) v[n] = __uint_as_float((unsigned)w[n]);
                    r = kl_merge(r, KlPart{v[0], v[1], v[2], v[3], v[4]});
                }
                const unsigned long long who = __ballot(missing >= 0);
                const int first = who ? __shfl(missing, __ffsll(who) - 1) : -1;
                r = kl_wave_merge(r);
                if (lane == 0) {
                    s_missing = first;
                    if (first < 0) {
                        const float qT = r.mT + logf(r.sT), qS = r.mS + logf(r.sS);
                        s_lse[0] = qT;
                        s_lse[1] = qS;
                        if (t == 0) a.loss[i] = a.scale * (r.aT / r.sT - qT + qS);
                    }
                }
            }
            __syncthreads();
            const int take = __builtin_amdgcn_readfirstlane(s_missing);     // (uniform over the workgroup)
            if (take < 0) break;
            const KlPart p2 = kl_tile_again(a.T + (size_t)i * a.V, a.S + (size_t)i * a.V, take * KT, a.V, sw);
            if (threadIdx.x == 0) {
                const float v[5] = {p2.mT, p2.sT, p2.aT, p2.mS, p2.sS};
#pragma unroll
                for (int n = 0; n < 5; ++n) {
                    unsigned long long none = 0;
                    __hip_atomic_compare_exchange_strong(words + n * a.stride + take, &none, (1ull << 32) | __float_as_uint(v[n]),
                                                         __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        lT = s_lse[0];
        lS = s_lse[1];
    } else if (t == 0 && threadIdx.x == 0) {
        a.loss[i] = 0.f;
    }
    kl_write(a, t, i, on, xt, xs, lT, lS);
}

// The same from a second read; tile 0 also writes the row's loss
__device__ __forceinline__ void kl_second(const KlArgs &a, int t, int i) {
    const bool on = !a.mask || a.mask[i];     // (uniform over the workgroup)
    float4 xt[8], xs[8];
    float lT = 0.f, lS = 0.f;
    if (on) {
        kl_fetch(a.T + (size_t)i * a.V, t * KT, a.V, xt);     // in flight while the row's partials are merged
        kl_fetch(a.S + (size_t)i * a.V, t * KT, a.V, xs);
        const KlPart p = kl_row(a.part, a.stride, a.nT, i);
        lT = p.mT + logf(p.sT);
        lS = p.mS + logf(p.sS);
        if (t == 0 && threadIdx.x == 0) a.loss[i] = a.scale * (p.aT / p.sT - lT + lS);
    } else if (t == 0 && threadIdx.x == 0) {
        a.loss[i] = 0.f;
    }
    kl_write(a, t, i, on, xt, xs, lT, lS);
}

// Two passes: one launch takes the partials of one group of rows and the gradient of the group before it, alternating
// while both have rows left, so that the reads of the one run beside the writes of the other.
__global__ __launch_bounds__(256) void kl_two_pass_kernel(const KlArgs a) {
    __shared__ KlPart sw[4];
    const int t = blockIdx.x, y = blockIdx.y, both = 2 * (a.nP < a.nG ? a.nP : a.nG);
    const bool part = y < both ? (y & 1) == 0 : a.nP > a.nG;
    const int r = y < both ? y >> 1 : y - both / 2;
    if (part) kl_partial(a, t, a.p0 + r, sw);
    else kl_second(a, t, a.g0 + r);
}

}  // namespace

int kl_tiles(int V) { return (V + KT - 1) / KT; }

size_t kl_part_bytes(size_t stride) { return (5 * stride + 16 * MAX_Q) * sizeof(unsigned long long); }

// Counters for the gradient of M rows of nT tiles in one pass, 0 for two passes.  What waits (counters x (nT - 1) workgroups,
// four to a CU) may hold an eighth of the device.  An odd number, so that every counter serves all eight XCDs and the rows
// read at one time lie apart differently from time to time: 1024 rows of 151936 take 408 us with one counter, 402 with 2, 391 with 3, 438 with
// 4, 387 with 5, 383 with 7, 502 with 8 (plain instead of non-temporal stores with 4: 453).
// With fewer tiles than two rounds of resident workgroups the second pass reads from the caches and costs less than clearing
// and drawing.  Measured, us, two passes (with the rows in groups that fit the last-level cache) / one: 496 / 383 at 1024 rows of
// 151936, 991 / 753 at 2048, 93 / 71 at 300 with half of them masked out, 116 / 78 at 1024 of 32000; but with 4 counters
// 35.0 / 35.7 at 64 of 151936 (1216 tiles), 12.8 / 14.1 at 16, 13.6 / 14.5 at 64 of 50257.
// Fewer CUs (a stream limited to some of them, a partition) don't draw what the memory gives, and the second read is the
// caches' for longer: two passes / one on 64 CUs 95 / 124 at 128 of 151936, 453 / 499 at 512, 156 / 174 at 1024 of 32000; on 128 CUs 68 / 76,
// 285 / 284, 122 / 105.
int kl_counters(int M, int nT, int nCU) {
    if (nCU < 128 || (long)M * nT * nCU < 2048 * 256) return 0;
    for (int nq = MAX_Q; nq > 0; nq -= 2)
        if (nq * (nT - 1) <= nCU / 2) return nq;
    return 0;
}

// Rows taken together in two passes: a group's rows are read for the partials and once more, one launch later, for the
// gradient.  What is live in between, two tensors of two groups, has to fit the 256 MB last-level cache; smaller groups
// only add launches.  Measured, us, in one group / in groups of 52 MB per tensor: 533 / 495 at 128 rows of 1.2 M (560 with 32 MB, 518
// with 40, 501 with 64), 901 / 848 at 128 of 2 M, 1059 / 1029 at 100 of 3 M (4 rows a group); but 887 / 908 at 64 of 4 M, 869 / 951 at
// 32 of 8 M.
int kl_group_rows(int M, int V) {
    constexpr size_t GROUP_BYTES = (size_t)52 << 20;
    const size_t row_bytes = V * sizeof(float), fit = GROUP_BYTES / row_bytes;
    const int rows = fit < 4 || M * row_bytes < GROUP_BYTES * 3 / 2 ? M : (int)fit;
    return rows < M && rows > 32767 ? 32767 : rows;      // (grid limit: two groups in one launch)
}

// the words' first n entries of each of the five arrays, and the counters
__global__ __launch_bounds__(256) void kl_clear_kernel(unsigned long long *words, size_t stride, int n) {
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o < n && blockIdx.y < 5) words[blockIdx.y * stride + o] = 0;
    if (o < MAX_Q && blockIdx.y == 5) words[5 * stride + 16 * o] = 0;
}

// loss alone: one wavefront per row
__global__ __launch_bounds__(256) void kl_finish_kernel(const KlArgs a, int M) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= M) return;
    float loss = 0.f;
    if (!a.mask || a.mask[i]) {
        const KlPart p = kl_row(a.part, a.stride, a.nT, i);
        loss = a.scale * (p.aT / p.sT - (p.mT + logf(p.sT)) + (p.mS + logf(p.sS)));
    }
    if ((threadIdx.x & 63) == 0) a.loss[i] = loss;
}

hipError_t launch_kl_loss(int M, int V, const float *teacher, const float *student, const uint8_t *mask, float scale,
                          float *part, size_t part_stride, float *loss_rows, float *grad, int nCU, int spin, hipStream_t st) {
    const KlArgs a = {teacher, student, mask, V, kl_tiles(V), scale, part, reinterpret_cast<unsigned long long *>(part), part_stride,
                      loss_rows, grad, M, grad ? kl_counters(M, kl_tiles(V), nCU) : 0, spin, 0, 0, 0, 0};
    if (a.nq) {
        const int n = M * a.nT;
        hipLaunchKernelGGL(kl_clear_kernel, dim3((n + 255) / 256, 6), dim3(256), 0, st, a.words, part_stride, n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kl_grad_kernel, dim3((M + a.nq - 1) / a.nq * a.nq * a.nT), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    if (grad) {
        KlArgs b = a;
        const int rows = kl_group_rows(M, V);
        for (int r0 = 0; r0 < M + rows; r0 += rows) {
            b.g0 = b.p0; b.nG = b.nP;
            b.p0 = r0;
            b.nP = r0 >= M ? 0 : (M - r0 < rows ? M - r0 : rows);
            if (b.nP + b.nG == 0) break;
            hipLaunchKernelGGL(kl_two_pass_kernel, dim3(b.nT, b.nP + b.nG), dim3(256), 0, st, b);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    hipLaunchKernelGGL(kl_partial_kernel, dim3(a.nT, M), dim3(256), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kl_finish_kernel, dim3((M + 3) / 4), dim3(256), 0, st, a, M);
    return hipGetLastError();
}

}  // namespace mrp
