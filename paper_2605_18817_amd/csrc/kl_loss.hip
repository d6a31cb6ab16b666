// Training-side loss of the MRP head (paper Section 3.3, Equation 3): per masked row
//     L_i = KL( softmax(l_{t-1}[i]) || softmax(l_t[i] + delta_t[i]) )
// and its gradient with respect to the student logits (hence to delta_t),
//     dL_i / ds[i][v] = softmax(s[i])[v] - softmax(l_{t-1}[i])[v],
// with teacher T = l_{t-1} and student S = l_t + delta_t given as fp32 [M][V].
//
// Both passes are memory streams.  Every (row, 8192-wide vocabulary tile) keeps the online partial
//     (m_T, s_T = sum e^{T - m_T}, a_T = sum e^{T - m_T} (T - S),  m_S, s_S = sum e^{S - m_S})
// of the forward pass, and a row's partials merge to
//     L_i = a_T / s_T - (m_T + log s_T) + (m_S + log s_S).
// No softmax is written.  The gradient reads both tensors once more and writes the difference of the two
// softmaxes.  Algorithmic bytes: 8 M V forward, 4 M V for the gradient; its second read of the tensors comes
// largely from the last-level cache where the rows are taken in groups (see launch_kl_loss): at 1024 rows, V = 151936,
// 80 % of them in the mask, 2.6 GB leave the L2s in 425 us, 6.2 TB/s, where a large copy moves 4.7.
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
    float *part;
    size_t stride;
    float *loss, *grad;
    int p0, nP;      // rows p0 .. p0 + nP - 1: partials
    int g0, nG;      // rows g0 .. g0 + nG - 1: loss and gradient (their partials are complete)
};

// The 32 entries of a tensor's row that a thread handles in tile t: eight 16-byte pieces, -inf past the row's end
__device__ __forceinline__ void kl_fetch(const float *row, int v0, int V, float4 (&x)[8]) {
#pragma unroll
    for (int n = 0; n < 8; ++n) x[n] = load4_row(row, v0 + 4 * (threadIdx.x + 256 * n), V, -INFINITY);
}
__device__ __forceinline__ float kl_at(const float4 (&x)[8], int n) {
    const float4 &q = x[n >> 2];
    return (n & 3) == 0 ? q.x : ((n & 3) == 1 ? q.y : ((n & 3) == 2 ? q.z : q.w));
}

// partial of one KT-wide tile of one row
__device__ __forceinline__ void kl_partial(const KlArgs &a, int t, int i, KlPart *sw) {
    if (a.mask && !a.mask[i]) return;   // (uniform over the workgroup)
    float4 xt[8], xs[8];
    kl_fetch(a.T + (size_t)i * a.V, t * KT, a.V, xt);
    kl_fetch(a.S + (size_t)i * a.V, t * KT, a.V, xs);
    KlPart p = kl_identity();
#pragma unroll
    for (int n = 0; n < 32; ++n) { p.mT = fmaxf(p.mT, kl_at(xt, n)); p.mS = fmaxf(p.mS, kl_at(xs, n)); }
    if (p.mT > -INFINITY) {
#pragma unroll
        for (int n = 0; n < 32; ++n) {
            const float vt = kl_at(xt, n), vs = kl_at(xs, n);
            if (vt > -INFINITY) {   // (padding past V is -inf in both tensors: skip, T - S would be NaN)
                const float e = __expf(vt - p.mT);
                p.sT += e;
                p.aT += e * (vt - vs);
                p.sS += __expf(vs - p.mS);
            }
        }
    }
    p = kl_wave_merge(p);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sw[wave] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        p = sw[0];
        for (int w = 1; w < 4; ++w) p = kl_merge(p, sw[w]);
        const size_t o = (size_t)i * a.nT + t;
        a.part[o] = p.mT; a.part[a.stride + o] = p.sT; a.part[2 * a.stride + o] = p.aT;
        a.part[3 * a.stride + o] = p.mS; a.part[4 * a.stride + o] = p.sS;
    }
}

// gradient of one KT-wide tile of one row; tile 0 also writes the row's loss
__device__ __forceinline__ void kl_gradient(const KlArgs &a, int t, int i) {
    const bool on = !a.mask || a.mask[i];     // (uniform over the workgroup)
    float *gr = a.grad + (size_t)i * a.V;
    const int v0 = t * KT;
    float4 xt[8], xs[8];
    float lT = 0.f, lS = 0.f;
    if (on) {
        kl_fetch(a.T + (size_t)i * a.V, v0, a.V, xt);     // in flight while the row's partials are merged
        kl_fetch(a.S + (size_t)i * a.V, v0, a.V, xs);
        const KlPart p = kl_row(a.part, a.stride, a.nT, i);
        lT = p.mT + logf(p.sT);
        lS = p.mS + logf(p.sS);
        if (t == 0 && threadIdx.x == 0) a.loss[i] = a.scale * (p.aT / p.sT - lT + lS);
    } else if (t == 0 && threadIdx.x == 0) {
        a.loss[i] = 0.f;
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int v = v0 + 4 * (threadIdx.x + 256 * n);
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) {
            g.x = a.scale * (__expf(xs[n].x - lS) - __expf(xt[n].x - lT));
            g.y = a.scale * (__expf(xs[n].y - lS) - __expf(xt[n].y - lT));
            g.z = a.scale * (__expf(xs[n].z - lS) - __expf(xt[n].z - lT));
            g.w = a.scale * (__expf(xs[n].w - lS) - __expf(xt[n].w - lT));
        }
        if (v + 4 <= a.V) {
            // (not kept in the last-level cache, which the rows still to be read again need)
            const f32x4_any gv = {g.x, g.y, g.z, g.w};
            __builtin_nontemporal_store(gv, reinterpret_cast<f32x4_any *>(gr + v));
        } else if (v < a.V) {
            gr[v] = g.x;
            if (v + 1 < a.V) gr[v + 1] = g.y;
            if (v + 2 < a.V) gr[v + 2] = g.z;
        }
    }
}

// One launch takes the partials of one group of rows and the gradient of the group before it, alternating while
// both have rows left, so that the reads of the one run beside the writes of the other.
__global__ __launch_bounds__(256) void kl_kernel(const KlArgs a) {
    __shared__ KlPart sw[4];
    const int t = blockIdx.x, y = blockIdx.y, both = 2 * (a.nP < a.nG ? a.nP : a.nG);
    const bool part = y < both ? (y & 1) == 0 : a.nP > a.nG;
    const int r = y < both ? y >> 1 : y - both / 2;
    if (part) kl_partial(a, t, a.p0 + r, sw);
    else kl_gradient(a, t, a.g0 + r);
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

// Rows taken together when there is a gradient: a group's teacher and student rows are read for the partials and
// once more, one launch later, for the gradient.  What is live in between, two tensors of two groups, has to fit the
// 256 MB last-level cache; smaller groups only add launches.  Measured at 1024 rows, V = 151936: 503 us with groups of
// 52 MB per tensor, 523 of 40, 542 of 30, 612 of 20, 601 of 80, 558 in one group (579 with a launch per pass and the
// scalar merge between them); at 64 rows one group, 34 us.
constexpr size_t GROUP_BYTES = (size_t)52 << 20;

}  // namespace

int kl_tiles(int V) { return (V + KT - 1) / KT; }

hipError_t launch_kl_loss(int M, int V, const float *teacher, const float *student, const uint8_t *mask, float scale,
                          float *part, size_t part_stride, float *loss_rows, float *grad, hipStream_t st) {
    KlArgs a = {teacher, student, mask, V, kl_tiles(V), scale, part, part_stride, loss_rows, grad, 0, M, 0, 0};
    if (!grad) {
        hipLaunchKernelGGL(kl_kernel, dim3(a.nT, M), dim3(256), 0, st, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kl_finish_kernel, dim3((M + 3) / 4), dim3(256), 0, st, a, M);
        return hipGetLastError();
    }
    const size_t bytes = (size_t)M * V * sizeof(float);
    int groups = (int)((bytes + GROUP_BYTES / 2) / GROUP_BYTES);
    groups = groups < 1 ? 1 : (groups > M ? M : groups);
    int rows = (M + groups - 1) / groups;
    if (groups > 1 && rows > 32767) rows = 32767;    // (grid limit: two groups in one launch)
    for (int r0 = 0; r0 < M + rows; r0 += rows) {
        a.g0 = a.p0; a.nG = r0 ? a.nP : 0;
        a.p0 = r0;
        a.nP = r0 >= M ? 0 : (M - r0 < rows ? M - r0 : rows);
        if (a.nP + a.nG == 0) break;
        hipLaunchKernelGGL(kl_kernel, dim3(a.nT, a.nP + a.nG), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace mrp
