// The whole MLP head body of one sequence in one workgroup, for the narrowest models (paper Section 3.2 and Algorithm 2,
// inner loop: u = W2 SiLU(W1 [h ; e]), h <- h + u, y = RMSNorm(u)), together with the decision on the state before it
// that picks the embedding e (select_sequence.h).
//
// At d <= 256 both weight matrices are 0.4 MB: one CU pulls them out of the L2 in a few microseconds, less than the five
// dependent launches of the general path spend on starting and on waiting for each other (merge 5.5, GEMM 5.8, GEMM 3.5,
// norm 2.7 us a head for 4 rows).  What bounds it is that pull and the chain of latencies.  Wave w computes features
// 16 w .. of both GEMMs over the whole k (v_mfma_f32_16x16x32_f16 on 16 rows; fragments of 16 rows x 32 k are four 256-byte
// runs of two packed blocks); its hidden-state weights are requested ahead of the decision, the activations stand in LDS as
// two fp16 planes, and the hidden, embedding and low-plane products have accumulators of their own (the first two a pair
// each: with one, u is 1.5 % further from 64 bits than from the general path, whose eight waves split the k).
#include "select_sequence.h"

namespace mrp {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int HY_THREADS = 1024;

__device__ __forceinline__ f32x4 mma(const u32x4 &w, const u32x4 &x, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0, 0);
}

template <int D>
__global__ __launch_bounds__(HY_THREADS) void head_tiny_kernel(const HeadTinyArgs a) {
    constexpr int KP = D / 32;                       // 32-wide k steps per D columns
    __shared__ u32x4 xs[2][KP][64];                  // planes of h, then of s: [plane][k step][lane]
    __shared__ u32x4 ss[2][KP][64];
    __shared__ float red[D / 16][16];
    const int b = blockIdx.x, L = a.L, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, cq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool busy = wave < D / 16;                 // (uniform over the wave; all of them at D = 256)

    // this wave's fragments of W1's hidden half (all of W1 would not fit the registers next to the merge's)
    const int frag = 16 * (wave & 1) + l16 + 32 * (cq & 1) + 64 * (cq >> 1);
    const u32x4 *w1p = reinterpret_cast<const u32x4 *>(a.W1p) + (size_t)(wave >> 1) * (2 * D / 16) * 64 + frag;
    u32x4 w1[KP];
    if (busy) {
#pragma unroll
        for (int k = 0; k < KP; ++k) w1[k] = w1p[k * 128];
    }
    // the sequence's hidden state as planes; rows past its L are zero
    if (tid < 16 * (D / 8)) {
        const int r = tid & 15, c8 = tid >> 4;
        const size_t at = (size_t)(b * L + r) * D + 8 * c8;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = 0.f;
        if (r < L) {
            if (a.h) {
                unpack_bf16x8(*reinterpret_cast<const uint4 *>(a.h + at), x);
            } else {
                const float4 p = *reinterpret_cast<const float4 *>(a.hrun + at), q = *reinterpret_cast<const float4 *>(a.hrun + at + 4);
                x[0] = p.x; x[1] = p.y; x[2] = p.z; x[3] = p.w; x[4] = q.x; x[5] = q.y; x[6] = q.z; x[7] = q.w;
            }
        }
        split_store(x, reinterpret_cast<uint4 *>(&xs[0][c8 >> 2][r + 16 * (c8 & 3)]), 0, KP * 64);
    }
    // this lane's four entries of the hidden state and of the gain: row l16, features 16 wave + 4 cq ..
    const int i = b * L + (l16 < L ? l16 : L - 1), f0 = 16 * wave + 4 * cq;
    float4 hv = make_float4(0.f, 0.f, 0.f, 0.f);
    uint2 gv = make_uint2(0, 0);
    if (busy) {
        if (a.h) {
            const uint2 p = *reinterpret_cast<const uint2 *>(a.h + (size_t)i * D + f0);
            hv = make_float4(bf16_to_f32(p.x & 0xffff), bf16_to_f32(p.x >> 16), bf16_to_f32(p.y & 0xffff), bf16_to_f32(p.y >> 16));
        } else {
            hv = *reinterpret_cast<const float4 *>(a.hrun + (size_t)i * D + f0);
        }
        gv = *reinterpret_cast<const uint2 *>(a.gamma + f0);
    }

    int tok;
    if (a.decide) {
        tok = merge_select_sequence<HY_THREADS, 4>(a.sel, b);
    } else {
        tok = a.cond_tok[b];
        __syncthreads();
    }
    if ((tok < 0 || tok >= a.V) && tid == 0 && a.err_flag) atomicOr(a.err_flag, ERR_COND_TOK);   // clamped and reported
    tok = tok < 0 ? 0 : (tok >= a.V ? a.V - 1 : tok);

    u32x4 w2[KP];
    if (busy) {
        const uint4 *e = reinterpret_cast<const uint4 *>(a.E + (size_t)tok * D) + cq;
        uint4 ef[KP];
        u32x4 we[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) { ef[k] = e[4 * k]; we[k] = w1p[(KP + k) * 128]; }
        const u32x4 *p = reinterpret_cast<const u32x4 *>(a.W2p) + (size_t)(wave >> 1) * (D / 16) * 64 + frag;
#pragma unroll
        for (int k = 0; k < KP; ++k) w2[k] = p[k * 128];
        f32x4 hi[2] = {}, em[2] = {}, lo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            hi[k & 1] = mma(w1[k], xs[0][k][lane], hi[k & 1]);
            lo = mma(w1[k], xs[1][k][lane], lo);
        }
#pragma unroll
        for (int k = 0; k < KP; ++k) em[k & 1] = mma(we[k], __builtin_bit_cast(u32x4, bf16x8_to_f16x8(ef[k])), em[k & 1]);
        uint16_t sh[4], sl[4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const float v = ((hi[0][e4] + hi[1][e4]) + (em[0][e4] + em[1][e4])) + lo[e4];
            split2(v / (1.0f + expf(-v)), sh[e4], sl[e4]);
        }
        // features 4 cq .. of the wave's 16: half of a 16-byte chunk
        uint2 *s0 = reinterpret_cast<uint2 *>(&ss[0][wave >> 1][l16 + 16 * (2 * (wave & 1) + (cq >> 1))]) + (cq & 1);
        s0[0] = make_uint2(pack2(sh[0], sh[1]), pack2(sh[2], sh[3]));
        s0[2 * KP * 64] = make_uint2(pack2(sl[0], sl[1]), pack2(sl[2], sl[3]));
    }
    __syncthreads();
    f32x4 u = {0.f, 0.f, 0.f, 0.f};
    if (busy) {
        f32x4 hi[2] = {}, lo = u;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            hi[k & 1] = mma(w2[k], ss[0][k][lane], hi[k & 1]);
            lo = mma(w2[k], ss[1][k][lane], lo);
        }
        u = (hi[0] + hi[1]) + lo;
        float q = (u[0] * u[0] + u[1] * u[1]) + (u[2] * u[2] + u[3] * u[3]);
        q += __shfl_xor(q, 16);
        q += __shfl_xor(q, 32);
        if (cq == 0) red[wave][l16] = q;
    }
    __syncthreads();
    if (busy && l16 < L) {
        float q = 0.f;
#pragma unroll
        for (int w = 0; w < D / 16; ++w) q += red[w][l16];
        const float inv = 1.0f / sqrtf(q / (float)D + a.eps);
        const float g[4] = {bf16_to_f32(gv.x & 0xffff), bf16_to_f32(gv.x >> 16), bf16_to_f32(gv.y & 0xffff), bf16_to_f32(gv.y >> 16)};
        uint16_t y[4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) y[e4] = f32_to_bf16_rne(u[e4] * inv * g[e4]);
        reinterpret_cast<uint2 *>(a.Y)[2 * act_chunk_index(i, f0 >> 3, a.nIb) + (cq & 1)] = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
        if (a.carry) hv = make_float4(hv.x + u[0], hv.y + u[1], hv.z + u[2], hv.w + u[3]);
        if (a.carry || a.h) *reinterpret_cast<float4 *>(a.hrun + (size_t)i * D + f0) = hv;
    }
}

}  // namespace

hipError_t launch_head_tiny(const HeadTinyArgs &a, int B, int d, hipStream_t st) {
    if (a.L < 1 || a.L > 16) return hipErrorInvalidValue;
    if (d == 128) hipLaunchKernelGGL(head_tiny_kernel<128>, dim3(B), dim3(HY_THREADS), 0, st, a);
    else if (d == 256) hipLaunchKernelGGL(head_tiny_kernel<256>, dim3(B), dim3(HY_THREADS), 0, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace mrp
