// proposal.hip -- kernels of the learned direction proposal: parameter
// packing, batched network evaluation, the weighted-likelihood gradient
// (forward and backward on the matrix cores), the Adam step, and the
// compaction of recorded histories into training samples.
//
// Training objective: the negative log-likelihood of the vMF mixture at the
// directions a plain run actually took, each event weighted by the image flux
// its packet produced afterwards per unit of its luminosity after the event,
// normalised by the sum of those weights.
#include <hip/hip_runtime.h>

#define MCRT_HD __device__ __forceinline__
#include "transport_core.h"
#include "internal.h"
#include "proposal.h"

namespace mcrt {

// ---------------------------------------------------------------------------
// Parameters: FP32 master -> fragments (bf16), biases (FP32) and the FP64
// copy the scalar network of the FP64 validation kernel reads.
// ---------------------------------------------------------------------------
__global__ void pack_kernel(const float *theta, uint16_t *frags, float *bias, double *theta64)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kFragAll * kFragElems) {
        int F = i / kFragElems, r = i % kFragElems, lane = r >> 2, e = r & 3;
        frags[i] = bf16_bits(frag_value(theta, F, lane, e));
    }
    if (i < kBiasFloats) {
        float b = 0.0f;
        if (i < 64) b = theta[kOffB1 + i];
        else if (i < 128) b = theta[kOffB2 + i - 64];
        else if (i < 168) b = theta[kOffB3 + i - 128];
        bias[i] = b;
    }
    if (i < kMlpParams) {
        bool weight = i < kOffB1 || (i >= kOffW2 && i < kOffB2) || (i >= kOffW3 && i < kOffB3);
        theta64[i] = weight ? (double)bf16_float(bf16_bits(theta[i])) : (double)theta[i];
    }
}

hipError_t launch_proposal_pack(const float *theta, uint16_t *frags, float *bias, double *theta64,
                                hipStream_t stream)
{
    const int n = kFragAll * kFragElems; // the largest of the three ranges
    hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, theta, frags, bias, theta64);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched forward pass: out[s][0..39] for features X[s][0..8].  One wave per
// 16 samples at a time; the same tile routine as inside the transport kernel.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) forward_kernel(const uint16_t *frags, const float *bias_g, const float *X,
                                                      int64_t n, float *out)
{
    __shared__ bf16x4 s_wf[kFragFwd * 64];
    __shared__ float s_bias[kBiasFloats];
    const bf16x4 *wf = reinterpret_cast<const bf16x4 *>(frags);
    for (int i = threadIdx.x; i < kFragFwd * 64; i += blockDim.x) s_wf[i] = wf[i];
    for (int i = threadIdx.x; i < kBiasFloats; i += blockDim.x) s_bias[i] = bias_g[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t nblk = (n + 15) / 16;
    for (int64_t b = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); b < nblk; b += waves) {
        const int64_t s = 16 * b + (lane & 15);
        float xv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int q = 4 * (lane >> 4) + i;
            xv[i] = (s < n && q < 9) ? X[s * 9 + q] : 0.0f;
        }
        f32x4 o[3];
        mlp_forward16<false>(s_wf, s_bias, pack_bf16(xv[0], xv[1], xv[2], xv[3]), lane, o);
        if (s < n) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int row = 16 * t + 4 * (lane >> 4) + i;
                    if (row < 40) out[s * 40 + row] = o[t][i];
                }
        }
    }
}

hipError_t launch_proposal_forward(const uint16_t *frags, const float *bias, const float *X, int64_t n, float *out,
                                   hipStream_t stream)
{
    int64_t blocks = (n + 63) / 64;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(forward_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, frags, bias, X, n, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Loss gradient of one sample with respect to the 40 network outputs o, by
// the four lanes l, l + 16, l + 32, l + 48 of a wave: lane part p = lane / 16
// takes lobes 2p and 2p + 1.  Returns log q_vMF(kp) (in every lane);
// dl, da, dk: d(w * -log q) / d of its lobes' logits, axes and concentrations.
// Sums over lobes run in lobe order in every lane.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float nll_grad2(const float *o, const float kp[3], float w, int lane, float dl[2],
                                           float da[2][3], float dk[2])
{
    const float two_pi = 6.28318530717958647692f;
    const int p = lane >> 4;
    float mx = o[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) mx = fmaxf(mx, o[j]);
    float e[8], sum = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        e[j] = expf(o[j] - mx);
        sum += e[j];
    }
    float f[2], kap[2], dkds[2], dot[2], mu[2][3], nrm[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int j = 2 * p + h;
        float a = o[8 + 3 * j], b = o[9 + 3 * j], c = o[10 + 3 * j];
        nrm[h] = sqrtf(a * a + b * b + c * c);
        if (nrm[h] > 0.0f) {
            mu[h][0] = a / nrm[h];
            mu[h][1] = b / nrm[h];
            mu[h][2] = c / nrm[h];
        } else {
            mu[h][0] = 0.0f;
            mu[h][1] = 0.0f;
            mu[h][2] = 1.0f;
        }
        float s = o[32 + j];
        float sp = log1pf(expf(-fabsf(s))) + fmaxf(s, 0.0f) + 1e-3f;
        kap[h] = fminf(fmaxf(sp, 1e-3f), 1e3f);
        dkds[h] = (sp > 1e-3f && sp < 1e3f) ? 1.0f / (1.0f + expf(-s)) : 0.0f;
        // one rounding per product; lobes 5 to 7 start from the second one, as
        // in every training run so far (training amplifies a last bit: 1e-7 of
        // a gradient became 4e-4 of the weights in 97 steps)
        const float m0 = mu[h][0] * kp[0], m1 = mu[h][1] * kp[1];
        dot[h] = fmaf(mu[h][2], kp[2], j < 5 ? fmaf(mu[h][1], kp[1], m0) : fmaf(mu[h][0], kp[0], m1));
        f[h] = kap[h] / (two_pi * -expm1f(-2.0f * kap[h])) * expf(kap[h] * (dot[h] - 1.0f));
    }
    float q = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) q += e[j] / sum * __shfl(f[j & 1], (lane & 15) + 16 * (j >> 1), 64);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float pi = (p == 0 ? e[h] : p == 1 ? e[2 + h] : p == 2 ? e[4 + h] : e[6 + h]) / sum;
        const float r = pi * f[h] / q;
        dl[h] = -w * (r - pi);
        const float gm = nrm[h] > 0.0f ? r * kap[h] / nrm[h] : 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) da[h][a] = -w * gm * (kp[a] - dot[h] * mu[h][a]);
        const float e2 = expf(-2.0f * kap[h]);
        const float dlogf = 1.0f / kap[h] - 2.0f * e2 / (-expm1f(-2.0f * kap[h])) + (dot[h] - 1.0f);
        dk[h] = -w * r * dlogf * dkds[h];
    }
    return logf(q);
}

// ---------------------------------------------------------------------------
// Gradient kernel: a workgroup of four waves takes groups of 64 samples.
// Wave w runs the forward pass, the loss gradient (four lanes to a sample)
// and the backward products dZ2, dZ1 of its 16 samples; X^T, H1^T, H2^T (bf16)
// and dO, dZ2, dZ1 (bf16 high + low parts, about 16 significant bits) of the
// group meet in LDS, and wave w then takes hidden rows 16 w .. 16 w + 15 of
// every weight gradient over all 64 samples.  The gradients stay in registers over
// all of the workgroup's groups and are written once to
// partial[workgroup][7400] (summed in a fixed order by the Adam kernel).
// Bound by the latency of its chain of small products, not by the matrix
// cores (13 MFLOP per group): a minibatch of 16384 is one group per compute
// unit.  One wave per compute unit doing all of this took 40.5 us, this takes 16.1
// (1e5 samples: 201 and 69 us).
// ---------------------------------------------------------------------------
constexpr int kSX = 68;  // row stride (bf16) of [rows][64 samples] tiles
constexpr int kSO = 52;  // row stride of dO [64 samples][48 outputs]
constexpr int kGradStride = kGradStrideFloats;

// Sample of position si in this pass.
__device__ __forceinline__ int64_t sample_index(const GradArgs &g, int64_t si)
{
    if (!g.random) return si;
    U4 r = philox((uint32_t)si, (uint32_t)((uint64_t)si >> 32), g.step, 0x5A4D504Cu, g.key0, g.key1);
    uint64_t w = ((uint64_t)r.x << 32) | (uint64_t)r.y;
    return (int64_t)__umul64hi(w, (uint64_t)g.n); // floor(w n / 2^64)
}

__device__ __forceinline__ bf16x4 lds4(const uint16_t *p) { return *reinterpret_cast<const bf16x4 *>(p); }

__device__ __forceinline__ void split_bf16(f32x4 x, bf16x4 &hi, bf16x4 &lo)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint16_t h = bf16_bits(x[i]);
        hi[i] = (short)h;
        lo[i] = (short)bf16_bits(x[i] - bf16_float(h));
    }
}

// acc += A B^T over 64 samples, B in high and low parts: a, hi, lo point to
// this lane's row (samples consecutive) of the tiles.
__device__ __forceinline__ f32x4 mfma_samples(const uint16_t *a, const uint16_t *hi, const uint16_t *lo, f32x4 acc)
{
#pragma unroll
    for (int j = 0; j < 64; j += 16) {
        acc = mfma16(lds4(a + j), lds4(hi + j), acc);
        acc = mfma16(lds4(a + j), lds4(lo + j), acc);
    }
    return acc;
}

__global__ void __launch_bounds__(256) grad_kernel(GradArgs g)
{
    // bf16 tiles are read 4 values (8 bytes) at a time
    __shared__ __attribute__((aligned(16))) bf16x4 s_wf[kFragAll * 64];
    __shared__ float s_bias[kBiasFloats];
    __shared__ __attribute__((aligned(16))) uint16_t s_xt[16 * kSX];
    __shared__ __attribute__((aligned(16))) uint16_t s_h1t[64 * kSX];
    __shared__ __attribute__((aligned(16))) uint16_t s_h2t[64 * kSX];
    __shared__ float s_stage[64 * 41];
    __shared__ __attribute__((aligned(16))) uint16_t s_dos[2][64 * kSO]; // dO by sample: high, low parts
    __shared__ __attribute__((aligned(16))) uint16_t s_doo[2][48 * kSX]; // dO by output
    __shared__ __attribute__((aligned(16))) uint16_t s_dz2[2][64 * kSX];
    __shared__ __attribute__((aligned(16))) uint16_t s_dz1[2][64 * kSX];
    __shared__ float s_db[2][4][64];                                    // the waves' sums of dZ1, dZ2
    __shared__ float2 s_nll[64]; // weight and negative log-likelihood by sample

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(g.frags);
        uint4 *dst = reinterpret_cast<uint4 *>(s_wf);
        for (int i = threadIdx.x; i < kFragAll * 32; i += 256) dst[i] = src[i];
    }
    for (int i = threadIdx.x; i < kBiasFloats; i += 256) s_bias[i] = g.bias[i];
    // outputs 40 .. 47 are padding
    for (int i = threadIdx.x; i < 64 * 8; i += 256) {
        const int s = i >> 3, j = 40 + (i & 7);
        s_dos[0][s * kSO + j] = s_dos[1][s * kSO + j] = 0;
        s_doo[0][j * kSX + s] = s_doo[1][j * kSX + s] = 0;
    }
    __syncthreads();

    const int r16 = lane & 15, p = lane >> 4, q4 = 4 * p;
    const int mine = 16 * wave + r16; // this lane's sample of the group, and its hidden row
    const f32x4 zero = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 acc3[3], acc2[4], acc1 = zero;
#pragma unroll
    for (int b = 0; b < 3; ++b) acc3[b] = zero;
#pragma unroll
    for (int b = 0; b < 4; ++b) acc2[b] = zero;
    // wave 0: sums of dZ1 and dZ2 by hidden unit, wave 1: of dO by output, wave 2: of the loss by sample
    float db1 = 0.0f, db2 = 0.0f, db3 = 0.0f, loss = 0.0f;

    for (int64_t grp = blockIdx.x; 64 * grp < g.m; grp += gridDim.x) {
        const int64_t si = 64 * grp + mine;
        const bool valid = si < g.m;
        const int64_t id = valid ? sample_index(g, si) : 0;
        float xv[4], kp[3], w = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) xv[i] = (valid && q4 + i < 9) ? g.X[id * 9 + q4 + i] : 0.0f;
#pragma unroll
        for (int i = 0; i < 3; ++i) kp[i] = valid ? g.KP[id * 3 + i] : 0.0f;
        if (valid) w = g.C[id] * g.scale;
        // ---- forward ----
        bf16x4 h1[4], h2[4];
        {
            const bf16x4 x = pack_bf16(xv[0], xv[1], xv[2], xv[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i) s_xt[(q4 + i) * kSX + mine] = (uint16_t)x[i];
            f32x4 o[3];
            mlp_forward16<true>(s_wf, s_bias, x, lane, o, h1, h2);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    s_h1t[(16 * t + q4 + i) * kSX + mine] = (uint16_t)h1[t][i];
                    s_h2t[(16 * t + q4 + i) * kSX + mine] = (uint16_t)h2[t][i];
                }
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (16 * t + q4 + i < 40) s_stage[mine * 41 + 16 * t + q4 + i] = o[t][i];
        }
        wave_lds_sync();
        // ---- loss gradient: four lanes to a sample ----
        {
            float dl[2], da[2][3], dk[2];
            const float lq = nll_grad2(s_stage + mine * 41, kp, w, lane, dl, da, dk);
            if (p == 0) s_nll[mine] = valid ? make_float2(w, -lq) : make_float2(0.0f, 0.0f);
            wave_lds_sync(); // all lanes have read the outputs
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const int l = 2 * p + h, j = c == 0 ? l : c < 4 ? 8 + 3 * l + c - 1 : 32 + l;
                    const float d = valid ? (c == 0 ? dl[h] : c < 4 ? da[h][c - 1] : dk[h]) : 0.0f;
                    const uint16_t hi = bf16_bits(d), lo = bf16_bits(d - bf16_float(hi));
                    s_dos[0][mine * kSO + j] = hi;
                    s_dos[1][mine * kSO + j] = lo;
                    s_doo[0][j * kSX + mine] = hi;
                    s_doo[1][j * kSX + mine] = lo;
                    s_stage[mine * 41 + j] = d;
                }
        }
        wave_lds_sync();
        // ---- dH2^T = W3 dO^T, masked by ReLU -> dZ2 ----
        bf16x4 z2hi[4], z2lo[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 c = zero;
            // output slices 0 and 1, high then low parts, on two 32-deep MFMAs; slice 2 (outputs
            // 32..47) on a third that pairs the slice with itself: A = (A2, A2), B = (high, low)
            // sums A2 high + A2 low.  One MFMA form per accumulator chain (see mfma32).
            const bf16x4 A0 = s_wf[(32 + 3 * t) * 64 + lane], A1 = s_wf[(33 + 3 * t) * 64 + lane];
            const bf16x4 A2 = s_wf[(34 + 3 * t) * 64 + lane];
            const uint16_t *hi = s_dos[0] + mine * kSO + q4, *lo = s_dos[1] + mine * kSO + q4;
            c = mfma32(A0, A1, lds4(hi), lds4(hi + 16), c);
            c = mfma32(A0, A1, lds4(lo), lds4(lo + 16), c);
            c = mfma32(A2, A2, lds4(hi + 32), lds4(lo + 32), c);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (!(bf16_float((uint16_t)h2[t][i]) > 0.0f)) c[i] = 0.0f;
            split_bf16(c, z2hi[t], z2lo[t]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s_dz2[0][(16 * t + q4 + i) * kSX + mine] = (uint16_t)z2hi[t][i];
                s_dz2[1][(16 * t + q4 + i) * kSX + mine] = (uint16_t)z2lo[t][i];
            }
        }
        // ---- dH1^T = W2 dZ2^T, masked -> dZ1 ----
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 c = zero;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x4 A0 = s_wf[(44 + 4 * t + 2 * j) * 64 + lane];
                const bf16x4 A1 = s_wf[(45 + 4 * t + 2 * j) * 64 + lane];
                c = mfma32(A0, A1, z2hi[2 * j], z2hi[2 * j + 1], c);
                c = mfma32(A0, A1, z2lo[2 * j], z2lo[2 * j + 1], c);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (!(bf16_float((uint16_t)h1[t][i]) > 0.0f)) c[i] = 0.0f;
            bf16x4 hi, lo;
            split_bf16(c, hi, lo);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s_dz1[0][(16 * t + q4 + i) * kSX + mine] = (uint16_t)hi[i];
                s_dz1[1][(16 * t + q4 + i) * kSX + mine] = (uint16_t)lo[i];
            }
        }
        wave_lds_sync();
        {
            float a1 = 0.0f, a2 = 0.0f; // hidden unit `lane` over the wave's samples
#pragma unroll
            for (int s = 0; s < 16; s += 4) {
                const bf16x4 h2v = lds4(s_dz2[0] + lane * kSX + 16 * wave + s), l2v = lds4(s_dz2[1] + lane * kSX + 16 * wave + s);
                const bf16x4 h1v = lds4(s_dz1[0] + lane * kSX + 16 * wave + s), l1v = lds4(s_dz1[1] + lane * kSX + 16 * wave + s);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a2 += bf16_float((uint16_t)h2v[i]) + bf16_float((uint16_t)l2v[i]);
                    a1 += bf16_float((uint16_t)h1v[i]) + bf16_float((uint16_t)l1v[i]);
                }
            }
            s_db[0][wave][lane] = a1;
            s_db[1][wave][lane] = a2;
        }
        __syncthreads(); // the group's tiles are complete
        // ---- bias gradients and loss, in sample order ----
        if (wave == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                db1 += s_db[0][k][lane];
                db2 += s_db[1][k][lane];
            }
        } else if (wave == 1) {
            float sacc = 0.0f;
            if (lane < 40)
#pragma unroll
                for (int s = 0; s < 64; ++s) sacc += s_stage[s * 41 + lane];
            db3 += sacc;
        } else if (wave == 2) {
            loss = fmaf(s_nll[lane].x, s_nll[lane].y, loss); // one rounding for product and sum
        }
        // ---- weight gradients: hidden rows 16 wave .. of dW3 += H2^T dO and
        //      dW2 += H1^T dZ2, hidden columns 16 wave .. of dW1 += X^T dZ1 ----
#pragma unroll
        for (int to = 0; to < 3; ++to)
            acc3[to] = mfma_samples(s_h2t + mine * kSX + q4, s_doo[0] + (16 * to + r16) * kSX + q4,
                                    s_doo[1] + (16 * to + r16) * kSX + q4, acc3[to]);
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2)
            acc2[t2] = mfma_samples(s_h1t + mine * kSX + q4, s_dz2[0] + (16 * t2 + r16) * kSX + q4,
                                    s_dz2[1] + (16 * t2 + r16) * kSX + q4, acc2[t2]);
        acc1 = mfma_samples(s_xt + r16 * kSX + q4, s_dz1[0] + mine * kSX + q4, s_dz1[1] + mine * kSX + q4, acc1);
        __syncthreads(); // before the next group's tiles
    }

    // ---- the workgroup's gradient ----
    float *out = g.partial + (int64_t)blockIdx.x * kGradStride;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int f = q4 + i;
        if (f < 9) out[kOffW1 + f * 64 + mine] = acc1[i];
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2) out[kOffW2 + (16 * wave + f) * 64 + 16 * t2 + r16] = acc2[t2][i];
#pragma unroll
        for (int to = 0; to < 3; ++to)
            if (16 * to + r16 < 40) out[kOffW3 + (16 * wave + f) * 40 + 16 * to + r16] = acc3[to][i];
    }
    if (wave == 0) {
        out[kOffB1 + lane] = db1;
        out[kOffB2 + lane] = db2;
    }
    if (wave == 1 && lane < 40) out[kOffB3 + lane] = db3;
    if (wave == 2) {
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
        if (lane == 0) g.loss_partial[blockIdx.x] = (double)loss;
    }
}

hipError_t launch_proposal_grad(const GradArgs &g, int groups, hipStream_t stream)
{
    hipLaunchKernelGGL(grad_kernel, dim3(groups), dim3(256), 0, stream, g);
    return hipGetLastError();
}

// Writes parameter i (new value x) to the packed copies: its fragment
// elements (the inverse of frag_value), the FP32 biases and the FP64 copy.
__device__ __forceinline__ void put_param(int i, float x, uint16_t *frags, float *bias, double *theta64)
{
    if (i >= kOffB1 && i < kOffW2) bias[i - kOffB1] = x;
    else if (i >= kOffB2 && i < kOffW3) bias[64 + i - kOffB2] = x;
    else if (i >= kOffB3) bias[128 + i - kOffB3] = x;
    else {
        const uint16_t h = bf16_bits(x);
        theta64[i] = (double)bf16_float(h);
        // element (F, row r, reduction index q) of a fragment
        auto put = [&](int F, int r, int q) { frags[F * kFragElems + (((q >> 2) << 4) + r) * 4 + (q & 3)] = h; };
        if (i < kOffB1) {
            const int k = i / 64, m = i % 64;
            put(m >> 4, m & 15, k);
        } else if (i < kOffB2) {
            const int k = (i - kOffW2) / 64, m = (i - kOffW2) % 64;
            put(4 + 4 * (m >> 4) + (k >> 4), m & 15, k & 15);
            put(44 + 4 * (k >> 4) + (m >> 4), k & 15, m & 15);
        } else {
            const int h3 = (i - kOffW3) / 40, o = (i - kOffW3) % 40;
            put(20 + 4 * (o >> 4) + (h3 >> 4), o & 15, h3 & 15);
            put(32 + 3 * (h3 >> 4) + (o >> 4), h3 & 15, o & 15);
        }
        return;
    }
    theta64[i] = (double)x;
}

// Sum of the workgroups' gradients in a fixed order (32 parameters x 8
// slices of the partials per workgroup, slices combined in index order), then
// optionally one Adam step on the FP32 master parameters, which also writes
// the packed copies that the next pass reads.  step >= 1 is the Adam time
// step.  Bound by the latency of its loads (7.6 MB from the L2 and the
// Infinity Cache): a thread has 16 partials in flight.  With the loads one by
// one, the loss summed by one thread and the packing in a kernel of its own it
// took 22 + 4.7 us, this takes 4.5.
constexpr int kAdamSlices = 8;
__global__ void __launch_bounds__(32 * kAdamSlices) adam_kernel(const float *partial, int n, const double *loss_partial,
                                                                AdamArgs a)
{
    __shared__ float red[kAdamSlices][33];
    __shared__ double s_loss[kAdamSlices];
    const int c = threadIdx.x & 31, j = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + c;
    float s = 0.0f;
    if (i < kMlpParams) {
#pragma unroll 16
        for (int w = j; w < n; w += kAdamSlices) s += partial[(int64_t)w * kGradStride + i];
    }
    red[j][c] = s;
    if (blockIdx.x == 0 && a.loss_out) { // 32 lanes to a slice, then the slices in order
        double l = 0.0;
        for (int w = threadIdx.x; w < n; w += 32 * kAdamSlices) l += loss_partial[w];
        for (int o = 16; o > 0; o >>= 1) l += __shfl_xor(l, o, 32);
        if (c == 0) s_loss[j] = l;
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.loss_out) {
        double l = 0.0;
        for (int k = 0; k < kAdamSlices; ++k) l += s_loss[k];
        *a.loss_out = l;
    }
    if (j != 0 || i >= kMlpParams) return;
    float gsum = red[0][c];
#pragma unroll
    for (int k = 1; k < kAdamSlices; ++k) gsum += red[k][c];
    if (a.grad_out) a.grad_out[i] = gsum;
    if (!a.update) return;
    float m = a.b1 * a.m[i] + (1.0f - a.b1) * gsum;
    float v = a.b2 * a.v[i] + (1.0f - a.b2) * gsum * gsum;
    a.m[i] = m;
    a.v[i] = v;
    float mh = m / (1.0f - powf(a.b1, (float)a.step));
    float vh = v / (1.0f - powf(a.b2, (float)a.step));
    const float x = a.theta[i] - a.lr * mh / (sqrtf(vh) + a.eps);
    a.theta[i] = x;
    put_param(i, x, a.frags, a.bias, a.theta64);
}

hipError_t launch_proposal_adam(const float *partial, int n, const double *loss_partial, const AdamArgs &a,
                                hipStream_t stream)
{
    hipLaunchKernelGGL(adam_kernel, dim3((kMlpParams + 31) / 32), dim3(32 * kAdamSlices), 0, stream, partial, n,
                       loss_partial, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Histories -> training samples.  Record (slot, e) is an event when its
// luminosity is positive; its weight is C = (packet total - flux so far) / L.
// Samples with C > 0 are kept, in (slot, event) order: a count per tile of
// kHistTile records, an exclusive scan over the tiles, then the writes.  Bound
// by reading the records (all of their lines) twice and writing the samples once:
// a tile's samples are contiguous, so its threads write them as one array (a
// thread per packet, writing its samples by itself: 0.47 ms for 2.7e6 samples of
// 320 000 packets, now 85 us, and 50 for the count).
// ---------------------------------------------------------------------------
constexpr int kHistTile = 1024;

// Weight of record i of the tile that starts with event rem0 of packet slot0.
template <typename Real>
__device__ __forceinline__ float hist_weight(const Real *h, const Real *tot, int64_t slot0, uint32_t rem0, int E,
                                             int64_t base, uint32_t i)
{
    const Real *r = h + (base + i) * kHistFloats;
    if (!(r[12] > Real(0))) return 0.0f;
    return (float)((tot[slot0 + (rem0 + i) / (uint32_t)E] - r[13]) / r[12]);
}

template <typename Real>
__global__ void __launch_bounds__(256) hist_count_kernel(const Real *h, const Real *tot, int64_t n, int E,
                                                         uint32_t *count)
{
    __shared__ uint32_t part[4];
    const int64_t base = (int64_t)blockIdx.x * kHistTile, slot0 = base / E;
    const uint32_t rem0 = (uint32_t)(base % E);
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < kHistTile / 256; ++q) {
        const uint32_t i = q * 256 + threadIdx.x;
        const bool keep = base + i < n && hist_weight(h, tot, slot0, rem0, E, base, i) > 0.0f;
        c += (uint32_t)__popcll(__ballot(keep));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) count[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Exclusive scan in three passes over blocks of 1024 elements.
__global__ void scan_block_kernel(const uint32_t *in, uint64_t *out, int64_t n, uint64_t *block_sums)
{
    __shared__ uint64_t s[1024];
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    uint64_t v = i < n ? in[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        uint64_t t = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0;
        __syncthreads();
        s[threadIdx.x] += t;
        __syncthreads();
    }
    if (i < n) out[i] = s[threadIdx.x] - v;
    if (threadIdx.x == 1023) block_sums[blockIdx.x] = s[1023];
}

__global__ void scan_sums_kernel(uint64_t *block_sums, int64_t nb, uint64_t *total)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    uint64_t run = 0;
    for (int64_t b = 0; b < nb; ++b) {
        uint64_t v = block_sums[b];
        block_sums[b] = run;
        run += v;
    }
    *total = run;
}

__global__ void scan_add_kernel(uint64_t *out, int64_t n, const uint64_t *block_sums)
{
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    if (i < n) out[i] += block_sums[blockIdx.x];
}

template <typename Real>
__global__ void __launch_bounds__(256) hist_write_kernel(const Real *h, const Real *tot, int64_t n, int E,
                                                         const uint64_t *offset, float *X, float *KP, float *C)
{
    __shared__ uint32_t part[kHistTile / 64];
    __shared__ uint16_t rec[kHistTile];
    __shared__ float weight[kHistTile];
    const int64_t base = (int64_t)blockIdx.x * kHistTile, slot0 = base / E;
    const uint32_t rem0 = (uint32_t)(base % E);
    float c[kHistTile / 256];
    uint32_t below[kHistTile / 256];
#pragma unroll
    for (int q = 0; q < kHistTile / 256; ++q) {
        const uint32_t i = q * 256 + threadIdx.x;
        c[q] = base + i < n ? hist_weight(h, tot, slot0, rem0, E, base, i) : 0.0f;
        const unsigned long long keep = __ballot(c[q] > 0.0f);
        below[q] = (uint32_t)__popcll(keep & ((1ull << (threadIdx.x & 63)) - 1));
        if ((threadIdx.x & 63) == 0) part[i >> 6] = (uint32_t)__popcll(keep);
    }
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int g = 0; g < kHistTile / 64; ++g) {
        const uint32_t k = part[g];
#pragma unroll
        for (int q = 0; q < kHistTile / 256; ++q)
            if ((int)((q * 256 + threadIdx.x) >> 6) > g) below[q] += k;
        total += k;
    }
#pragma unroll
    for (int q = 0; q < kHistTile / 256; ++q)
        if (c[q] > 0.0f) {
            rec[below[q]] = (uint16_t)(q * 256 + threadIdx.x);
            weight[below[q]] = c[q];
        }
    __syncthreads();
    const uint64_t k0 = offset[blockIdx.x];
    const Real *r = h + base * kHistFloats;
    for (uint32_t i = threadIdx.x; i < 9 * total; i += 256)
        X[9 * k0 + i] = (float)r[(uint32_t)rec[i / 9] * kHistFloats + i % 9];
    for (uint32_t i = threadIdx.x; i < 3 * total; i += 256)
        KP[3 * k0 + i] = (float)r[(uint32_t)rec[i / 3] * kHistFloats + 9 + i % 3];
    for (uint32_t i = threadIdx.x; i < total; i += 256) C[k0 + i] = weight[i];
}

int64_t hist_tiles(int64_t n_slots, int E) { return (n_slots * E + kHistTile - 1) / kHistTile; }

template <typename Real>
hipError_t hist_count_impl(const Real *h, const Real *tot, int64_t n_slots, int E, uint32_t *count, uint64_t *offset,
                           uint64_t *block_sums, uint64_t *total, hipStream_t st)
{
    const int64_t tiles = hist_tiles(n_slots, E);
    const unsigned nb = (unsigned)((tiles + 1023) / 1024);
    hipLaunchKernelGGL((hist_count_kernel<Real>), dim3((unsigned)tiles), dim3(256), 0, st, h, tot, n_slots * E, E,
                       count);
    hipLaunchKernelGGL(scan_block_kernel, dim3(nb), dim3(1024), 0, st, count, offset, tiles, block_sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(64), 0, st, block_sums, (int64_t)nb, total);
    hipLaunchKernelGGL(scan_add_kernel, dim3(nb), dim3(1024), 0, st, offset, tiles, block_sums);
    return hipGetLastError();
}

template <typename Real>
hipError_t hist_write_impl(const Real *h, const Real *tot, int64_t n_slots, int E, const uint64_t *offset, float *X,
                           float *KP, float *C, hipStream_t st)
{
    hipLaunchKernelGGL((hist_write_kernel<Real>), dim3((unsigned)hist_tiles(n_slots, E)), dim3(256), 0, st, h, tot,
                       n_slots * E, E, offset, X, KP, C);
    return hipGetLastError();
}

hipError_t launch_hist_count(const void *h, const void *tot, bool fp64, int64_t n_slots, int E, uint32_t *count,
                             uint64_t *offset, uint64_t *block_sums, uint64_t *total, hipStream_t st)
{
    if (fp64)
        return hist_count_impl((const double *)h, (const double *)tot, n_slots, E, count, offset, block_sums, total, st);
    return hist_count_impl((const float *)h, (const float *)tot, n_slots, E, count, offset, block_sums, total, st);
}

hipError_t launch_hist_write(const void *h, const void *tot, bool fp64, int64_t n_slots, int E,
                             const uint64_t *offset, float *X, float *KP, float *C, hipStream_t st)
{
    if (fp64) return hist_write_impl((const double *)h, (const double *)tot, n_slots, E, offset, X, KP, C, st);
    return hist_write_impl((const float *)h, (const float *)tot, n_slots, E, offset, X, KP, C, st);
}

// Sum of n floats in FP64, in a fixed order: 1024 columns, then a tree over
// them.  A column is a chain of additions whose loads are taken 32 ahead, and the
// columns are spread over 16 workgroups (2.7e6 floats: 35 us; by one
// workgroup, a load at a time, 520).
__global__ void __launch_bounds__(64) sum_columns_kernel(const float *x, int64_t n, double *cols)
{
    const int c = blockIdx.x * 64 + threadIdx.x;
    double a = 0.0;
    int64_t i = c;
    for (; i + 31 * 1024 < n; i += 32 * 1024) {
        float v[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = x[i + k * 1024];
#pragma unroll
        for (int k = 0; k < 32; ++k) a += (double)v[k];
    }
    for (; i < n; i += 1024) a += (double)x[i];
    cols[c] = a;
}

__global__ void __launch_bounds__(1024) sum_tree_kernel(const double *cols, double *out)
{
    __shared__ double s[1024];
    s[threadIdx.x] = cols[threadIdx.x];
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < (unsigned)o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

hipError_t launch_sum_f32(const float *x, int64_t n, double *cols, double *out, hipStream_t stream)
{
    hipLaunchKernelGGL(sum_columns_kernel, dim3(16), dim3(64), 0, stream, x, n, cols);
    hipLaunchKernelGGL(sum_tree_kernel, dim3(1), dim3(1024), 0, stream, cols, out);
    return hipGetLastError();
}

} // namespace mcrt
