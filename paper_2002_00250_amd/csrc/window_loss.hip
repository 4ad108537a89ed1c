// The adjoint's loss: mean binary cross-entropy of sigmoid(Z / tau) against 0/255 ground truth,
// weighted by the term flags, and its gradient with respect to Z.  Composed of elementwise
// operations it takes some fifteen passes over the scores (64 frames of 640x480: about 600 us of
// a training step, as much as the window's two kernels).  Here, back to back on that window: the loss
// alone is one pass that reads 6 bytes a score (29.5 us, 4.0 TB/s, bound by some 60 vector
// instructions a score); with a gradient to follow it also writes 5 (39.4 us, 5.5 TB/s), and the
// gradient's pass reads 4 and writes 4 (24.3 us, 6.5 TB/s, the copy rate).  A gradient from Z, has
// and gt themselves, 26.3 + 28.6 us, needs them unchanged until the backward.
//
// Per score i >= i0 (x = Z * (1 / tau), y = gt != 0, w = has), in float32:
//   loss      w * ((1 - y) * x - logsigmoid(x)),  logsigmoid(x) = min(x, 0) - log1p(exp(-|x|))
//   slope     (sigmoid(x) - y) * w
//   gradient  (slope * (g / max(sum w, 1))) * (1 / tau),  0 for i < i0
// The loss pass can keep the slopes and the weights (5 bytes a score) for a gradient that does not
// read Z, has and gt again, which the caller may have refilled by then.
// Sums are kept in fp64, in a fixed order (lane, wavefront, block, then one block over the
// partials): deterministic.
#include "device_common.h"
#include "fgs_internal.h"

namespace fgs {

namespace {

constexpr int kBlock = 256;
constexpr int kGroup = 4;  // scores a lane takes at a time: 16 bytes of Z, 4 of the flags and truth

// Scores i .. i + 3, their flags and their truth, a byte each; 0 past the last one.  VEC: the arrays
// are aligned for whole groups.
struct Group {
    float z[kGroup];
    uint32_t h, t;
};
template <bool VEC>
__device__ __forceinline__ Group read_group(const float* Z, const uint8_t* has, const uint8_t* gt, int64_t i, int64_t n) {
    Group r;
    if (VEC && i + kGroup <= n) {
        const float4 z = *reinterpret_cast<const float4*>(Z + i);
        r.z[0] = z.x;
        r.z[1] = z.y;
        r.z[2] = z.z;
        r.z[3] = z.w;
        r.h = *reinterpret_cast<const uint32_t*>(has + i);
        r.t = *reinterpret_cast<const uint32_t*>(gt + i);
        return r;
    }
    r.h = r.t = 0u;
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
        const bool in = i + k < n;
        r.z[k] = in ? Z[i + k] : 0.0f;
        r.h |= (in ? (uint32_t)has[i + k] : 0u) << (8 * k);
        r.t |= (in ? (uint32_t)gt[i + k] : 0u) << (8 * k);
    }
    return r;
}
__device__ __forceinline__ uint32_t byte_at(uint32_t w, int k) { return (w >> (8 * k)) & 0xFFu; }

__device__ __forceinline__ void block_sum2(double& a, double& b, double (*sh)[2]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6][0] = a;
        sh[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) {
            a += sh[w][0];
            b += sh[w][1];
        }
}

// log(1 + e) for 0 <= e <= 1 to 0.63 ulp (over all of it, with a reciprocal up to an ulp off):
// log(1 + e) = 2 atanh(s), s = e / (2 + e) <= 1/3, with s in two parts (2 + e and the quotient
// corrected by what their rounding lost) and (2 atanh(s) / s - 2) / s^2 by its Chebyshev interpolation
// of degree 4 in s^2 on [0, 1/9], 2e-8 off at most.  The quotient in one part and a series gave 2.4 to
// 3.7 ulp; the library's log1p, which serves every argument, three times the instructions.
__device__ __forceinline__ float log1p_unit(float e) {
    const float t = 2.0f + e, te = e - (t - 2.0f), r = __builtin_amdgcn_rcpf(t), s0 = e * r;
    const float lo = __builtin_fmaf(-s0, te, __builtin_fmaf(-s0, t, e)) * r;
    const float s = s0 + lo, q = s * s;
    float p = 0.2322433f;
    p = __builtin_fmaf(p, q, 0.21706575f);
    p = __builtin_fmaf(p, q, 0.28592357f);
    p = __builtin_fmaf(p, q, 0.39999706f);
    p = __builtin_fmaf(p, q, 0.6666667f);
    return (s0 + s0) + __builtin_fmaf(s, q * p, lo + lo);
}

// sigmoid(x) by e = exp(-|x|): 1 / (1 + e) or e / (1 + e), the quotient corrected by its remainder.
__device__ __forceinline__ float sigmoid_of(float x, float e) {
    const float t = 1.0f + e, n = x >= 0.0f ? 1.0f : e, r = __builtin_amdgcn_rcpf(t), q = n * r;
    return __builtin_fmaf(__builtin_fmaf(-t, q, n), r, q);
}

// work[2 + 2 b], work[3 + 2 b]: block b's sums of the weighted losses and of the weights.  KEEP: also
// slope and weight (0 for i < i0).  Groups are counted from the first score's, so the sums are the
// same with and without.
template <bool VEC, bool KEEP>
__global__ __launch_bounds__(kBlock) void bce_sum_kernel(const float* __restrict__ Z, const uint8_t* __restrict__ has,
                                                         const uint8_t* __restrict__ gt, int64_t i0, int64_t n, float by_tau,
                                                         double* __restrict__ work, float* __restrict__ slope,
                                                         uint8_t* __restrict__ weight) {
    __shared__ double sh[kBlock / 64][2];
    double sl = 0.0, sw = 0.0;
    const int64_t step = (int64_t)gridDim.x * kBlock * kGroup;
    const int64_t first = i0 - i0 % kGroup, lane = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kGroup;
    if (KEEP)
        for (int64_t i = lane; i < first; i += step) {
#pragma unroll
            for (int k = 0; k < kGroup; ++k) {
                slope[i + k] = 0.0f;
                weight[i + k] = 0;
            }
        }
    for (int64_t i = first + lane; i < n; i += step) {
        Group g = read_group<VEC>(Z, has, gt, i, n);
        if (i < i0) {  // (the first group alone: scores before i0 count for nothing)
#pragma unroll
            for (int k = 0; k < kGroup; ++k)
                if (i + k < i0) {
                    g.z[k] = 0.0f;
                    g.h &= ~(0xFFu << (8 * k));
                }
        }
        float l = 0.0f, d[kGroup];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) {
            const float x = g.z[k] * by_tau;
            const float y = byte_at(g.t, k) ? 1.0f : 0.0f, w = (float)byte_at(g.h, k);
            const float e = expf(-fabsf(x));
            const float ls = fminf(x, 0.0f) - log1p_unit(e);
            l += w * ((1.0f - y) * x - ls);
            if (KEEP) d[k] = (sigmoid_of(x, e) - y) * w;
        }
        sl += (double)l;
        sw += (double)__builtin_amdgcn_sad_u8(g.h, 0u, 0u);  // the four flags' sum
        if (!KEEP) continue;
        if (VEC && i + kGroup <= n) {
            *reinterpret_cast<float4*>(slope + i) = make_float4(d[0], d[1], d[2], d[3]);
            *reinterpret_cast<uint32_t*>(weight + i) = g.h;
            continue;
        }
#pragma unroll
        for (int k = 0; k < kGroup; ++k)
            if (i + k < n) {
                slope[i + k] = d[k];
                weight[i + k] = (uint8_t)byte_at(g.h, k);
            }
    }
    block_sum2(sl, sw, sh);
    if (threadIdx.x == 0) {
        work[2 + 2 * blockIdx.x] = sl;
        work[3 + 2 * blockIdx.x] = sw;
    }
}

// work[0], work[1]: the sum of the losses and max(sum of the weights, 1); *loss their quotient.
__global__ __launch_bounds__(kBlock) void bce_finish_kernel(double* work, int blocks, float* loss) {
    __shared__ double sh[kBlock / 64][2];
    double sl = 0.0, sw = 0.0;
    for (int b = threadIdx.x; b < blocks; b += kBlock) {
        sl += work[2 + 2 * b];
        sw += work[3 + 2 * b];
    }
    block_sum2(sl, sw, sh);
    if (threadIdx.x == 0) {
        sw = sw < 1.0 ? 1.0 : sw;
        work[0] = sl;
        work[1] = sw;
        *loss = (float)(sl / sw);
    }
}

template <bool VEC>
__global__ __launch_bounds__(kBlock) void bce_grad_kernel(const float* __restrict__ Z, const uint8_t* __restrict__ has,
                                                          const uint8_t* __restrict__ gt, int64_t i0, int64_t n, float by_tau,
                                                          const double* __restrict__ work, const float* __restrict__ gloss,
                                                          float* __restrict__ dZ) {
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kGroup;
    if (i >= n) return;
    const float scale = gloss[0] / (float)work[1];
    const Group g = read_group<VEC>(Z, has, gt, i, n);
    float d[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
        const float x = g.z[k] * by_tau;
        const float y = byte_at(g.t, k) ? 1.0f : 0.0f, w = (float)byte_at(g.h, k);
        const float s = 1.0f / (1.0f + expf(-x));
        d[k] = i + k >= i0 ? ((s - y) * w * scale) * by_tau : 0.0f;
    }
    if (VEC && i + kGroup <= n) {
        *reinterpret_cast<float4*>(dZ + i) = make_float4(d[0], d[1], d[2], d[3]);
        return;
    }
#pragma unroll
    for (int k = 0; k < kGroup; ++k)
        if (i + k < n) dZ[i + k] = d[k];
}

// The gradient from the kept slopes.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void bce_kept_grad_kernel(const float* __restrict__ slope, int64_t i0, int64_t n,
                                                               float by_tau, const double* __restrict__ work,
                                                               const float* __restrict__ gloss, float* __restrict__ dZ) {
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kGroup;
    if (i >= n) return;
    const float scale = gloss[0] / (float)work[1];
    auto of = [&](float d, int k) { return i + k >= i0 ? (d * scale) * by_tau : 0.0f; };
    if (VEC && i + kGroup <= n) {
        const float4 d = *reinterpret_cast<const float4*>(slope + i);
        *reinterpret_cast<float4*>(dZ + i) = make_float4(of(d.x, 0), of(d.y, 1), of(d.z, 2), of(d.w, 3));
        return;
    }
#pragma unroll
    for (int k = 0; k < kGroup; ++k)
        if (i + k < n) dZ[i + k] = of(slope[i + k], k);
}

bool aligned(const float* Z, const uint8_t* has, const uint8_t* gt) {
    return (((uintptr_t)Z & 15) | ((uintptr_t)has & 3) | ((uintptr_t)gt & 3)) == 0;
}

template <bool VEC>
void launch_sum(dim3 grid, hipStream_t s, const float* Z, const uint8_t* has, const uint8_t* gt, int64_t i0, int64_t n,
                float by_tau, double* work, float* slope, uint8_t* weight) {
    if (slope)
        hipLaunchKernelGGL((bce_sum_kernel<VEC, true>), grid, dim3(kBlock), 0, s, Z, has, gt, i0, n, by_tau, work, slope,
                           weight);
    else
        hipLaunchKernelGGL((bce_sum_kernel<VEC, false>), grid, dim3(kBlock), 0, s, Z, has, gt, i0, n, by_tau, work, slope,
                           weight);
}

}  // namespace

hipError_t window_bce_launch(const float* Z, const uint8_t* has, const uint8_t* gt, int64_t i0, int64_t n, float tau,
                             double* work, float* loss, float* slope, uint8_t* weight, hipStream_t s) {
    const int64_t groups = (n - (i0 - i0 % kGroup) + kGroup - 1) / kGroup;
    int64_t blocks = (groups + kBlock - 1) / kBlock;
    blocks = blocks < 1 ? 1 : (blocks > kBceBlocks ? kBceBlocks : blocks);
    const dim3 grid((unsigned)blocks);
    if (aligned(Z, has, gt) && aligned(slope, weight, nullptr))
        launch_sum<true>(grid, s, Z, has, gt, i0, n, 1.0f / tau, work, slope, weight);
    else
        launch_sum<false>(grid, s, Z, has, gt, i0, n, 1.0f / tau, work, slope, weight);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bce_finish_kernel, dim3(1), dim3(kBlock), 0, s, work, (int)blocks, loss);
    return hipGetLastError();
}

hipError_t window_bce_grad_launch(const float* Z, const uint8_t* has, const uint8_t* gt, int64_t i0, int64_t n, float tau,
                                  const double* work, const float* gloss, float* dZ, hipStream_t s) {
    const int64_t blocks = ((n + kGroup - 1) / kGroup + kBlock - 1) / kBlock;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kBlock);
    if (aligned(Z, has, gt) && ((uintptr_t)dZ & 15) == 0)
        hipLaunchKernelGGL(bce_grad_kernel<true>, grid, block, 0, s, Z, has, gt, i0, n, 1.0f / tau, work, gloss, dZ);
    else
        hipLaunchKernelGGL(bce_grad_kernel<false>, grid, block, 0, s, Z, has, gt, i0, n, 1.0f / tau, work, gloss, dZ);
    return hipGetLastError();
}

hipError_t window_bce_kept_grad_launch(const float* slope, int64_t i0, int64_t n, float tau, const double* work,
                                       const float* gloss, float* dZ, hipStream_t s) {
    const int64_t blocks = ((n + kGroup - 1) / kGroup + kBlock - 1) / kBlock;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kBlock);
    if ((((uintptr_t)slope | (uintptr_t)dZ) & 15) == 0)
        hipLaunchKernelGGL(bce_kept_grad_kernel<true>, grid, block, 0, s, slope, i0, n, 1.0f / tau, work, gloss, dZ);
    else
        hipLaunchKernelGGL(bce_kept_grad_kernel<false>, grid, block, 0, s, slope, i0, n, 1.0f / tau, work, gloss, dZ);
    return hipGetLastError();
}

}  // namespace fgs
