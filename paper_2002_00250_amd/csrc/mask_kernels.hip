// Copies of a mask plane (H x W bytes, contiguous) to a caller's rows: device memory, or pinned
// host memory that the host reads after the stream is done.  A lane reads 16 consecutive bytes of
// the plane and stores them as wide as the destination allows.  Bound by its launch at camera sizes.
// The runtime's two-dimensional copy to pageable memory goes row by row: reading a 640x480 mask
// took 3,270 us, through pinned memory 26.
#include "device_common.h"
#include "fgs_internal.h"

namespace fgs {

namespace {

// The first `count` bytes of the plane to rows of W bytes `stride` apart, byte i being row i / W,
// column i % W.
__global__ __launch_bounds__(256) void mask_copy_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                                        int64_t stride, uint32_t W, FastDiv by_w, uint32_t count) {
    const uint32_t i = (blockIdx.x * 256u + threadIdx.x) * 16u;
    if (i >= count) return;
    const uint32_t n = min(16u, count - i);
    uint32_t y = div_by(i, by_w);
    uint32_t x = i - y * W;
    uint32_t w[4];
    if (n == 16u) {
        const uint4 v = *reinterpret_cast<const uint4*>(src + i);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    } else {
        w[0] = w[1] = w[2] = w[3] = 0u;
#pragma unroll
        for (uint32_t k = 0; k < 16u; ++k)
            if (k < n) w[k >> 2] |= (uint32_t)src[i + k] << (8 * (k & 3));
    }
    uint8_t* d = dst + (int64_t)y * stride + x;
    if (n == 16u && x + 16u <= W) {
        if (((uintptr_t)d & 15u) == 0) {
            *reinterpret_cast<uint4*>(d) = make_uint4(w[0], w[1], w[2], w[3]);
            return;
        }
        if (((uintptr_t)d & 3u) == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) reinterpret_cast<uint32_t*>(d)[k] = w[k];
            return;
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < 16u; ++k) {
        if (k < n) {
            *d++ = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
            if (++x == W) {
                x = 0;
                d = dst + (int64_t)++y * stride;
            }
        }
    }
}

}  // namespace

hipError_t mask_launch_copy(const uint8_t* plane, int W, uint8_t* dst, int64_t stride, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t groups = (count + 15) / 16;
    hipLaunchKernelGGL(mask_copy_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, plane, dst, stride,
                       (uint32_t)W, fast_div((uint32_t)W), (uint32_t)count);
    return hipGetLastError();
}

}  // namespace fgs
