// RGB-D Gaussian mixture background model: one fused classify-and-update kernel
// per frame (Sec. 3.1).  One lane per pixel; the pixel's whole state (both
// mixtures) is read once and written once per frame with 16-byte accesses, and
// everything in between stays in registers.  No contraction anywhere: the path
// is a streaming state update bound by HBM bandwidth.
//
// Arithmetic is IEEE binary32, each operation rounded on its own (the library is
// built with -ffp-contract=off; division and square root are correctly rounded),
// in the order of the method (the approximate decisions of gmm_device.h give the same results):
//   q_k = d2_k / v_k,  d2 = ((e0*e0) + e1*e1) + e2*e2
//   decision on the ranked pre-update mixture: B = leading Gaussians whose
//     weights first sum past T_bg (else those with w > 0), delta = min_{k<B} q_k,
//     Z = (delta_c - lambda^2) + w_d*(delta_d - lambda^2), depth term only where
//     D > 0 and the depth mixture has data; foreground iff Z >= 0
//   update (colour always, depth where D > 0): first k with w_k > 0 and
//     q_k < lambda^2 matches; w = (1-alpha) w (+ alpha if matched); matched
//     mu += alpha (X - mu); v += alpha (|X - mu_new|^2 - v); v >= v_min; no match:
//     Gaussian K-1 = (w_init, X, v_init); w /= sum(w); stable sort by w/sqrt(v).
#include <cstring>

#include "device_common.h"
#include "fgs_internal.h"
#include "gmm_device.h"

namespace fgs {

namespace {

// 256 lanes per workgroup, and where the state is streamed three workgroups per CU: HBM serves
// a few pages of every plane better than many.  Measured on 8 models of 1280x720, K = 5, non-
// temporal, a static background with moving objects, us per launch by waves per CU: 8 288, 12 269.4,
// 16 283, 20 and more 294 (512-lane workgroups 277 with 16 waves, 286 with 24; 192 lanes 282-294; 128
// lanes 272 at best).  Against the 512-lane kernel without the approximate decisions and scalar plane
// addresses (gmm_device.h): K = 5 280.4 -> 269.4, 8 x K = 3 186 -> 177, 6 x 7/3 228 -> 220, one 7/3
// 1920x1080 91.5 -> 88.4; the benchmark's scene, whose objects change more sectors, 300 -> 287 (6.1 TB/s
// of measured HBM traffic).  Two planes a pixel (K = 1) and four (K = 2) are too few bytes per wave for
// the limit (76 -> 91 us; 8 models 134.4 -> 141.7, 12 206.5 -> 215.8, 3840x2160 152.3 -> 160.2), so it holds
// from six planes (K = 3) on; without it they are within 3 % of the 512-lane kernel either way.  A
// cache-resident state wants every wave it can get: K = 3 per-channel variances at 853x487, 17.6 -> 16.1.
constexpr int kBlock = 256;
constexpr int kStreamPlanes = 6;
constexpr unsigned kStreamLds = 48u << 10;  // 3 of these fit a CU's 160 KiB; nothing is kept there

// GEN = false: the default rate and decision compiled in; GEN = true: both read
// from the constants (any other choice).  CV = 3: per-channel colour variances.
// One launch steps b.n models (one for a single push): workgroup w takes pixels
// kBlock (w - first[i]) .. + kBlock - 1 of model i, first[i] <= w < first[i + 1].
template <int NB, int KC, int KD, bool NT, bool GEN, int CV>
__global__ __launch_bounds__(kBlock) void gmm_step_kernel(GmmBatch<NB> b) {
    const int w = (int)blockIdx.x;
    int i = 0;
#pragma unroll
    for (int j = 1; j < NB; ++j) i = w >= b.first[j] ? j : i;  // (first[j] is the grid size for j >= n)
    const GmmStepArgs& a = b.a[i];
    const int p0 = (w - b.first[i]) * kBlock, lane = (int)threadIdx.x;
    if (p0 + lane < a.npix) gmm_pixel<KC, KD, NT, GEN ? 2 : 0, GEN ? 2 : 0, CV>(a, p0, lane);
}

// Run-time Kc, Kd indices of the extra-plane fields (fgs_internal.h).
__device__ __forceinline__ int x_vd(int Kc, int Kd, int k) { return gmm_x_vd(Kc, Kd, k); }
__device__ __forceinline__ int x_vg(int Kc, int Kd, int k) { return gmm_x_vg(Kc, Kd, k); }
__device__ __forceinline__ int x_vb(int Kc, int Kd, int k) { return gmm_x_vb(Kc, Kd, k); }

__device__ __forceinline__ float* f4(float4* s, int64_t i) { return reinterpret_cast<float*>(s + i); }
__device__ __forceinline__ float* xf(float4* s, int Kc, int64_t n, int64_t p, int idx) {
    return f4(s, (int64_t)(Kc + idx / 4) * n + p) + idx % 4;
}
// Fresh model: w = 0, mu = 0, v = v_init (both mixtures; every colour channel's
// variance when they are per channel).
__global__ void gmm_init_kernel(float4* state, int Kc, int Kd, int var_mode, int npix, float v_init_c,
                                float v_init_d) {
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    const int E = gmm_extra_planes(Kc, Kd, var_mode);
    for (int k = 0; k < Kc; ++k) state[(int64_t)k * n + p] = make_float4(0.f, 0.f, 0.f, v_init_c);
    for (int e = 0; e < E; ++e) state[(int64_t)(Kc + e) * n + p] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < Kd; ++k) *xf(state, Kc, n, p, x_vd(Kc, Kd, k)) = v_init_d;
    if (var_mode)
        for (int k = 0; k < Kc; ++k) {
            *xf(state, Kc, n, p, x_vg(Kc, Kd, k)) = v_init_c;
            *xf(state, Kc, n, p, x_vb(Kc, Kd, k)) = v_init_c;
        }
}

// Canonical order: w_c[Kc], mu_c[Kc][3], v_c[Kc] (per-channel: v_c[Kc][3]), w_d[Kd],
// mu_d[Kd], v_d[Kd], planes of npix.  The plane of float i of the extra planes, -1: padding.
__device__ __forceinline__ int canon_plane(int i, int Kc, int Kd, int nv) {
    const int d0 = (4 + nv) * Kc;
    if (i < Kc) return i;
    i -= Kc;
    if (i < Kd) return d0 + i;
    i -= Kd;
    if (i < 2 * Kd) return d0 + (1 + (i & 1)) * Kd + (i >> 1);
    i -= 2 * Kd;
    return nv == 3 && i < 2 * Kc ? 4 * Kc + 3 * (i >> 1) + 1 + (i & 1) : -1;
}

// One 16-byte read per plane and pixel, one store per float (and the reverse).
__global__ __launch_bounds__(kBlock) void gmm_export_kernel(const float4* __restrict__ state, float* __restrict__ out,
                                                            int Kc, int Kd, int var_mode, int npix, int has_header,
                                                            StateWords header) {
    write_header(reinterpret_cast<uint32_t*>(out), has_header, header);
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    const int nv = var_mode ? 3 : 1, E = gmm_extra_planes(Kc, Kd, var_mode);
#pragma unroll 4
    for (int k = 0; k < Kc; ++k) {
        const float4 c = state[(int64_t)k * n + p];
        out[(int64_t)(Kc + 3 * k) * n + p] = c.x;
        out[(int64_t)(Kc + 3 * k + 1) * n + p] = c.y;
        out[(int64_t)(Kc + 3 * k + 2) * n + p] = c.z;
        out[(int64_t)(4 * Kc + nv * k) * n + p] = c.w;
    }
#pragma unroll 4
    for (int e = 0; e < E; ++e) {
        const float4 x = state[(int64_t)(Kc + e) * n + p];
        const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int plane = canon_plane(4 * e + i, Kc, Kd, nv);
            if (plane >= 0) out[(int64_t)plane * n + p] = v[i];
        }
    }
}

__global__ __launch_bounds__(kBlock) void gmm_import_kernel(float4* __restrict__ state, const float* __restrict__ in,
                                                            int Kc, int Kd, int var_mode, int npix, StateCheck check) {
    if (!header_matches(check)) return;
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    const int nv = var_mode ? 3 : 1, E = gmm_extra_planes(Kc, Kd, var_mode);
#pragma unroll 4
    for (int k = 0; k < Kc; ++k)
        state[(int64_t)k * n + p] = make_float4(in[(int64_t)(Kc + 3 * k) * n + p], in[(int64_t)(Kc + 3 * k + 1) * n + p],
                                                in[(int64_t)(Kc + 3 * k + 2) * n + p], in[(int64_t)(4 * Kc + nv * k) * n + p]);
#pragma unroll 4
    for (int e = 0; e < E; ++e) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int plane = canon_plane(4 * e + i, Kc, Kd, nv);
            v[i] = plane >= 0 ? in[(int64_t)plane * n + p] : 0.0f;
        }
        state[(int64_t)(Kc + e) * n + p] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

template <int NB, int KC, int KD, bool GEN, int CV>
void launch_step_g(const GmmBatch<NB>& b, unsigned grid, hipStream_t s) {
    constexpr int kPlanes = KC + GmmLayout<KC, KD, CV>::E;
    if (b.a[0].streaming)
        hipLaunchKernelGGL((gmm_step_kernel<NB, KC, KD, true, GEN, CV>), dim3(grid), dim3(kBlock),
                           kPlanes >= kStreamPlanes ? kStreamLds : 0, s, b);
    else
        hipLaunchKernelGGL((gmm_step_kernel<NB, KC, KD, false, GEN, CV>), dim3(grid), dim3(kBlock), 0, s, b);
}

// Kernel variant of a model's constants: 2 per-channel variances, 1 rate or decision
// variant, 0 the defaults compiled in.
int variant(const GmmConsts& c) { return c.var_mode ? 2 : ((c.rho_mode || c.decision) ? 1 : 0); }

template <int NB, int KC, int KD>
hipError_t launch_step_t(const GmmBatch<NB>& b, unsigned grid, hipStream_t s) {
    switch (variant(b.a[0].c)) {
        case 2: launch_step_g<NB, KC, KD, true, 3>(b, grid, s); break;
        case 1: launch_step_g<NB, KC, KD, true, 1>(b, grid, s); break;
        default: launch_step_g<NB, KC, KD, false, 1>(b, grid, s); break;
    }
    return hipGetLastError();
}

template <int NB>
hipError_t launch_batch(const GmmStepArgs* a, int n, int Kc, int Kd, hipStream_t s) {
    GmmBatch<NB> b;
    std::memset(&b, 0, sizeof b);
    b.n = n;
    int64_t grid = 0;
    for (int i = 0; i < n; ++i) {
        b.a[i] = a[i];
        b.first[i] = (int32_t)grid;
        grid += (a[i].npix + kBlock - 1) / kBlock;
    }
    for (int i = n; i <= NB; ++i) b.first[i] = (int32_t)grid;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    const unsigned g = (unsigned)grid;
    switch (Kc * 8 + Kd) {
        case 1 * 8 + 1: return launch_step_t<NB, 1, 1>(b, g, s);
        case 2 * 8 + 2: return launch_step_t<NB, 2, 2>(b, g, s);
        case 3 * 8 + 3: return launch_step_t<NB, 3, 3>(b, g, s);
        case 4 * 8 + 4: return launch_step_t<NB, 4, 4>(b, g, s);
        case 5 * 8 + 5: return launch_step_t<NB, 5, 5>(b, g, s);
        case 6 * 8 + 6: return launch_step_t<NB, 6, 6>(b, g, s);
        case 7 * 8 + 7: return launch_step_t<NB, 7, 7>(b, g, s);
        case 7 * 8 + 3: return launch_step_t<NB, 7, 3>(b, g, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool gmm_supported(int Kc, int Kd) {
    if (Kc == Kd && Kc >= 1 && Kc <= 7) return true;
    return Kc == 7 && Kd == 3;
}

int gmm_batch_key(const GmmStepArgs& a, int Kc, int Kd) {
    return ((Kc * 8 + Kd) * 4 + variant(a.c)) * 2 + (a.streaming ? 1 : 0);
}

hipError_t gmm_launch_step_batch(const GmmStepArgs* a, int n, int Kc, int Kd, hipStream_t s) {
    if (n < 1 || n > kBatchMax) return hipErrorInvalidValue;
    for (int i = 1; i < n; ++i)
        if (gmm_batch_key(a[i], Kc, Kd) != gmm_batch_key(a[0], Kc, Kd)) return hipErrorInvalidValue;
    return n == 1 ? launch_batch<1>(a, n, Kc, Kd, s) : launch_batch<kBatchMax>(a, n, Kc, Kd, s);
}

hipError_t gmm_launch_step(const GmmStepArgs& a, int Kc, int Kd, hipStream_t s) {
    return gmm_launch_step_batch(&a, 1, Kc, Kd, s);
}

hipError_t gmm_launch_init(float4* state, int Kc, int Kd, int npix, const GmmConsts& c,
                           hipStream_t s) {
    const unsigned grid = (unsigned)((npix + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(gmm_init_kernel, dim3(grid), dim3(kBlock), 0, s, state, Kc, Kd, c.var_mode, npix,
                       c.v_init_c, c.v_init_d);
    return hipGetLastError();
}

hipError_t gmm_launch_export(const float4* state, float* out, int Kc, int Kd, int var_mode, int npix,
                             const StateWords* header, hipStream_t s) {
    const unsigned grid = (unsigned)((npix + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(gmm_export_kernel, dim3(grid), dim3(kBlock), 0, s, state, out, Kc, Kd, var_mode, npix,
                       header ? 1 : 0, header ? *header : StateWords());
    return hipGetLastError();
}

hipError_t gmm_launch_import(float4* state, const float* in, int Kc, int Kd, int var_mode, int npix,
                             const StateCheck& check, hipStream_t s) {
    const unsigned grid = (unsigned)((npix + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(gmm_import_kernel, dim3(grid), dim3(kBlock), 0, s, state, in, Kc, Kd, var_mode, npix, check);
    return hipGetLastError();
}

}  // namespace fgs
