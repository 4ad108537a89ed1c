// Adjoint of the RGB-D GMM recursion over a window of frames.
//
// Parameters theta = (alpha, lambda, w_d), read from device memory.  The window
// starts from a fresh model; every frame yields the pre-update score
//   Z_t = (delta_c - lambda^2) + w_d (delta_d - lambda^2)
// (terms only where the model has data; depth only where D > 0), exactly the
// quantity the plain kernel thresholds at 0 for the mask (Sec. 3.1 reading).
//
// Forward: one lane per pixel runs all T frames with the state in registers,
// writing Z_t, the term flags, a 64-bit record of the step's discrete choices
// (argmin of delta, matched Gaussian or replacement, variance floor, ranking)
// for both mixtures, the means and variances before each segment of frames but the
// first and before the last frame, and what the last segment's steps changed.
//
// Backward: with the recorded choices held fixed the weights reach Z only through
// discrete choices, so their adjoints vanish; alpha's gradient flows through the
// matched Gaussian's mean and variance updates.  A step changes one Gaussian of each
// mixture and reorders them, so the reverse sweep undoes it from the recorded ranking and
// the changed Gaussian's mean and variance before the step (16 bytes of the colour mixture,
// 8 of the depth mixture).  The forward has kept those of the last segment where that is the whole
// window (ALL) or one of two segments.  For the others each lane replays the
// segment's means and variances from its checkpoint (the forward's operations, so the same
// values) into the same buffer, then sweeps it; a backward after that replays the last segment too
// (`kept`, in device memory: a captured backward may run again without its forward).  Per-lane
// gradients accumulate in fp64 and are reduced in a fixed order (wavefront and block tree, then
// one block over the block partials), so the result is deterministic.
//
// Measured, 64 frames of 640x480, K = 3 (forward, backward): with the whole state stored to
// scratch per frame (72 bytes a pixel and frame) 310 and 657 us; with the changed Gaussians and
// a replay 275 and 409; with the changed Gaussians of every frame kept 273 and 240; with weights
// and ranks as in gmm_device.h 240 and 251; with 32-bit lane offsets (lane_of, opaque) 231 and 217.
// That takes 2,120 bytes a pixel; within the 1,952 that checkpoint_every = 16 asks for, 54 frames are
// kept and 10 replayed: 237 and 222 (both passes 459 us against 434).
// The forward is bound by its vector instructions (450 per wavefront and frame, the ALUs all but
// always busy); the backward reads 41 bytes a pixel and frame (3.7 TB/s) beside 380 instructions.
// 4,800 wavefronts are 4.7 a SIMD, hence the launch bound of 5 (96 registers) for K <= 3: with 111
// registers a sixth of them ran in a second round.
#include <type_traits>

#include "device_common.h"
#include "fgs_internal.h"
#include "gmm_device.h"

namespace fgs {

namespace {

constexpr int kBlock = 256;

// Record layout, per mixture (colour in bits 0..31, depth in 32..63):
//   bit 0 term, bits 1-3 argmin, bit 4 active, bits 5-7 matched (7 = replaced),
//   bit 8 floor applied, bits 9.. ranking (3 bits per rank).
template <int C>
__device__ __forceinline__ uint32_t pack_rec(const MixRec<C>& r, bool term, bool active) {
    return (term ? 1u : 0u) | ((uint32_t)r.argmin << 1) | (active ? 16u : 0u) |
           ((uint32_t)(r.kstar < 0 ? 7 : r.kstar) << 5) | (r.clamp ? 256u : 0u) | (r.perm << 9);
}

// Element p of a plane whose base is the same for the whole launch, through a 32-bit byte offset
// (p < 2^28 and elements of at most 16 bytes): the base stays in scalar registers.
template <class T>
__device__ __forceinline__ T& lane_of(T* base, uint32_t p) {
    char* b = reinterpret_cast<char*>(const_cast<std::remove_const_t<T>*>(base));
    return *reinterpret_cast<T*>(b + (uint32_t)(p * (uint32_t)sizeof(T)));
}

// The lane's pixel, opaque to the compiler in each frame: it would otherwise carry a 64-bit address
// per plane and lane through the loop (two registers and a 64-bit addition each), and keep the
// addresses used in the last frame only in scratch memory.
__device__ __forceinline__ uint32_t opaque(uint32_t p) {
    asm volatile("" : "+v"(p));
    return p;
}

// Plane order of the mean/variance snapshots: colour mu[k][c], colour v[k],
// depth mu[k], depth v[k]; F = 6K floats per pixel.
template <int K>
struct MV {
    float muc[K][3], vc[K], mud[K], vd[K];
};

template <int K>
__device__ __forceinline__ void store_mv(const MV<K>& s, float* base, int64_t npix, uint32_t p, bool colour, bool depth) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (colour) {
#pragma unroll
            for (int c = 0; c < 3; ++c) lane_of(base + (int64_t)(3 * k + c) * npix, p) = s.muc[k][c];
            lane_of(base + (int64_t)(3 * K + k) * npix, p) = s.vc[k];
        }
        if (depth) {
            lane_of(base + (int64_t)(4 * K + k) * npix, p) = s.mud[k];
            lane_of(base + (int64_t)(5 * K + k) * npix, p) = s.vd[k];
        }
    }
}

template <int K>
__device__ __forceinline__ void load_mv(MV<K>& s, const float* base, int64_t npix, uint32_t p) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) s.muc[k][c] = lane_of(base + (int64_t)(3 * k + c) * npix, p);
        s.vc[k] = lane_of(base + (int64_t)(3 * K + k) * npix, p);
        s.mud[k] = lane_of(base + (int64_t)(4 * K + k) * npix, p);
        s.vd[k] = lane_of(base + (int64_t)(5 * K + k) * npix, p);
    }
}

struct Input {
    float Xc[3];
    float Xd[1];
    bool valid;
};

// The bytes of one pixel of frame t as read; a frame's base is the same for the whole launch,
// so a lane keeps one 32-bit offset.  Read one frame ahead of their use: a window is a serial
// chain of frames per lane, with few wavefronts beside it to hide a read's latency.
struct Raw {
    uint32_t r, g, b, d;
};
__device__ __forceinline__ Raw read_input(const GmmWindowArgs& a, int t, uint32_t p) {
    const uint8_t* px = a.rgb + (int64_t)t * a.npix * 3 + 3u * p;
    return Raw{px[0], px[1], px[2], lane_of(a.depth + (int64_t)t * a.npix, p)};
}
__device__ __forceinline__ Input input_of(const GmmWindowArgs& a, const Raw& raw) {
    Input in;
    in.Xc[0] = (float)raw.r;
    in.Xc[1] = (float)raw.g;
    in.Xc[2] = (float)raw.b;
    in.valid = raw.d > 0u;
    in.Xd[0] = (float)depth_code(raw.d, a.c.depth_max_mm, a.c.depth_div);
    return in;
}

// SPLIT: the mixtures of a pixel run on two wavefronts of a workgroup of 128 pixels, the depth
// mixture's handing its term to the colour mixture's through LDS once a frame.  A small window
// leaves SIMDs idle while each wavefront walks its chain of T frames through both mixtures.
template <int K, bool ALL, bool SPLIT>
__global__ __launch_bounds__(kBlock, K <= 3 ? 5 : 3) void gmm_window_forward_kernel(GmmWindowArgs a) {
    constexpr int kPixels = SPLIT ? kBlock / 2 : kBlock;
    __shared__ float term_of[SPLIT ? 2 : 1][SPLIT ? kPixels : 1];  // by frame parity: w_d (delta_d - lambda^2)
    __shared__ uint8_t used_of[SPLIT ? 2 : 1][SPLIT ? kPixels : 1];
    const int lane = (int)threadIdx.x % kPixels;
    const int part = SPLIT ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kPixels) : 0;
    const bool do_c = !SPLIT || part == 0, do_d = !SPLIT || part == 1;
    const bool inside = (int)blockIdx.x * kPixels + lane < a.npix;
    if (!SPLIT && !inside) return;
    const uint32_t p = inside ? blockIdx.x * kPixels + lane : a.npix - 1;  // (every lane meets the barriers)
    const float alpha = a.theta[0], lam = a.theta[1], wd = a.theta[2];
    const float lam2 = lam * lam;
    const bool sane = alpha > 0.0f && alpha < 1.0f &&
                      gmm_sane(lam, wd, a.c.v_min_c, a.c.v_min_d, a.c.v_init_c, a.c.v_init_d);
    Mix<K, 3> mc;
    Mix<K, 1> md;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        mc.w[k] = 0.f;
        mc.mu[k][0] = mc.mu[k][1] = mc.mu[k][2] = 0.f;
        mc.v[k] = a.c.v_init_c;
        md.w[k] = 0.f;
        md.mu[k][0] = 0.f;
        md.v[k] = a.c.v_init_d;
    }
    const int64_t F = 6 * K;
    auto snapshot = [&](int slot, uint32_t up) __attribute__((always_inline)) {
        if (!inside) return;
        MV<K> s;
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int c = 0; c < 3; ++c) s.muc[k][c] = mc.mu[k][c];
            s.vc[k] = mc.v[k];
            s.mud[k] = md.mu[k][0];
            s.vd[k] = md.v[k];
        }
        store_mv<K>(s, a.ckpt + (int64_t)slot * F * a.npix, a.npix, up, do_c, do_d);
    };
    const int kept_from = ALL ? 0 : a.keeps() ? a.T - a.E : a.T;
    Raw next = read_input(a, 0, p);
    auto frame = [&](int t, auto keep) __attribute__((always_inline)) {
        constexpr bool KEEP = decltype(keep)::value;
        const Raw raw = next;
        const uint32_t up = opaque(p);
        next = read_input(a, min(t + 1, a.T - 1), up);
        __builtin_amdgcn_sched_barrier(0);
        if (KEEP && t + 1 == a.T) snapshot(0, up);
        const int64_t row = (int64_t)(t - kept_from) * a.npix;
        const Input in = input_of(a, raw);
        const int64_t o = (int64_t)t * a.npix;
        bool used_c = false, used_d = false;
        float dc = 0.0f, dd = 0.0f;
        MixRec<3> rc;
        MixRec<1> rd;
        if (do_c) {
            mixture_step_rec(mc, in.Xc, true, alpha, lam2, a.c.T_bg, a.c.w_init, a.c.v_init_c, a.c.v_min_c, sane,
                             used_c, dc, rc);
            if (KEEP && inside) lane_of(a.scratch4() + row, up) = make_float4(rc.mu[0], rc.mu[1], rc.mu[2], rc.v);
        }
        if (do_d) {
            mixture_step_rec(md, in.Xd, in.valid, alpha, lam2, a.c.T_bg, a.c.w_init, a.c.v_init_d, a.c.v_min_d, sane,
                             used_d, dd, rd);
            if (KEEP && inside) lane_of(a.scratch2() + row, up) = make_float2(rd.mu[0], rd.v);
        }
        const bool term_c = used_c;
        bool term_d = in.valid && used_d;
        const float tc = dc - lam2;
        float td = wd * (dd - lam2);
        if (SPLIT) {
            uint32_t* halves = reinterpret_cast<uint32_t*>(a.rec + o);
            if (do_d) {
                term_of[t & 1][lane] = td;
                used_of[t & 1][lane] = term_d ? 1 : 0;
                if (inside) lane_of(halves + 1, 2 * up) = pack_rec(rd, term_d, in.valid);
            }
            __syncthreads();  // (the other parity's slots are written while these are read)
            if (!do_c) return;
            td = term_of[t & 1][lane];
            term_d = used_of[t & 1][lane] != 0;
            if (!inside) return;
            lane_of(halves, 2 * up) = pack_rec(rc, term_c, true);
        } else {
            lane_of(a.rec + o, up) =
                (uint64_t)pack_rec(rc, term_c, true) | ((uint64_t)pack_rec(rd, term_d, in.valid) << 32);
        }
        const float Z = term_c ? (term_d ? tc + td : tc) : (term_d ? td : 0.0f);
        lane_of(a.Z + o, up) = Z;
        lane_of(a.has + o, up) = (term_c || term_d) ? 1 : 0;
    };
    if (!ALL) {
        const int replayed = a.keeps() ? a.nseg - 1 : a.nseg;
        for (int seg = 0; seg < replayed; ++seg) {
            if (seg > 0) snapshot(seg, opaque(p));
            const int t1 = a.first_of(seg + 1);
#pragma unroll 1
            for (int t = a.first_of(seg); t < t1; ++t) frame(t, std::false_type{});
        }
        if (a.keeps() && a.E > 1) snapshot(a.nseg - 1, opaque(p));
    }
#pragma unroll 1
    for (int t = kept_from; t < a.T; ++t) frame(t, std::true_type{});
    if (!ALL && threadIdx.x == 0) a.kept[blockIdx.x] = a.keeps() ? 1u : 0u;
}

// A recorded choice, unpacked.
struct Choice {
    bool term, active, matched, clamp, ranked;  // ranked: the step reordered the Gaussians
    int amin, tgt;                              // tgt: the Gaussian matched, or replaced (the last)
};
template <int K>
__device__ __forceinline__ Choice choice_of(uint32_t r) {
    uint32_t id = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) id |= (uint32_t)k << (3 * k);
    Choice c;
    const int ks = (int)((r >> 5) & 7u);
    c.term = (r & 1u) != 0u;
    c.active = (r & 16u) != 0u;
    c.matched = ks != 7;
    c.clamp = (r & 256u) != 0u;
    c.ranked = (r >> 9) != id;
    c.amin = (int)((r >> 1) & 7u);
    c.tgt = c.matched ? ks : K - 1;
    return c;
}

// One Gaussian's mean and variance (or their adjoints) out of K, and back into its place.
template <int K, int C>
__device__ __forceinline__ void pick(const float (&m)[K][C], const float (&v)[K], int at, float (&pm)[C], float& pv) {
#pragma unroll
    for (int c = 0; c < C; ++c) pm[c] = m[0][c];
    pv = v[0];
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const bool here = k == at;
#pragma unroll
        for (int c = 0; c < C; ++c) pm[c] = here ? m[k][c] : pm[c];
        pv = here ? v[k] : pv;
    }
}
template <int K, int C>
__device__ __forceinline__ void put(float (&m)[K][C], float (&v)[K], int at, const float (&pm)[C], float pv) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool here = k == at;
#pragma unroll
        for (int c = 0; c < C; ++c) m[k][c] = here ? pm[c] : m[k][c];
        v[k] = here ? pv : v[k];
    }
}

// Rank r holds the Gaussian that was at (perm >> 3r) & 7: into that order (rank), and back.
template <int K, int C, bool BACK>
__device__ __forceinline__ void reorder(float (&m)[K][C], float (&v)[K], uint32_t perm) {
    float om[K][C], ov[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int c = 0; c < C; ++c) om[k][c] = m[0][c];
        ov[k] = v[0];
    }
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const int src = (int)((perm >> (3 * r)) & 7u);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int to = BACK ? k : r, from = BACK ? r : k;
            if (from == 0) continue;
            const bool here = src == k;
#pragma unroll
            for (int c = 0; c < C; ++c) om[to][c] = here ? m[from][c] : om[to][c];
            ov[to] = here ? v[from] : ov[to];
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int c = 0; c < C; ++c) m[k][c] = om[k][c];
        v[k] = ov[k];
    }
}

// Replay of one mixture's means/variances with recorded choices (fp32, the forward's operations
// in the forward's order).  pm, pv: the changed Gaussian before the step.  `last`: only those are
// wanted, the state stays.
template <int K, int C>
__device__ __forceinline__ void replay_mix(float (&mu)[K][C], float (&v)[K], const float (&X)[C], uint32_t r,
                                           float alpha, float v_init, float v_min, bool last, float (&pm)[C],
                                           float& pv) {
    const Choice ch = choice_of<K>(r);
    pick(mu, v, ch.tgt, pm, pv);
    if (last) return;
    if (!ch.active) return;
    float mn[C];
#pragma unroll
    for (int c = 0; c < C; ++c) mn[c] = pm[c] + alpha * (X[c] - pm[c]);
    float e = X[0] - mn[0];
    float d2 = e * e;
#pragma unroll
    for (int c = 1; c < C; ++c) {
        e = X[c] - mn[c];
        d2 = d2 + e * e;
    }
    const float vt = pv + alpha * (d2 - pv);
    const float vn = ch.matched ? (ch.clamp ? v_min : vt) : v_init;
#pragma unroll
    for (int c = 0; c < C; ++c) mn[c] = ch.matched ? mn[c] : X[c];
    put(mu, v, ch.tgt, mn, vn);
    if (__any(ch.ranked)) reorder<K, C, false>(mu, v, r >> 9);
}

// x / v with r = 1 / v at hand: one correction step (a quotient that is not finite stays).
__device__ __forceinline__ float quotient(float x, float v, float r) {
    const float q = x * r;
    const float c = __builtin_fmaf(__builtin_fmaf(-v, q, x), r, q);
    return __builtin_isfinite(c) ? c : q;
}

// One step backwards for one mixture.  In: the means/variances after the step (`undo`) or before
// it, the adjoint (am, av) of those after it, and the changed Gaussian before it (pm, pv).  Out:
// the means/variances before the step, their adjoint with the score's added (g = dL/dZ times
// the mixture's factor in Z), the step's contribution to d/d alpha, and delta.
template <int K, int C>
__device__ __forceinline__ void reverse_mix(float (&mu)[K][C], float (&v)[K], const float (&X)[C], uint32_t r,
                                            float alpha, bool undo, const float (&pm)[C], float pv, float g,
                                            float (&am)[K][C], float (&av)[K], double& ga, float& delta) {
    const Choice ch = choice_of<K>(r);
    if (ch.active) {
        if (__any(ch.ranked)) {
            reorder<K, C, true>(am, av, r >> 9);
            if (undo) reorder<K, C, true>(mu, v, r >> 9);
        }
        if (undo) put(mu, v, ch.tgt, pm, pv);
        float bm[C], bv;
        pick(am, av, ch.tgt, bm, bv);
        float mn[C];
#pragma unroll
        for (int c = 0; c < C; ++c) mn[c] = pm[c] + alpha * (X[c] - pm[c]);
        float d2 = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c) d2 += (X[c] - mn[c]) * (X[c] - mn[c]);
        const float avt = ch.clamp ? 0.f : bv;
        float gam = avt * (d2 - pv);
        float nm[C], nv = (1.0f - alpha) * avt;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float amn = bm[c] + avt * alpha * (-2.0f) * (X[c] - mn[c]);
            gam += amn * (X[c] - pm[c]);
            nm[c] = ch.matched ? (1.0f - alpha) * amn : 0.f;
        }
        nv = ch.matched ? nv : 0.f;
        put(am, av, ch.tgt, nm, nv);
        ga += (double)(ch.matched ? gam : 0.f);
    }
    if (ch.term) {  // Z depends on the state before the step through delta = |X - mu_a|^2 / v_a
        float sm[C], sv, tm[C], tv;
        pick(mu, v, ch.amin, sm, sv);
        pick(am, av, ch.amin, tm, tv);
        float e = X[0] - sm[0];
        float d2 = e * e;
#pragma unroll
        for (int c = 1; c < C; ++c) {
            e = X[c] - sm[c];
            d2 = d2 + e * e;
        }
        const float rv = 1.0f / sv;
        delta = quotient(d2, sv, rv);
#pragma unroll
        for (int c = 0; c < C; ++c) tm[c] += quotient(g * (-2.0f) * (X[c] - sm[c]), sv, rv);
        tv += g * quotient(-delta, sv, rv);
        put(am, av, ch.amin, tm, tv);
    }
}

// Sums of three values over the block, in a fixed order; the result is lane 0's.
__device__ __forceinline__ void block_sum3(double (&x)[3], double (*sh)[3]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < 3; ++i) x[i] += __shfl_xor(x[i], off, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < 3; ++i) sh[threadIdx.x >> 6][i] = x[i];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w)
#pragma unroll
            for (int i = 0; i < 3; ++i) x[i] += sh[w][i];
}

// What the reverse sweep reads for one frame, one frame ahead of its use.
struct BackRead {
    Raw raw;
    uint64_t rec;
    float4 pc;   // the colour Gaussian the step changed, before it: mean, variance
    float2 pd;   // the depth one
    float g;
};

// SPLIT: the mixtures on wavefronts of their own, as in the forward (they share nothing here).
template <int K, bool ALL, bool SPLIT>
__global__ __launch_bounds__(kBlock, K <= 3 ? 5 : 3) void gmm_window_backward_kernel(GmmWindowArgs a) {
    __shared__ double sh[kBlock / 64][3];
    constexpr int kPixels = SPLIT ? kBlock / 2 : kBlock;
    const int part = SPLIT ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kPixels) : 0;
    const bool do_c = !SPLIT || part == 0, do_d = !SPLIT || part == 1;
    const int p = blockIdx.x * kPixels + (int)threadIdx.x % kPixels;
    double acc[3] = {0.0, 0.0, 0.0};  // alpha, lambda, w_depth
    if (p < a.npix) {
        const float alpha = a.theta[0], lam = a.theta[1], wd = a.theta[2];
        const float lam2 = lam * lam;
        const int64_t F = 6 * K, npix = a.npix;
        float4* sc = a.scratch4();
        float2* sd = a.scratch2();
        float amc[K][3], avc[K], amd[K][1], avd[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            amc[k][0] = amc[k][1] = amc[k][2] = 0.f;
            avc[k] = 0.f;
            amd[k][0] = 0.f;
            avd[k] = 0.f;
        }
        const bool kept = ALL || a.kept[blockIdx.x] != 0u;
        for (int seg = ALL ? 0 : a.nseg - 1; seg >= 0; --seg) {
            const bool there = ALL || (kept && seg == a.nseg - 1);  // the forward's, and the state before t1 - 1
            const int t0 = ALL ? 0 : a.first_of(seg), t1 = ALL ? a.T : a.first_of(seg + 1);
            float muc[K][3], vc[K], mud[K][1], vd[K];
            if (!ALL && !there && seg == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    muc[k][0] = muc[k][1] = muc[k][2] = mud[k][0] = 0.f;
                    vc[k] = a.c.v_init_c;
                    vd[k] = a.c.v_init_d;
                }
            } else {
                MV<K> s;
                load_mv<K>(s, a.ckpt + (int64_t)(there ? 0 : a.ckpt_of(seg)) * F * npix, npix, opaque(p));
#pragma unroll
                for (int k = 0; k < K; ++k) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) muc[k][c] = s.muc[k][c];
                    vc[k] = s.vc[k];
                    mud[k][0] = s.mud[k];
                    vd[k] = s.vd[k];
                }
            }
            if (!ALL && !there) {
                Raw nraw = read_input(a, t0, p);
                uint64_t nrec = lane_of(a.rec + (int64_t)t0 * npix, p);
#pragma unroll 1
                for (int t = t0; t < t1; ++t) {
                    const Raw raw = nraw;
                    const uint64_t rr = nrec;
                    const uint32_t up = opaque(p);
                    const int tn = min(t + 1, t1 - 1);
                    nraw = read_input(a, tn, up);
                    nrec = lane_of(a.rec + (int64_t)tn * npix, up);
                    __builtin_amdgcn_sched_barrier(0);
                    const Input in = input_of(a, raw);
                    const bool last = t + 1 == t1;
                    float pm[3] = {}, pv = 0.0f, qm[1] = {}, qv = 0.0f;
                    if (do_c) replay_mix<K, 3>(muc, vc, in.Xc, (uint32_t)rr, alpha, a.c.v_init_c, a.c.v_min_c, last, pm, pv);
                    if (do_d) replay_mix<K, 1>(mud, vd, in.Xd, (uint32_t)(rr >> 32), alpha, a.c.v_init_d, a.c.v_min_d, last, qm,
                                     qv);
                    if (do_c) lane_of(sc + (int64_t)(t - t0) * npix, up) = make_float4(pm[0], pm[1], pm[2], pv);
                    if (do_d) lane_of(sd + (int64_t)(t - t0) * npix, up) = make_float2(qm[0], qv);
                }
            }
            auto read = [&](int t) {
                BackRead b = {};
                const uint32_t up = opaque(p);
                b.raw = read_input(a, t, up);
                b.rec = lane_of(a.rec + (int64_t)t * npix, up);
                if (do_c) b.pc = lane_of(sc + (int64_t)(t - t0) * npix, up);
                if (do_d) b.pd = lane_of(sd + (int64_t)(t - t0) * npix, up);
                b.g = lane_of(a.dZ + (int64_t)t * npix, up);
                return b;
            };
            BackRead next = read(t1 - 1);
#pragma unroll 1
            for (int t = t1 - 1; t >= t0; --t) {
                const BackRead b = next;
                next = read(max(t - 1, t0));
                __builtin_amdgcn_sched_barrier(0);
                const Input in = input_of(a, b.raw);
                const bool undo = t + 1 != t1;
                const uint32_t rc = (uint32_t)b.rec, rd = (uint32_t)(b.rec >> 32);
                const float pm[3] = {b.pc.x, b.pc.y, b.pc.z}, qm[1] = {b.pd.x};
                float dc = 0.f, dd = 0.f;
                if (do_c) reverse_mix<K, 3>(muc, vc, in.Xc, rc, alpha, undo, pm, b.pc.w, b.g, amc, avc, acc[0], dc);
                if (do_d) reverse_mix<K, 1>(mud, vd, in.Xd, rd, alpha, undo, qm, b.pd.y, b.g * wd, amd, avd, acc[0], dd);
                if (do_c && (rc & 1u)) acc[1] += (double)(b.g * (-2.0f * lam));
                if (do_d && (rd & 1u)) {
                    acc[1] += (double)(b.g * (-2.0f * lam) * wd);
                    acc[2] += (double)(b.g * (dd - lam2));
                }
            }
        }
    }
    block_sum3(acc, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) a.partial[3 * blockIdx.x + i] = acc[i];
        if (!ALL) a.kept[blockIdx.x] = 0u;  // (read before block_sum3's barrier)
    }
}

__global__ __launch_bounds__(kBlock) void gmm_window_reduce_kernel(const double* partial, int nblocks, double* out) {
    __shared__ double sh[kBlock / 64][3];
    double acc[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nblocks; b += kBlock)
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[i] += partial[3 * b + i];
    block_sum3(acc, sh);
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < 3; ++i) out[i] = acc[i];
}

}  // namespace

bool gmm_window_supported(int K) { return K >= 1 && K <= 5; }

namespace {

// Up to kSplitPixels (with the mixtures split: four wavefronts a SIMD) and with three Gaussians or more
// the mixtures run on wavefronts of their own: forward of 24 frames, with its call, 131x93, K = 5: 95.6 ->
// 70.5 us, K = 3: 70.7 -> 56.2; 400x300, K = 5: 104 -> 90, K = 3: 77.5 -> 70.5.  Larger windows fill the
// SIMDs anyway and read their frames twice for nothing (480x360, K = 3: 88 -> 92.6, K = 5: 126.5 ->
// 124.7; 640x480, K = 3: 118 -> 157); K = 1, whose mixtures are short, 40-44 either way.  The
// kernels alone, 131x93, K = 5: forward 71.3 -> 53.2 us, backward 39.2 -> 29.6.
constexpr int kSplitPixels = 1 << 17;
constexpr bool splits(int K, int npix) { return K >= 3 && npix <= kSplitPixels; }

}  // namespace

int gmm_window_blocks(int K, int npix) {
    const int pixels = splits(K, npix) ? kBlock / 2 : kBlock;
    return (npix + pixels - 1) / pixels;
}

namespace {

template <int K, bool ALL>
void launch_forward_of(const GmmWindowArgs& a, hipStream_t s) {
    if constexpr (splits(K, 1)) {
        if (splits(K, a.npix)) {
            hipLaunchKernelGGL((gmm_window_forward_kernel<K, ALL, true>), dim3((unsigned)gmm_window_blocks(K, a.npix)),
                               dim3(kBlock), 0, s, a);
            return;
        }
    }
    hipLaunchKernelGGL((gmm_window_forward_kernel<K, ALL, false>), dim3((unsigned)gmm_window_blocks(K, a.npix)),
                       dim3(kBlock), 0, s, a);
}
template <int K>
void launch_forward(const GmmWindowArgs& a, hipStream_t s) {
    if (a.nseg == 1) launch_forward_of<K, true>(a, s);
    else launch_forward_of<K, false>(a, s);
}
template <int K, bool ALL>
void launch_backward_of(const GmmWindowArgs& a, int blocks, hipStream_t s) {
    if constexpr (splits(K, 1)) {
        if (splits(K, a.npix)) {
            hipLaunchKernelGGL((gmm_window_backward_kernel<K, ALL, true>), dim3(blocks), dim3(kBlock), 0, s, a);
            return;
        }
    }
    hipLaunchKernelGGL((gmm_window_backward_kernel<K, ALL, false>), dim3(blocks), dim3(kBlock), 0, s, a);
}
template <int K>
void launch_backward(const GmmWindowArgs& a, int blocks, hipStream_t s) {
    if (a.nseg == 1) launch_backward_of<K, true>(a, blocks, s);
    else launch_backward_of<K, false>(a, blocks, s);
}

}  // namespace

hipError_t gmm_window_launch_forward(const GmmWindowArgs& a, int K, hipStream_t s) {
    switch (K) {
        case 1: launch_forward<1>(a, s); break;
        case 2: launch_forward<2>(a, s); break;
        case 3: launch_forward<3>(a, s); break;
        case 4: launch_forward<4>(a, s); break;
        case 5: launch_forward<5>(a, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t gmm_window_launch_backward(const GmmWindowArgs& a, int K, hipStream_t s) {
    const int nb = gmm_window_blocks(K, a.npix);
    switch (K) {
        case 1: launch_backward<1>(a, nb, s); break;
        case 2: launch_backward<2>(a, nb, s); break;
        case 3: launch_backward<3>(a, nb, s); break;
        case 4: launch_backward<4>(a, nb, s); break;
        case 5: launch_backward<5>(a, nb, s); break;
        default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gmm_window_reduce_kernel, dim3(1), dim3(kBlock), 0, s, a.partial, nb, a.dtheta);
    return hipGetLastError();
}

}  // namespace fgs
