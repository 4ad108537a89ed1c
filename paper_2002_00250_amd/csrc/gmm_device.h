// The per-pixel step of one Gaussian mixture (colour: C = 3 channels, depth:
// C = 1), shared by the plain per-frame kernel and the adjoint window kernels so
// that both run the same IEEE binary32 operations in the same order (Sec. 3.1 and
// the Stauffer-Grimson recursion it builds on).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"
#include "fgs_internal.h"

namespace fgs {

// One mixture: K Gaussians over C channels.  CV = 1: one variance per Gaussian (v);
// CV = 3: one per channel, channel 0 in v and channels 1, 2 in vx.
template <int K, int C, int CV = 1>
struct Mix {
    float w[K];
    float mu[K][C];
    float v[K];
    float vx[K][CV == 3 ? 2 : 1];
};

// The single variance of Gaussian k: v, or the sum of the per-channel variances.
template <int K, int C, int CV>
__device__ __forceinline__ float var_sum(const Mix<K, C, CV>& m, int k) {
    if constexpr (CV == 3) return (m.v[k] + m.vx[k][0]) + m.vx[k][1];
    else return m.v[k];
}

// The discrete choices of one step, recorded for the adjoint: the Gaussian that
// attains delta, the matched Gaussian (-1: replacement), whether the variance floor
// applied, and the ranking (3 bits per rank: the pre-ranking index now at that rank).
template <int C>
struct MixRec {
    int argmin;
    int kstar;
    bool clamp;
    uint32_t perm;
    float mu[C], v;  // the changed Gaussian's mean and variance before the step
};

// Correctly rounded divisions and square roots are most of a step's arithmetic (K = 3, both
// mixtures: 18 divisions and 6 square roots, about 280 of 800 vector instructions), and most
// of them only feed comparisons: is q below lambda^2, which q is the least, is the score
// negative, is one rank key above the next.  Those are decided on approximate values
// (hardware reciprocals, a relative error below 2^-21) where these differ by more than
// kMargin = 2^-17 of themselves; a wavefront in which some lane's values are closer than that
// decides on the correctly rounded ones instead, so every result is bit for bit that of the
// rounded operations (K = 5 on the 1280x720 scene: 950 -> 710 vector instructions per
// wavefront executed).  Margins also rule out what the approximations do not carry: NaN,
// infinities and the ends of the exponent range all come out as "not certain".
constexpr float kMargin = 1.0f / 131072.0f;
constexpr float kBig = 1.0e30f;
constexpr float kTiny = 1.0e-35f;

__device__ __forceinline__ bool any_lane(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// What the classification of one mixture finds.
struct MixClass {
    bool used;    // the mixture has data
    float delta;  // min q over the background Gaussians (rounded if `rounded`)
    int amin;     // the first rank attaining it
    int ks;       // the matched rank, -1: none
    bool sure;    // the approximate choices are certain to be the rounded ones', and every
                  // weight, variance and distance is in [0, kBig)
    float d2, v;  // classify_approx with ARG: delta's squared distance and variance
};

// Squared distance of X to Gaussian k.
template <int K, int C, int CV>
__device__ __forceinline__ float dist2(const Mix<K, C, CV>& m, const float (&X)[C], int k) {
    float e = X[0] - m.mu[k][0];
    float d2 = e * e;
#pragma unroll
    for (int c = 1; c < C; ++c) {
        e = X[c] - m.mu[k][c];
        d2 = d2 + e * e;
    }
    return d2;
}

// Squared distance of X to Gaussian k over its variance, correctly rounded step by step.
template <int K, int C, int CV>
__device__ __forceinline__ float q_rounded(const Mix<K, C, CV>& m, const float (&X)[C], int k) {
    if constexpr (CV == 3) {  // squared Mahalanobis distance, diagonal covariance
        float e = X[0] - m.mu[k][0];
        float acc = (e * e) / m.v[k];
        e = X[1] - m.mu[k][1];
        acc = acc + (e * e) / m.vx[k][0];
        e = X[2] - m.mu[k][2];
        acc = acc + (e * e) / m.vx[k][1];
        return acc;
    } else {
        return dist2(m, X, k) / m.v[k];
    }
}

// The same with approximate reciprocals; d2 (CV = 1): the squared distance.
template <int K, int C, int CV>
__device__ __forceinline__ float q_approx(const Mix<K, C, CV>& m, const float (&X)[C], int k, float& d2) {
    if constexpr (CV == 3) {
        d2 = 0.0f;
        float e = X[0] - m.mu[k][0];
        float acc = (e * e) * __builtin_amdgcn_rcpf(m.v[k]);
        e = X[1] - m.mu[k][1];
        acc = acc + (e * e) * __builtin_amdgcn_rcpf(m.vx[k][0]);
        e = X[2] - m.mu[k][2];
        return acc + (e * e) * __builtin_amdgcn_rcpf(m.vx[k][1]);
    } else {
        d2 = dist2(m, X, k);
        return d2 * __builtin_amdgcn_rcpf(m.v[k]);
    }
}

// The background set: the leading ranks whose weights first sum past T_bg; if they never do,
// as many leading ranks as have data.
template <int K, int C, int CV>
__device__ __forceinline__ void background(const Mix<K, C, CV>& m, float T_bg, bool (&bg)[K]) {
    int n = 0;
    bool found = false;
    float cum = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        bg[k] = !found;
        cum = cum + m.w[k];
        found = found || cum > T_bg;
        n += (m.w[k] > 0.0f) ? 1 : 0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) bg[k] = bg[k] && (found || k < n);
}

// delta, its rank and the matched rank for the values q; the least background value that is
// not delta's own (infinity if there is none).
template <int K, int C, int CV>
__device__ __forceinline__ float choose(MixClass& r, const Mix<K, C, CV>& m, const float (&q)[K], const bool (&bg)[K],
                                        float lam2) {
    float next = INFINITY;
    r.delta = q[0];
    r.amin = 0;
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const bool less = bg[k] && q[k] < r.delta;
        const float other = less ? r.delta : (bg[k] ? q[k] : INFINITY);
        next = other < next ? other : next;
        r.delta = less ? q[k] : r.delta;
        r.amin = less ? k : r.amin;
    }
    r.ks = -1;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) r.ks = m.w[k] > 0.0f && q[k] < lam2 ? k : r.ks;
    return next;
}

// Classify on rounded values.
template <int K, int C, int CV>
__device__ __forceinline__ MixClass classify_rounded(const Mix<K, C, CV>& m, const float (&X)[C], float lam2, float T_bg) {
    float q[K];
#pragma unroll
    for (int k = 0; k < K; ++k) q[k] = q_rounded(m, X, k);
    MixClass r;
    r.used = m.w[0] > 0.0f;
    r.sure = true;
    bool bg[K];
    background(m, T_bg, bg);
    choose(r, m, q, bg, lam2);
    return r;
}

// Classify on approximate values; `sure` says where every choice is certain.  ARG: the rank
// attaining delta counts as a choice too (its runner-up must be clearly above it).
template <int K, int C, int CV, bool ARG>
__device__ __forceinline__ MixClass classify_approx(const Mix<K, C, CV>& m, const float (&X)[C], float lam2, float T_bg) {
    float q[K], d2[K];
    uint32_t top = 0u;  // the largest bit pattern: at or above kBig's for a sign, an infinity or a NaN
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        q[k] = q_approx(m, X, k, d2[k]);
        ok = ok && fabsf(q[k] - lam2) > kMargin * lam2;
        top = umax(top, umax(__float_as_uint(q[k]), __float_as_uint(m.v[k])));
        top = umax(top, __float_as_uint(m.w[k]));
        if constexpr (CV == 3) top = umax(top, umax(__float_as_uint(m.vx[k][0]), __float_as_uint(m.vx[k][1])));
    }
    bool bg[K];
    background(m, T_bg, bg);
    MixClass r;
    r.used = m.w[0] > 0.0f;
    const float next = choose(r, m, q, bg, lam2);
    if constexpr (ARG) {
        r.d2 = d2[0];
        r.v = m.v[0];
#pragma unroll
        for (int k = 1; k < K; ++k) {
            r.d2 = k == r.amin ? d2[k] : r.d2;
            r.v = k == r.amin ? m.v[k] : r.v;
        }
    }
    if constexpr (ARG && K > 1) ok = ok && next > __builtin_fmaf(kMargin, r.delta, r.delta) + kTiny;
    r.sure = ok && top < __float_as_uint(kBig);
    return r;
}

// w[k] / S, correctly rounded, S the sum of the w.  Where no lane holds a value outside
// [2^-60, 2^60] but zero weights, the quotients share one reciprocal (Markstein's method: the
// hardware's refined once, then each product corrected by its fused remainder: 3 instructions a
// quotient instead of a division's 11 and its own reciprocal); no step there rounds in the
// subnormal range or overflows.  Compared with the division over all 2^46 pairs of significands
// on gfx950: no quotient differs (without the refinement 47,045 do).  With the ranking on
// products below, the window's forward at 640x480, K = 3, 64 frames, bound by its instructions:
// 270 -> 251 us; the per-frame steps, bound by memory, within 1 % (K = 5 at 640x480 14.56 -> 14.40).
template <int K>
__device__ __forceinline__ void normalise(float (&w)[K], float S, bool plain) {
    constexpr uint32_t kLow = 67u << 23, kHigh = 187u << 23;  // 2^-60, 2^60
    uint32_t low = 0xFFFFFFFFu;  // the least nonzero pattern, less one
#pragma unroll
    for (int k = 0; k < K; ++k) low = umin(low, __float_as_uint(w[k]) - 1u);
    const bool safe = low >= kLow - 1u && __float_as_uint(S) - kLow <= kHigh - kLow;
    if (plain && !any_lane(!safe)) {
        const float r0 = __builtin_amdgcn_rcpf(S);
        const float r = __builtin_fmaf(__builtin_fmaf(-S, r0, 1.0f), r0, r0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float q = w[k] * r;
            w[k] = __builtin_fmaf(__builtin_fmaf(-S, q, w[k]), r, q);
        }
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) w[k] = w[k] / S;
    }
}

// Sort the Gaussians by key, descending, with an insertion network of adjacent
// compare-exchanges; equal keys keep their order.  idx: their ranks before; AGAIN: the Gaussians
// may have been moved already, and equal keys go by idx.
template <bool AGAIN, int K, int C, int CV>
__device__ __forceinline__ void sort_ranks(Mix<K, C, CV>& m, float (&key)[K], int (&idx)[K]) {
#pragma unroll
    for (int i = 1; i < K; ++i) {
#pragma unroll
        for (int j = i; j > 0; --j) {
            const bool sw = key[j] > key[j - 1] || (AGAIN && key[j] == key[j - 1] && idx[j] < idx[j - 1]);
            auto swap = [sw](auto& a, auto& b) {
                const auto t = sw ? a : b;
                a = sw ? b : a;
                b = t;
            };
            swap(key[j], key[j - 1]);
            swap(idx[j], idx[j - 1]);
            swap(m.w[j], m.w[j - 1]);
            swap(m.v[j], m.v[j - 1]);
            if constexpr (CV == 3) {
                swap(m.vx[j][0], m.vx[j - 1][0]);
                swap(m.vx[j][1], m.vx[j - 1][1]);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) swap(m.mu[j][c], m.mu[j - 1][c]);
        }
    }
}

// Update of the mixture after its classification found the match ks: weights, the matched
// Gaussian or the replaced last one, renormalisation, ranking.  With `chg`, also report which
// ranks may hold a different (mean, variance) than before the step: bit r is set when the
// ranking moved another Gaussian to rank r or when the Gaussian at rank r was matched or
// replaced (clear bits are certain).  With REC, *rec records the choices.  `plain`: in no lane
// of the wavefront is a weight or a variance negative, infinite or NaN.
template <int K, int C, bool REC, int CV>
__device__ __forceinline__ void mixture_update(Mix<K, C, CV>& m, const float (&X)[C], int ks, float alpha, float w_init,
                                               float v_init, float v_min, int rho_mode, bool plain, uint32_t* chg,
                                               MixRec<C>* rec) {
    const bool matched = ks >= 0;
    const int tgt = matched ? ks : K - 1;
    // the Gaussian to change, selected once (its update then runs once for the wavefront,
    // whatever ranks its lanes matched)
    float mu[C], v = m.v[0], vx[CV == 3 ? 2 : 1];
#pragma unroll
    for (int c = 0; c < C; ++c) mu[c] = m.mu[0][c];
#pragma unroll
    for (int c = 0; c < (CV == 3 ? 2 : 0); ++c) vx[c] = m.vx[0][c];
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const bool here = k == tgt;
#pragma unroll
        for (int c = 0; c < C; ++c) mu[c] = here ? m.mu[k][c] : mu[c];
        v = here ? m.v[k] : v;
#pragma unroll
        for (int c = 0; c < (CV == 3 ? 2 : 0); ++c) vx[c] = here ? m.vx[k][c] : vx[c];
    }

    const float a = 1.0f - alpha;
    float wm = 0.0f;  // the matched weight after its update
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float wk = a * m.w[k];
        if (k == ks) {
            wk = wk + alpha;
            wm = wk;
        }
        m.w[k] = wk;
    }
    if (!matched) m.w[K - 1] = w_init;

    // rate of the matched mean and variance: alpha; alpha over the matched weight just
    // updated (>= alpha > 0); or alpha times the Eq. (1) density of the matched Gaussian at
    // the sample, before its update
    float rho = alpha;
    if (rho_mode != 0 && matched) {
        if (rho_mode == 1) {
            rho = alpha / wm;
        } else {
            float qm = 0.0f, vm = v;
            if constexpr (CV == 3) {
                float e = X[0] - mu[0];
                qm = (e * e) / v;
                e = X[1] - mu[1];
                qm = qm + (e * e) / vx[0];
                e = X[2] - mu[2];
                qm = qm + (e * e) / vx[1];
                vm = (v + vx[0]) + vx[1];
            } else {
                float e = X[0] - mu[0];
                float d2 = e * e;
#pragma unroll
                for (int c = 1; c < C; ++c) {
                    e = X[c] - mu[c];
                    d2 = d2 + e * e;
                }
                qm = d2 / v;
            }
            rho = alpha * (expf(-0.5f * qm) / (6.28318530717958647692f * vm));
        }
    }
    float mn[C];
#pragma unroll
    for (int c = 0; c < C; ++c) mn[c] = mu[c] + rho * (X[c] - mu[c]);
    bool cl = false;
    float vn, vxn[CV == 3 ? 2 : 1];
    if constexpr (CV == 3) {  // each channel's variance on its own deviation and floor
        float e = X[0] - mn[0];
        vn = fmaxf(v + rho * (e * e - v), v_min);
        e = X[1] - mn[1];
        vxn[0] = fmaxf(vx[0] + rho * (e * e - vx[0]), v_min);
        e = X[2] - mn[2];
        vxn[1] = fmaxf(vx[1] + rho * (e * e - vx[1]), v_min);
        vxn[0] = matched ? vxn[0] : v_init;
        vxn[1] = matched ? vxn[1] : v_init;
    } else {
        float e = X[0] - mn[0];
        float d2 = e * e;
#pragma unroll
        for (int c = 1; c < C; ++c) {
            e = X[c] - mn[c];
            d2 = d2 + e * e;
        }
        vn = v + rho * (d2 - v);
        cl = matched && vn < v_min;
        vn = fmaxf(vn, v_min);
    }
    vn = matched ? vn : v_init;
#pragma unroll
    for (int c = 0; c < C; ++c) mn[c] = matched ? mn[c] : X[c];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool here = k == tgt;
#pragma unroll
        for (int c = 0; c < C; ++c) m.mu[k][c] = here ? mn[c] : m.mu[k][c];
        m.v[k] = here ? vn : m.v[k];
#pragma unroll
        for (int c = 0; c < (CV == 3 ? 2 : 0); ++c) m.vx[k][c] = here ? vxn[c] : m.vx[k][c];
    }
    if (REC) {
        rec->clamp = cl;
#pragma unroll
        for (int c = 0; c < C; ++c) rec->mu[c] = mu[c];
        rec->v = v;
    }

    float S = m.w[0];
#pragma unroll
    for (int k = 1; k < K; ++k) S = S + m.w[k];
    normalise(m.w, S, plain);

    // Rank by w / sqrt(v), descending, stable.  In a static scene the order rarely changes, so
    // first look whether every adjacent pair is certain to be in order: the squared keys'
    // products clearly apart, or the lower one unused (w = 0, key 0).  A wavefront with a pair
    // that is not sorts by approximate keys if those decide, else by the rounded ones.
    uint32_t moved = 0u, pr = 0u;  // ranks that got another Gaussian; 3 bits per rank: which
#pragma unroll
    for (int k = 0; k < K; ++k) pr |= (uint32_t)k << (3 * k);
    uint32_t at = 1u << tgt;       // the ranks where the changed Gaussian is now
    bool inorder = plain, swapped = plain;  // swapped: certain to be out of order where not in order
#pragma unroll
    for (int k = 1; k < K; ++k) {
        // key above > key below as w^2 times the other's variance (weights are at most 1 here, so
        // that the first product holds all the precision the second can show); products below
        // kTiny, where rounding is no longer relative, are not apart
        const float above = (m.w[k - 1] * var_sum(m, k)) * m.w[k - 1];
        const float below = (m.w[k] * var_sum(m, k - 1)) * m.w[k];
        const bool apart = __builtin_fmaf(above, 1.0f - 2.0f * kMargin, -kTiny) > below || m.w[k] == 0.0f;
        inorder = inorder && apart;
        swapped = swapped && (apart || __builtin_fmaf(below, 1.0f - 2.0f * kMargin, -kTiny) > above);
    }
    if (K > 1 && any_lane(!inorder)) {
        float key[K];
        int idx[K];
#pragma unroll
        for (int k = 0; k < K; ++k) idx[k] = k;
        bool network = false, rounded = true;
        if (REC && !any_lane(!swapped)) {
            // Adjacent ranks are all clearly apart, some the other way round: sort by approximate
            // keys, and where the sorted ones are clearly apart too, that is the rounded keys' order.
#pragma unroll
            for (int k = 0; k < K; ++k) key[k] = m.w[k] * __builtin_amdgcn_rsqf(var_sum(m, k));
            sort_ranks<false>(m, key, idx);
            network = true;
            bool sure = true;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                sure = sure && (m.w[k] == 0.0f || key[k] > kTiny);
                if (k > 0) sure = sure && (m.w[k] == 0.0f || __builtin_fmaf(key[k - 1], 1.0f - kMargin, -kTiny) > key[k]);
            }
            rounded = any_lane(!sure);
        }
        if (rounded) {
#pragma unroll
            for (int k = 0; k < K; ++k) key[k] = m.w[k] / sqrtf(var_sum(m, k));
            bool unsorted = false;
#pragma unroll
            for (int k = 1; k < K; ++k)
                unsorted = unsorted || key[k] > key[k - 1] || (REC && key[k] == key[k - 1] && idx[k] < idx[k - 1]);
            if (any_lane(unsorted)) {
                sort_ranks<REC>(m, key, idx);
                network = true;
            }
        }
        if (network) {
            pr = 0u;
            at = 0u;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                pr |= (uint32_t)idx[k] << (3 * k);
                moved |= (idx[k] != k ? 1u : 0u) << k;
                at |= (idx[k] == tgt ? 1u : 0u) << k;
            }
        }
    }
    if (REC) rec->perm = pr;
    if (chg) *chg = moved | at;
}

// Classify on the pre-update mixture (used, delta) and, if `active`, update it in place,
// recording the step's discrete choices.  delta is correctly rounded.
template <int K, int C>
__device__ __forceinline__ void mixture_step_rec(Mix<K, C>& m, const float (&X)[C], bool active, float alpha, float lam2,
                                                 float T_bg, float w_init, float v_init, float v_min, bool sane,
                                                 bool& used, float& delta, MixRec<C>& rec) {
    // One Gaussian is one division either way, and the approximate choices only add to it (131x93, 24
    // frames, K = 1: forward 14.9 us, with them 19.5; 320x240, 64 frames: 44.3 and 53.5).
    MixClass r;
    bool plain = false;
    if constexpr (K > 1) {
        r = classify_approx<K, C, 1, true>(m, X, lam2, T_bg);
        plain = sane && !any_lane(!r.sure);
    }
    if (!plain) {
        r = classify_rounded(m, X, lam2, T_bg);
    } else {
        r.delta = r.d2 / r.v;  // one rounded division instead of K
    }
    used = r.used;
    delta = r.delta;
    rec.argmin = r.amin;
    rec.kstar = -1;
    rec.clamp = false;
    rec.perm = 0u;
#pragma unroll
    for (int k = 0; k < K; ++k) rec.perm |= (uint32_t)k << (3 * k);
#pragma unroll
    for (int c = 0; c < C; ++c) rec.mu[c] = 0.0f;
    rec.v = 0.0f;
    if (!active) return;
    rec.kstar = r.ks;
    mixture_update<K, C, true, 1>(m, X, r.ks, alpha, w_init, v_init, v_min, 0, plain, nullptr, &rec);
}

// State planes are touched once per frame.  When the device's resident model
// state exceeds the last-level (Infinity) cache the kernels stream it with
// non-temporal loads and stores; otherwise ordinary accesses let a cache-sized
// working set stay resident between frames.
// A plane is addressed through a raw buffer resource that starts at the workgroup's first
// pixel in that plane (scalar registers, rebuilt for the stores), so that one 32-bit lane
// offset serves every plane: ten 64-bit vector addresses held from the loads to the stores
// cost K = 5 twenty registers and an occupancy of 5 instead of 6.
typedef uint32_t st_u32x4 __attribute__((__vector_size__(4 * sizeof(uint32_t))));
constexpr int kStateWord3 = 0x00020000;  // raw 32-bit buffer, gfx9 family

// Plane k from pixel p0 on (p0 < npix, the same for the whole workgroup); an access past the
// plane's end is dropped (loads give 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t state_rsrc(const float4* state, int64_t npix, int64_t p0, int k) {
    const int64_t left = (npix - p0) * 16;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(state) + (int64_t)k * npix + p0, (short)0,
                                             (int)(left > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)left), kStateWord3);
}
template <bool NT>
__device__ __forceinline__ float4 ld_state(const float4* state, int64_t npix, int64_t p0, int k, uint32_t off) {
    const st_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(state_rsrc(state, npix, p0, k), off, 0, NT ? 2 : 0);
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}
template <bool NT>
__device__ __forceinline__ void st_state(float4* state, int64_t npix, int64_t p0, int k, uint32_t off, float4 v) {
    const st_u32x4 w = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
    __builtin_amdgcn_raw_buffer_store_b128(w, state_rsrc(state, npix, p0, k), off, 0, NT ? 2 : 0);
}

// Device layout of a GMM model (planes of npix float4, plane-major):
//   core plane k (k < Kc):  (mu_r, mu_g, mu_b, v) of colour rank k (with per-channel
//   colour variances, CV = 3: v is the red one);
//   extra planes (E of them): the floats w_c[0..Kc-1], w_d[0..Kd-1], then
//   (mu_d, v_d) of depth rank 0, 1, ..., then (CV = 3) the (v_g, v_b) of colour
//   rank 0, 1, ..., packed four to a plane, zero padded.
// Weights decay every frame, but a rank's mean and variance change only when its
// Gaussian is matched, replaced or moved by the ranking, so the planes that hold
// only means and variances can often be left unwritten.
template <int KC, int KD, int CV = 1>
struct GmmLayout {
    static constexpr int NX = KC + 3 * KD + (CV == 3 ? 2 * KC : 0);  // extra floats
    static constexpr int E = (NX + 3) / 4;                            // extra planes
    static constexpr int w_c(int k) { return gmm_x_wc(KC, KD, k); }
    static constexpr int w_d(int k) { return gmm_x_wd(KC, KD, k); }
    static constexpr int mu_d(int k) { return gmm_x_mud(KC, KD, k); }
    static constexpr int v_d(int k) { return gmm_x_vd(KC, KD, k); }
    static constexpr int v_g(int k) { return gmm_x_vg(KC, KD, k); }
    static constexpr int v_b(int k) { return gmm_x_vb(KC, KD, k); }
};

// Scaled Eq. (1) factor of the Gaussian attaining delta (decision 1), in the order
// the oracle rounds it: s * (exp(-delta/2) / (2 pi v)).
__device__ __forceinline__ float density_factor(float delta, float v, float s) {
    return s * (expf(-0.5f * delta) / (6.28318530717958647692f * v));
}

// One pixel of one frame: ingest, both mixtures' classify-and-update, the
// combined decision, the mask, and the state write-back.  RW selects the rate of
// the matched mean and variance: 0 alpha, 1 as a.c.rho_mode says;
// DEC the decision: 0 the Z rule, 1 the density product, 2 as a.c.decision says
// (a compile-time choice keeps the other path's registers out of the kernel).
// A plane is stored only where one of the 4 pixels sharing the lane's 64-byte
// sector of it (lanes 4i..4i+3: 16 bytes per pixel) may have changed it, so every
// store still covers whole sectors.
// Bit i of the result: bit i of `bits` set in any of lanes 4i..4i+3 (one plane per bit).
__device__ __forceinline__ uint32_t sector_or(uint32_t bits) {
    bits |= __shfl_xor(bits, 1, 64);
    bits |= __shfl_xor(bits, 2, 64);
    return bits;
}

// The pixel is p0 + lane; p0 is the same for the whole workgroup.
template <int KC, int KD, bool NT, int RW = 2, int DEC = 2, int CV = 1>
__device__ __forceinline__ void gmm_pixel(const GmmStepArgs& a, int p0, int lane) {
    using L = GmmLayout<KC, KD, CV>;
    constexpr int E = L::E;
    const int64_t npix = a.npix;
    const uint32_t off = (uint32_t)lane * 16u;

    // Every read is issued before any result is used (the frame first, then the
    // state planes): loads complete in order, and the depth code's branch would
    // otherwise wait for the frame before the state reads go out.
    const uint8_t* px;
    uint32_t dmm;
    if (a.geom.flat) {
        px = a.rgb + 3 * (int64_t)p0 + 3 * lane;
        dmm = *reinterpret_cast<const uint16_t*>(a.depth + 2 * (int64_t)p0 + 2 * lane);
    } else {
        const int p = p0 + lane;
        const int y = (int)div_by((uint32_t)p, a.geom.w);
        const int x = p - y * a.W;
        px = a.rgb + (int64_t)y * a.rgb_stride + 3 * x;
        dmm = load_depth(a.depth, a.depth_stride, x, y, a.W, a.H, a.depth_w, a.depth_h, a.geom);
    }
    const uint32_t r0 = px[0], r1 = px[1], r2 = px[2];
    float4 core[KC];
    float4 exv[E];
#pragma unroll
    for (int k = 0; k < KC; ++k) core[k] = ld_state<NT>(a.state, npix, p0, k, off);
#pragma unroll
    for (int e = 0; e < E; ++e) exv[e] = ld_state<NT>(a.state, npix, p0, KC + e, off);
    __builtin_amdgcn_sched_barrier(0);

    const float Xc[3] = {(float)r0, (float)r1, (float)r2};
    const bool valid = dmm > 0u;
    const float Xd[1] = {(float)depth_code(dmm, a.c.depth_max_mm, a.c.depth_div)};
    float ex[4 * E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        ex[4 * e + 0] = exv[e].x;
        ex[4 * e + 1] = exv[e].y;
        ex[4 * e + 2] = exv[e].z;
        ex[4 * e + 3] = exv[e].w;
    }
    Mix<KC, 3, CV> mc;
    Mix<KD, 1> md;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        mc.w[k] = ex[L::w_c(k)];
        mc.mu[k][0] = core[k].x;
        mc.mu[k][1] = core[k].y;
        mc.mu[k][2] = core[k].z;
        mc.v[k] = core[k].w;
        if constexpr (CV == 3) {
            mc.vx[k][0] = ex[L::v_g(k)];
            mc.vx[k][1] = ex[L::v_b(k)];
        }
    }
#pragma unroll
    for (int k = 0; k < KD; ++k) {
        md.w[k] = ex[L::w_d(k)];
        md.mu[k][0] = ex[L::mu_d(k)];
        md.v[k] = ex[L::v_d(k)];
    }

    const float lam2 = a.c.lam * a.c.lam;
    const int rw = RW == 0 ? 0 : a.c.rho_mode;
    const bool dec = DEC == 2 ? a.c.decision != 0 : DEC == 1;
    float4* so = a.state;
    asm volatile("" : "+s"(so));  // the stores' descriptors are built again, not kept since the loads
    // Both mixtures are classified first, on the pre-update state, and the mask is decided;
    // the density decision wants rounded values.
    MixClass cc = classify_approx<KC, 3, CV, false>(mc, Xc, lam2, a.c.T_bg);
    MixClass cd = classify_approx<KD, 1, 1, false>(md, Xd, lam2, a.c.T_bg);
    const bool term_c = cc.used;
    const bool term_d = valid && cd.used;
    bool fg, sure = cc.sure && (cd.sure || !valid) && a.c.sane != 0 && !(DEC != 0 && dec);
    {
        const float wd = a.c.w_depth;
        const float Z = (term_c ? cc.delta - lam2 : 0.0f) + (term_d ? wd * (cd.delta - lam2) : 0.0f);
        const float size = (term_c ? cc.delta + lam2 : 0.0f) + (term_d ? wd * (cd.delta + lam2) : 0.0f);
        fg = Z >= 0.0f;
        sure = sure && (fabsf(Z) > kMargin * size || !(term_c || term_d));
    }
    const bool plain = !any_lane(!sure);
    if (!plain) {
        cc = classify_rounded(mc, Xc, lam2, a.c.T_bg);
        cd = classify_rounded(md, Xd, lam2, a.c.T_bg);
        if (DEC != 0 && dec) {
            float vs_c = var_sum(mc, 0), vs_d = md.v[0];
#pragma unroll
            for (int k = 1; k < KC; ++k)
                if (k == cc.amin) vs_c = var_sum(mc, k);
#pragma unroll
            for (int k = 1; k < KD; ++k)
                if (k == cd.amin) vs_d = md.v[k];
            const float Pc = density_factor(cc.delta, vs_c, a.c.density_scale);
            const float Pd = density_factor(cd.delta, vs_d, a.c.density_scale);
            const float P = term_c ? (term_d ? Pc * Pd : Pc) : Pd;
            fg = P < a.c.density_threshold;
        } else {
            const float tc = cc.delta - lam2;
            const float td = a.c.w_depth * (cd.delta - lam2);
            const float Z = term_c ? (term_d ? tc + td : tc) : td;
            fg = Z >= 0.0f;
        }
    }
    a.mask[(int64_t)p0 + lane] = ((term_c || term_d) && fg) ? (uint8_t)255 : (uint8_t)0;

    uint32_t chg_c = 0u, chg_d = 0u;
    mixture_update<KC, 3, false, CV>(mc, Xc, cc.ks, a.c.alpha, a.c.w_init, a.c.v_init_c, a.c.v_min_c, rw, plain,
                                     &chg_c, nullptr);
    // the colour means and variances are final: store them before the depth step
    const uint32_t wc = sector_or(chg_c);
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if ((wc >> k) & 1u)
            st_state<NT>(so, npix, p0, k, off, make_float4(mc.mu[k][0], mc.mu[k][1], mc.mu[k][2], mc.v[k]));
    if (valid)
        mixture_update<KD, 1, false, 1>(md, Xd, cd.ks, a.c.alpha, a.c.w_init, a.c.v_init_d, a.c.v_min_d, rw, plain,
                                        &chg_d, nullptr);

    // Which extra floats may change: the colour weights always (the colour mixture
    // is updated every frame), the depth weights where depth > 0 (the depth mixture
    // is updated only there), a depth mean and variance as the depth mixture reports.
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        ex[L::w_c(k)] = mc.w[k];
        if constexpr (CV == 3) {
            ex[L::v_g(k)] = mc.vx[k][0];
            ex[L::v_b(k)] = mc.vx[k][1];
        }
    }
#pragma unroll
    for (int k = 0; k < KD; ++k) {
        ex[L::w_d(k)] = md.w[k];
        ex[L::mu_d(k)] = md.mu[k][0];
        ex[L::v_d(k)] = md.v[k];
    }
    uint32_t che = 0u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        bool ch = false;
#pragma unroll
        for (int i = 4 * e; i < 4 * e + 4; ++i) {
            if (i < KC) ch = true;
            else if (i < KC + KD) ch = ch || valid;
            else if (i < KC + 3 * KD) ch = ch || ((chg_d >> ((i - KC - KD) >> 1)) & 1u);
            else if (i < L::NX) ch = ch || ((chg_c >> ((i - KC - 3 * KD) >> 1)) & 1u);
        }
        che |= (ch ? 1u : 0u) << e;
    }
    const uint32_t we = sector_or(che);
#pragma unroll
    for (int e = 0; e < E; ++e)
        if ((we >> e) & 1u)
            st_state<NT>(so, npix, p0, KC + e, off,
                         make_float4(ex[4 * e + 0], ex[4 * e + 1], ex[4 * e + 2], ex[4 * e + 3]));
}

}  // namespace fgs
