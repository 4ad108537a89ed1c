// RGB-D PBAS with the base method's gradient-magnitude feature on the colour channels
// (opt-in; Sec. 3.2's RGB-D variant leaves it out).  Per colour channel j a sample slot
// holds the value v and the gradient magnitude m = (|gx| + |gy|) >> 3 of that channel's
// plane (3x3 Sobel, border replicated), and
//   dist = w_j * |m - B^m| + |v - B^v|   (float32, in that order, no contraction)
//   w_j  = alpha / max(mean of m_j over the previous frame, 1)
// with d_min, D and S in float32; the depth channel keeps the integer value distance.
// Everything else (fill frames, classification by match count, self-update, deferred
// neighbour update through fire bytes and the LDS scatter of pbas_device.h, R and T) is
// the plain variant's, so the random draws and decisions follow the same rules.
//
// Layout (fgs_internal.h, PbasGradPlanes): samples and magnitudes in the plain variant's quad
// planes, so that a wavefront moves 1 KiB contiguous per access and a changed sector is written
// back whole; D as one float4 per slot and pixel.
//
// Measured at 640x480, N = 20, static background (T = 2): the first version read slot by slot, each
// read behind the previous slot's possible write, and wrote single words and bytes: 60 us a frame
// (one model after another frame of its own, 81 in turn with two others); on quad planes held in
// registers 41 (2 models of 1280x720 392 -> 242, N = 35 93 -> 53); with five workgroups a CU 38.6.
// At 114 registers a CU held four: 1,200 tiles were 1.17 rounds.  T, R and S wait in LDS during the
// slot loop, the candidates' slots share a word, the weights are scalars and the second smallest
// distance replaces a count and R: 96 registers (forced to that before, spills cost more than the
// second round, 44.8 us).  N = 16: 39.0 -> 35.7, N = 24: 44.3 -> 42.1, N = 40: 56.9 -> 54.5.  With
// the magnitude sums in 16 lines instead of one, which 3,600 adds a frame waited for: N = 20 38.6 ->
// 38.1, N = 16 35.7 -> 34.5, N = 8 30.4 -> 25.5.
#include <cstring>

#include "device_common.h"
#include "fgs_internal.h"
#include "pbas_device.h"

namespace fgs {

using namespace pbas;

namespace {

// Register capacity classes (a sample and a magnitude word per slot): class NMAX serves N from
// grad_class_min(NMAX) to NMAX.  Fewer than the plain variant's: twelve registers a step.
constexpr int grad_class_min(int nmax) {
    return nmax <= 8 ? 2 : nmax <= 16 ? 9 : nmax <= 20 ? 17 : nmax <= 24 ? 21 : nmax <= 32 ? 25 : nmax <= 40 ? 33 : 41;
}

// Workgroups a CU is to hold (its four SIMDs a wavefront of each).
constexpr int grad_waves(int nmax) { return nmax <= 20 ? 5 : nmax <= 32 ? 4 : nmax <= 40 ? 3 : 2; }

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

struct __attribute__((packed, aligned(1))) Bytes12 {
    uint32_t w[3];
};

// Byte i (0..8) of three packed pixels.
__device__ __forceinline__ int byte_of(const uint32_t (&w)[3], int i) { return (int)((w[i >> 2] >> (8 * (i & 3))) & 0xFFu); }

// The three colour magnitudes of pixel (x, y) as bytes m_R | m_G << 8 | m_B << 16.  Inside the
// image a row's three pixels are one 12-byte read (9 of them used: it ends inside the row for
// x <= W - 3); at the sides they are read one by one at clamped columns.
__device__ __forceinline__ uint32_t colour_magnitudes(const uint8_t* rgb, int64_t stride, int x, int y, int W,
                                                      int H) {
    uint32_t w[3][3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        const uint8_t* row = rgb + (int64_t)clampi(y + dy - 1, 0, H - 1) * stride;
        if (x >= 1 && x <= W - 3) {
            const Bytes12 b = *reinterpret_cast<const Bytes12*>(row + 3 * (x - 1));
#pragma unroll
            for (int i = 0; i < 3; ++i) w[dy][i] = b.w[i];
        } else {
            uint32_t px[3];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const uint8_t* q = row + 3 * clampi(x + dx - 1, 0, W - 1);
                px[dx] = (uint32_t)q[0] | ((uint32_t)q[1] << 8) | ((uint32_t)q[2] << 16);
            }
            w[dy][0] = px[0] | (px[1] << 24);
            w[dy][1] = (px[1] >> 8) | (px[2] << 16);
            w[dy][2] = px[2] >> 16;
        }
    }
    uint32_t out = 0u;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        int v[3][3];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) v[dy][dx] = byte_of(w[dy], 3 * dx + j);
        const int gx = (v[0][2] + 2 * v[1][2] + v[2][2]) - (v[0][0] + 2 * v[1][0] + v[2][0]);
        const int gy = (v[2][0] + 2 * v[2][1] + v[2][2]) - (v[0][0] + 2 * v[0][1] + v[0][2]);
        out |= (uint32_t)((abs(gx) + abs(gy)) >> 3) << (8 * j);
    }
    return out;
}

// The word of part `part` of channel j's sum in slot f (frame number mod 3).
__device__ __forceinline__ int sum_index(uint32_t f, int part, int j) {
    return ((int)f * kGradSlots + part) * kGradSlotWords + j;
}

// Adds the block's colour magnitudes to frame t's sums (one 64-bit atomic per channel
// and block; integer sums, so the order does not matter), and block 0 clears frame
// t+1's parts, which nothing reads or writes during frame t.
__device__ __forceinline__ void add_magnitudes(unsigned long long* gsum, uint32_t t, uint32_t mw, bool inside) {
    __shared__ uint32_t part[kBlock / 64][3];
    // two channels per word: a wavefront's sum is at most 64 * 255 < 2^16
    uint32_t rb = inside ? mw & 0x00FF00FFu : 0u, g = inside ? (mw >> 8) & 0xFFu : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        rb += __shfl_xor(rb, off, 64);
        g += __shfl_xor(g, off, 64);
    }
    const uint32_t c[3] = {rb & 0xFFFFu, g, rb >> 16};
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int j = 0; j < 3; ++j) part[threadIdx.x >> 6][j] = c[j];
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long v = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) v += part[w][threadIdx.x];
        if (v) atomicAdd(gsum + sum_index(t % 3u, (int)(blockIdx.x % kGradSlots), (int)threadIdx.x), v);
    }
    if (blockIdx.x == 0 && threadIdx.x < 3 * kGradSlots)
        gsum[sum_index((uint32_t)(((uint64_t)t + 1u) % 3u), (int)threadIdx.x / 3, (int)threadIdx.x % 3)] = 0ull;
}

// A lane's part of slot f's sums: part s of channel j for lane 16 j + s of the first wavefront.
__device__ __forceinline__ unsigned long long sum_part(const unsigned long long* gsum, uint32_t f) {
    static_assert(kGradSlots == 16, "lanes 16 j + s");
    const int lane = (int)threadIdx.x;
    return lane < 48 ? gsum[sum_index(f, lane & 15, lane >> 4)] : 0ull;
}

__device__ __forceinline__ uint32_t frame_word(const PbasGradArgs& a, int x, int y, bool& valid) {
    const uint8_t* px = a.rgb + (int64_t)y * a.rgb_stride + 3 * x;
    const uint32_t dmm = load_depth(a.depth, a.depth_stride, x, y, a.W, a.H, a.depth_w, a.depth_h, a.geom);
    valid = dmm > 0u;
    return (uint32_t)px[0] | ((uint32_t)px[1] << 8) | ((uint32_t)px[2] << 16) |
           (depth_code(dmm, a.c.depth_max_mm, a.c.depth_div) << 24);
}

// Frames 0..N-1: slot t takes the frame's value and magnitudes; the mask is empty.
__global__ __launch_bounds__(kBlock) void pbas_grad_fill_kernel(PbasGradArgs a) {
    const int p = blockIdx.x * kBlock + threadIdx.x;
    const bool inside = p < a.npix;
    const int q = inside ? p : 0;
    const int y = (int)div_by((uint32_t)q, a.geom.w), x = q - y * a.W;
    bool valid;
    const uint32_t v = frame_word(a, x, y, valid);
    const uint32_t mw = colour_magnitudes(a.rgb, a.rgb_stride, x, y, a.W, a.H);
    add_magnitudes(a.m.gsum, a.t, mw, inside);
    if (!inside) return;
    *reinterpret_cast<uint32_t*>(sample_byte(a.m.samples, a.npix, (int)a.t, p, 0)) = v;
    *reinterpret_cast<uint32_t*>(sample_byte(a.m.gsamples, a.npix, (int)a.t, p, 0)) = mw;
    a.m.last[p] = v;
    a.m.last_g[p] = mw;
    a.m.mask[p] = 0;
}

// One updating frame on a 64x4 tile: the plain variant's tiling, fire-byte halo, LDS scatter of
// pending neighbour writes, register merges and whole-sector write-back (pbas_device.h), on two
// words per slot.
// TWO: min_matches = 2, decided by the second smallest distance (as in pbas_device.h; one v_med3_f32
// where a count takes a comparison and an addition), so that the slot loop needs no R.
template <int NMAX, bool NT, bool TWO>
__global__ __launch_bounds__(kBlock, grad_waves(NMAX)) void pbas_grad_step_kernel(PbasGradArgs a) {
    constexpr int NLO = grad_class_min(NMAX);
    constexpr int NW = PbasLds<NMAX>::NW;
    __shared__ PbasLds<NMAX> sh;
    __shared__ float weight[3];
    __shared__ float4 park[3][kBlock];  // a lane's T, R and S during the slot loop
    const int tid = threadIdx.x;
    const int tiles_x = (a.W + kTileW - 1) / kTileW;
    const int bx = (int)blockIdx.x % tiles_x, by = (int)blockIdx.x / tiles_x;
    const int x0 = bx * kTileW, y0 = by * kTileH;
    const int lx = tid % kTileW, ly = tid / kTileW;
    const bool inside = x0 + lx < a.W && y0 + ly < a.H;
    const int x = inside ? x0 + lx : x0, y = inside ? y0 + ly : y0;
    const int p = y * a.W + x;
    const int64_t npix = a.npix;
    const int N = a.c.N;

    FireIn fin = {{0u, 0u}, {0, 0}};
    if (a.apply_pending) {
#pragma unroll
        for (int w = 0; w < NW; ++w) sh.pend[w * kBlock + tid] = 0u;
        fin = load_fire(a.m.fire[(a.t - 1u) & 1u], x0, y0, a.H, a.W);
    }
    const unsigned long long sums = tid < 64 ? sum_part(a.m.gsum, (uint32_t)(((uint64_t)a.t + 2u) % 3u)) : 0ull;
    const float4 Tv = a.m.T[p];
    bool valid;
    const uint32_t Iw = frame_word(a, x, y, valid);
    const uint32_t Mw = colour_magnitudes(a.rgb, a.rgb_stride, x, y, a.W, a.H);
    const float4 Rv = a.m.R[p], Sv = a.m.S[p];
    const uint32_t lastw = a.m.last[p], lastg = a.m.last_g[p];

    uint32_t sm[NMAX], gm[NMAX];
    const int64_t p0 = (int64_t)y0 * a.W + x0;  // tile origin, < npix
    const int64_t qleft = (npix - p0) * 16;
    const uint32_t qrange = qleft > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)qleft;
    const uint32_t voff = (uint32_t)(p - p0) * 16u;
#pragma unroll
    for (int q = 0; q < NMAX / 4; ++q) {
        const bool used = 4 * q < NLO || 4 * q < N;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        const u32x4 v = used ? ld_quad<NT>(a.m.samples + p0 * 4, npix, qrange, q, voff) : zero;
        const u32x4 g = used ? ld_quad<NT>(a.m.gsamples + p0 * 4, npix, qrange, q, voff) : zero;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sm[4 * q + i] = v[i];
            gm[4 * q + i] = g[i];
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // weights from the previous frame's magnitude sums, by the first wavefront for all
    if (tid < 64) {
        unsigned long long sum = sums;
#pragma unroll
        for (int off = 1; off < kGradSlots; off <<= 1) sum += __shfl_xor(sum, off, 64);
        const float mean = (float)(double)sum / (float)a.npix;
        if (tid < 48 && (tid & 15) == 0) weight[tid >> 4] = a.c.grad_alpha / fmaxf(mean, 1.0f);
    }
    if (a.apply_pending) {
        __syncthreads();  // bit-words cleared
        scatter_fired<NMAX>(sh, fin, N, a.t - 1u, a.c.key0, a.c.key1);
    }
    // Self-update candidates (the 1/T test with T from before this frame) and the D they replace.
    const float T0[4] = {Tv.x, Tv.y, Tv.z, Tv.w};
    const bool active[4] = {true, true, true, valid};
    const float inv16 = 1.0f / 65536.0f;
    const U32x4 w0 = philox4x32_10((uint32_t)p, a.t, 0u, 0u, a.c.key0, a.c.key1);
    bool cand[4];
    uint32_t slots = 0u;  // the candidates' slots, a byte each
    float dold[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t a0 = w0.v[j];
        cand[j] = active[j] && (float)(a0 >> 16) * inv16 * T0[j] < 1.0f;
        const int k = (int)(__umul24(a0 & 0xFFFFu, (uint32_t)N) >> 16);
        slots |= (uint32_t)k << (8 * j);
        dold[j] = cand[j] ? reinterpret_cast<const float*>(a.m.D + (int64_t)k * npix + p)[j] : 0.0f;
    }
    park[0][tid] = Tv;
    park[1][tid] = Rv;
    park[2][tid] = Sv;
    if (a.apply_pending) __syncthreads();  // every write aimed at the tile recorded
    add_magnitudes(a.m.gsum, a.t, Mw, inside);  // frame t's sums; its barrier is the weights' too
    if (!inside) return;
    float wgt[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)  // (one value per frame: scalar registers)
        wgt[j] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(weight[j])));

    const float R0[4] = {Rv.x, Rv.y, Rv.z, Rv.w};

    // Frame t-1's neighbour writes into this pixel (its previous value and magnitudes) are
    // merged slot by slot, then each slot is classified: bytes become floats in one
    // instruction, differences and their absolute values are exact.
    uint32_t pw[NW];
    const uint32_t keep = (lastw >> 24) != 0u ? 0xFFFFFFFFu : 0x00FFFFFFu;  // depth at t-1?
#pragma unroll
    for (int w = 0; w < NW; ++w) pw[w] = a.apply_pending ? sh.pend[w * kBlock + tid] & keep : 0u;
    const float fi[4] = {(float)(Iw & 0xFFu), (float)((Iw >> 8) & 0xFFu), (float)((Iw >> 16) & 0xFFu), (float)(Iw >> 24)};
    const float fm[3] = {(float)(Mw & 0xFFu), (float)((Mw >> 8) & 0xFFu), (float)((Mw >> 16) & 0xFFu)};
    int cnt[4] = {0, 0, 0, 0};
    float dmin[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, dsec[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
    uint32_t dirty_s = 0u, dirty_g = 0u, chg_s = 0u, chg_g = 0u;
    uint32_t byte_ids;
    asm("v_mov_b32 %0, 0x03020100" : "=v"(byte_ids));
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
        if ((k & 3) == 0) __builtin_amdgcn_sched_barrier(0);  // a slot's work stays next to its words
        const uint32_t s0 = sm[k], g0 = gm[k];
        sm[k] = merge_slot(s0, lastw, pw[k >> 3], k, byte_ids);
        gm[k] = merge_slot(g0, lastg, pw[k >> 3], k, byte_ids);  // (byte 3 is 0 on both sides)
        chg_s |= sm[k] ^ s0;
        chg_g |= gm[k] ^ g0;
        if ((k & 3) == 3) {
            dirty_s |= (chg_s != 0u ? 1u : 0u) << (k >> 2);
            dirty_g |= (chg_g != 0u ? 1u : 0u) << (k >> 2);
            chg_s = chg_g = 0u;
            asm volatile("" : "+v"(dirty_s), "+v"(dirty_g));  // (each quad's test next to its slots)
        }
        if (k < NLO || k < N) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float dv = (float)((sm[k] >> (8 * j)) & 0xFFu) - fi[j];
                const float dm = (float)((gm[k] >> (8 * j)) & 0xFFu) - fm[j];
                const float d = wgt[j] * fabsf(dm) + fabsf(dv);
                if (TWO) dsec[j] = __builtin_amdgcn_fmed3f(dmin[j], dsec[j], d);
                else cnt[j] += d < R0[j] ? 1 : 0;
                dmin[j] = fminf(dmin[j], d);
            }
            const float sd = (float)(sm[k] >> 24);
            const float d = sd != 0.0f ? fabsf(sd - fi[3]) : INFINITY;  // a depth byte 0: nothing recorded
            if (TWO) dsec[3] = __builtin_amdgcn_fmed3f(dmin[3], dsec[3], d);
            else cnt[3] += d < R0[3] ? 1 : 0;
            dmin[3] = fminf(dmin[3], d);
            // (a slot is finished before the next: left to itself the scheduler keeps the
            // distances of many slots and needs 40 more registers)
            asm volatile("" : "+v"(dmin[0]), "+v"(dmin[1]), "+v"(dmin[2]), "+v"(dmin[3]));
            if (TWO) asm volatile("" : "+v"(dsec[0]), "+v"(dsec[1]), "+v"(dsec[2]), "+v"(dsec[3]));
            else asm volatile("" : "+v"(cnt[0]), "+v"(cnt[1]), "+v"(cnt[2]), "+v"(cnt[3]));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (dmin[3] == INFINITY) dmin[3] = 255.0f;
    int back = tid;  // (opaque: the parked values are read again, not kept)
    asm volatile("" : "+v"(back));
    const float4 Tp = park[0][back], Rp = park[1][back], Sp = park[2][back];
    float T[4] = {Tp.x, Tp.y, Tp.z, Tp.w};
    float R[4] = {Rp.x, Rp.y, Rp.z, Rp.w};
    float S[4] = {Sp.x, Sp.y, Sp.z, Sp.w};
    int ks[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) ks[j] = (int)((slots >> (8 * j)) & 0xFFu);

    bool F[4], upd[4];
    bool fg = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        F[j] = active[j] && !(TWO ? dsec[j] < R[j] : cnt[j] >= a.c.min_matches);
        fg = fg || F[j];
        upd[j] = cand[j] && !F[j];
    }
    a.m.mask[p] = fg ? (uint8_t)255 : (uint8_t)0;

    // Self-update: slot ks[j] of channel j takes the value (and magnitude), its D slot d_min,
    // S = (S - D_k) + d_min.
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (upd[j]) {
            S[j] = (S[j] - dold[j]) + dmin[j];
            if (__float_as_uint(dold[j]) != __float_as_uint(dmin[j]))
                reinterpret_cast<float*>(a.m.D + (int64_t)ks[j] * npix + p)[j] = dmin[j];
        }

    // Neighbour update with probability 1/T: record the channels that fired.
    const U32x4 w1 = philox4x32_10((uint32_t)p, a.t, 1u, 0u, a.c.key0, a.c.key1);
    uint32_t fire = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!active[j] || F[j]) continue;
        const uint32_t a1 = w1.v[j];
        if ((float)(a1 >> 16) * inv16 * T[j] < 1.0f) {
            const int d = (int)((a1 >> 13) & 7u);
            const int nx = x + nb_dx(d), ny = y + nb_dy(d);
            if (nx >= 0 && nx < a.W && ny >= 0 && ny < a.H) fire |= 1u << j;
        }
    }

    // Decision threshold and update rate (d_bar from the float sum).
    const float rdn = 1.0f - a.c.R_incdec, rup = 1.0f + a.c.R_incdec;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!active[j]) continue;
        const float dbar = S[j] / (float)N;
        const float r = (R[j] > dbar * a.c.R_scale) ? R[j] * rdn : R[j] * rup;
        R[j] = fmaxf(r, a.c.R_lower[j]);
        const float q = (F[j] ? a.c.T_inc : a.c.T_dec) / dbar;
        const float tt = F[j] ? T[j] + q : T[j] - q;
        T[j] = fminf(fmaxf(tt, a.c.T_lower), a.c.T_upper);
    }

    // The self-update's bit-words, built in the lane's own LDS words (read above, touched by no
    // other lane since the scatter's barrier), then merged quad by quad at the store; a quad goes
    // back only where a byte of it changed in one of the 4 pixels of its 64-byte sector.
    uint32_t sw[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) sh.pend[w * kBlock + tid] = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (upd[j])
            __hip_atomic_fetch_or(&sh.pend[(ks[j] >> 3) * kBlock + tid], 1u << (8 * j + (ks[j] & 7)),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int w = 0; w < NW; ++w) sw[w] = sh.pend[w * kBlock + tid];
    uint32_t* sbase = a.m.samples + p0 * 4;
    uint32_t* gbase = a.m.gsamples + p0 * 4;
    asm volatile("" : "+s"(sbase), "+s"(gbase));
#pragma unroll
    for (int q = 0; q < NMAX / 4; ++q) {
        if (!(4 * q < NLO || 4 * q < N)) continue;
        uint32_t cs = 0u, cg = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * q + i;
            const uint32_t s0 = sm[k], g0 = gm[k];
            sm[k] = merge_slot(s0, Iw, sw[k >> 3], k, byte_ids);
            gm[k] = merge_slot(g0, Mw, sw[k >> 3], k, byte_ids);
            cs |= sm[k] ^ s0;
            cg |= gm[k] ^ g0;
        }
        int d = (int)(((dirty_s >> q) & 1u) | (cs != 0u ? 1u : 0u)) | (int)((((dirty_g >> q) & 1u) | (cg != 0u ? 1u : 0u)) << 1);
        d |= __builtin_amdgcn_update_dpp(0, d, 0xB1, 0xF, 0xF, false);
        d |= __builtin_amdgcn_update_dpp(0, d, 0x4E, 0xF, 0xF, false);
        if (d & 1) {
            const u32x4 v = {sm[4 * q], sm[4 * q + 1], sm[4 * q + 2], sm[4 * q + 3]};
            st_quad<NT>(sbase, npix, qrange, q, voff, v);
        }
        if (d & 2) {
            const u32x4 g = {gm[4 * q], gm[4 * q + 1], gm[4 * q + 2], gm[4 * q + 3]};
            st_quad<NT>(gbase, npix, qrange, q, voff, g);
        }
    }
    const float4 Rn = make_float4(R[0], R[1], R[2], R[3]);
    const float4 Tn = make_float4(T[0], T[1], T[2], T[3]);
    const float4 Sn = make_float4(S[0], S[1], S[2], S[3]);
    if (differs(Rn, park[1][back])) a.m.R[p] = Rn;
    if (differs(Tn, park[0][back])) a.m.T[p] = Tn;
    if (differs(Sn, park[2][back])) a.m.S[p] = Sn;
    a.m.last[p] = Iw;
    a.m.last_g[p] = Mw;
    a.m.fire[a.t & 1u][p] = (uint8_t)fire;
}

// The neighbour writes of the last processed frame applied for a state read-out (as
// the plain variant's flush, writing the value and the colour magnitudes).
__global__ __launch_bounds__(256) void pbas_grad_flush_kernel(PbasGradPlanes m, int H, int W, uint32_t t_prev,
                                                              int N, uint32_t k0, uint32_t k1) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= H * W) return;
    const int y = p / W, x = p - y * W;
    const int64_t npix = (int64_t)H * W;
    const uint32_t lastw = m.last[p], lastg = m.last_g[p];
    const uint8_t* fire = m.fire[t_prev & 1u];
    for (int d = 0; d < 8; ++d) {
        const int qx = x + nb_dx(d), qy = y + nb_dy(d);
        if (qx < 0 || qx >= W || qy < 0 || qy >= H) continue;
        const int q = qy * W + qx;
        const uint32_t fb = fire[q] & 0xFu;  // channels that fired (the high nibble: R flags)
        if (fb == 0u) continue;
        const U32x4 w1 = philox4x32_10((uint32_t)q, t_prev, 1u, 0u, k0, k1);
        for (int j = 0; j < 4; ++j) {
            if (!((fb >> j) & 1u)) continue;
            int dq, slot;
            intent_of(w1.v[j], N, dq, slot);
            const uint32_t val = (lastw >> (8 * j)) & 0xFFu;
            if (dq != 7 - d || (j == 3 && val == 0u)) continue;
            *sample_byte(m.samples, npix, slot, p, j) = (uint8_t)val;
            if (j < 3) *sample_byte(m.gsamples, npix, slot, p, j) = (uint8_t)(lastg >> (8 * j));
        }
    }
}

__global__ void pbas_grad_init_kernel(PbasGradPlanes m, int npix, float4 Rl, float Tl) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    m.R[p] = Rl;
    m.T[p] = make_float4(Tl, Tl, Tl, Tl);
}

// Canonical planes: D [N][4] float32, R, T, S [4] float32 <-> float4 per pixel.
__global__ void pbas_grad_export_kernel(PbasGradPlanes m, int npix, int N, float* dout, float* rts, uint32_t* out,
                                        int has_header, StateWords header) {
    write_header(out, has_header, header);
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    for (int k = 0; k < N; ++k) {
        const float4 d = m.D[(int64_t)k * n + p];
        dout[(4 * k + 0) * n + p] = d.x;
        dout[(4 * k + 1) * n + p] = d.y;
        dout[(4 * k + 2) * n + p] = d.z;
        dout[(4 * k + 3) * n + p] = d.w;
    }
    const float4 r = m.R[p], t = m.T[p], s = m.S[p];
    const float v[12] = {r.x, r.y, r.z, r.w, t.x, t.y, t.z, t.w, s.x, s.y, s.z, s.w};
    for (int i = 0; i < 12; ++i) rts[i * n + p] = v[i];
}

__global__ void pbas_grad_import_kernel(PbasGradPlanes m, int npix, int N, const float* din, const float* rts,
                                        StateCheck check) {
    if (!header_matches(check)) return;
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    for (int k = 0; k < N; ++k)
        m.D[(int64_t)k * n + p] = make_float4(din[(4 * k + 0) * n + p], din[(4 * k + 1) * n + p],
                                              din[(4 * k + 2) * n + p], din[(4 * k + 3) * n + p]);
    m.R[p] = make_float4(rts[0 * n + p], rts[1 * n + p], rts[2 * n + p], rts[3 * n + p]);
    m.T[p] = make_float4(rts[4 * n + p], rts[5 * n + p], rts[6 * n + p], rts[7 * n + p]);
    m.S[p] = make_float4(rts[8 * n + p], rts[9 * n + p], rts[10 * n + p], rts[11 * n + p]);
}

// The last pushed frame's sums <-> slot (t - 1) mod 3; the other two slots cleared.
// The payload's sums are moved as 32-bit halves (a caller's buffer is 4-byte aligned).
// (An import whose header lies in device memory takes the frame count from there.)
__global__ void pbas_grad_sums_kernel(unsigned long long* gsum, uint32_t* canon, int64_t t, int to_canon,
                                      StateCheck check) {
    if (!header_matches(check)) return;
    if (check.header) t = (int64_t)check.header[8];
    const int j = threadIdx.x;  // 0..2
    const uint32_t prev = (uint32_t)((t + 2) % 3);
    if (to_canon) {
        unsigned long long v = 0ull;
        if (t > 0)
            for (int s = 0; s < kGradSlots; ++s) v += gsum[sum_index(prev, s, j)];
        canon[2 * j] = (uint32_t)v;
        canon[2 * j + 1] = (uint32_t)(v >> 32);
        return;
    }
    const unsigned long long v = (unsigned long long)canon[2 * j] | ((unsigned long long)canon[2 * j + 1] << 32);
    for (uint32_t f = 0; f < 3; ++f)
        for (int s = 0; s < kGradSlots; ++s) gsum[sum_index(f, s, j)] = f == prev && s == 0 && t > 0 ? v : 0ull;
}

inline unsigned blocks1d(int64_t n) { return (unsigned)((n + 255) / 256); }

template <int NMAX, bool TWO>
void launch_step_of(const PbasGradArgs& a, dim3 grid, hipStream_t s) {
    if (a.streaming) hipLaunchKernelGGL((pbas_grad_step_kernel<NMAX, true, TWO>), grid, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((pbas_grad_step_kernel<NMAX, false, TWO>), grid, dim3(kBlock), 0, s, a);
}
template <int NMAX>
void launch_step(const PbasGradArgs& a, dim3 grid, hipStream_t s) {
    if (a.c.min_matches == 2) launch_step_of<NMAX, true>(a, grid, s);
    else launch_step_of<NMAX, false>(a, grid, s);
}

}  // namespace

hipError_t pbas_grad_launch_init_state(const PbasGradPlanes& m, int npix, const PbasConsts& c, hipStream_t s) {
    hipLaunchKernelGGL(pbas_grad_init_kernel, dim3(blocks1d(npix)), dim3(256), 0, s, m, npix,
                       make_float4(c.R_lower[0], c.R_lower[1], c.R_lower[2], c.R_lower[3]), c.T_lower);
    return hipGetLastError();
}

hipError_t pbas_grad_launch_step(const PbasGradArgs& a, hipStream_t s) {
    if ((int64_t)a.t < a.c.N) {
        hipLaunchKernelGGL(pbas_grad_fill_kernel, dim3(blocks1d(a.npix)), dim3(kBlock), 0, s, a);
    } else {
        const int64_t tiles = (int64_t)((a.W + kTileW - 1) / kTileW) * ((a.H + kTileH - 1) / kTileH);
        if (tiles > 0x7fffffff) return hipErrorInvalidValue;
        const dim3 grid((unsigned)tiles);
        const int N = a.c.N;
        if (N <= 8) launch_step<8>(a, grid, s);
        else if (N <= 16) launch_step<16>(a, grid, s);
        else if (N <= 20) launch_step<20>(a, grid, s);
        else if (N <= 24) launch_step<24>(a, grid, s);
        else if (N <= 32) launch_step<32>(a, grid, s);
        else if (N <= 40) launch_step<40>(a, grid, s);
        else launch_step<64>(a, grid, s);
    }
    return hipGetLastError();
}

hipError_t pbas_grad_launch_flush(const PbasGradPlanes& m, int H, int W, uint32_t t_prev, const PbasConsts& c,
                                  hipStream_t s) {
    hipLaunchKernelGGL(pbas_grad_flush_kernel, dim3(blocks1d((int64_t)H * W)), dim3(256), 0, s, m, H, W, t_prev,
                       c.N, c.key0, c.key1);
    return hipGetLastError();
}

hipError_t pbas_grad_launch_export(const PbasGradPlanes& m, int npix, int N, int64_t t, uint8_t* out,
                                   const StateWords* header, hipStream_t s) {
    const size_t plane = (size_t)npix * 4;
    hipError_t e = pbas_launch_export_quads(m.samples, npix, N, out, s);
    if (e == hipSuccess) e = pbas_launch_export_quads(m.gsamples, npix, N, out + plane * N, s);
    if (e != hipSuccess) return e;
    float* dout = reinterpret_cast<float*>(out + 2 * plane * N);
    float* rts = reinterpret_cast<float*>(out + 6 * plane * N);
    hipLaunchKernelGGL(pbas_grad_export_kernel, dim3(blocks1d(npix)), dim3(256), 0, s, m, npix, N, dout, rts,
                       reinterpret_cast<uint32_t*>(out), header ? 1 : 0, header ? *header : StateWords());
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    uint32_t* canon = reinterpret_cast<uint32_t*>(out + 6 * plane * N + 12 * plane);
    hipLaunchKernelGGL(pbas_grad_sums_kernel, dim3(1), dim3(3), 0, s, m.gsum, canon, t, 1, StateCheck());
    return hipGetLastError();
}

hipError_t pbas_grad_launch_import(const PbasGradPlanes& m, int npix, int N, int64_t t, const uint8_t* in,
                                   const StateCheck& check, hipStream_t s) {
    const size_t plane = (size_t)npix * 4;
    hipError_t e = pbas_launch_import_quads(m.samples, npix, N, in, check, s);
    if (e == hipSuccess) e = pbas_launch_import_quads(m.gsamples, npix, N, in + plane * N, check, s);
    if (e != hipSuccess) return e;
    const float* din = reinterpret_cast<const float*>(in + 2 * plane * N);
    const float* rts = reinterpret_cast<const float*>(in + 6 * plane * N);
    hipLaunchKernelGGL(pbas_grad_import_kernel, dim3(blocks1d(npix)), dim3(256), 0, s, m, npix, N, din, rts, check);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    uint32_t* canon = const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(in + 6 * plane * N + 12 * plane));
    hipLaunchKernelGGL(pbas_grad_sums_kernel, dim3(1), dim3(3), 0, s, m.gsum, canon, t, 0, check);
    return hipGetLastError();
}

}  // namespace fgs
