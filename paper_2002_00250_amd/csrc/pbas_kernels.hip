// RGB-D Pixel-Based Adaptive Segmenter kernels (Sec. 3.2): one launch per frame
// (fill for the first N frames, then the tile update of pbas_device.h), the
// flush of pending neighbour writes for a state read-out, and the state
// import/export.
#include <cstring>

#include "device_common.h"
#include "fgs_internal.h"
#include "pbas_device.h"

namespace fgs {

using namespace pbas;

namespace {

// Frames 0..N-1: sample slot t takes the frame; the mask is empty.
__global__ __launch_bounds__(256) void pbas_fill_kernel(PbasStepArgs a) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < a.npix) fill_pixel(a, p);
}

// Register capacity class NMAX serves N in [class_min(NMAX), NMAX].
constexpr int class_min(int nmax) { return nmax <= 8 ? 2 : (nmax <= 40 ? nmax - 3 : nmax - 7); }

// One block per 64x4 tile on a one-dimensional grid (row-major tile order within a
// model): the grid's y extent is too small for the tile rows of a tall image.  One
// launch steps b.n models (one for a single push): workgroup w takes tile
// w - first[i] of model i, first[i] <= w < first[i + 1].
template <int NB, int NMAX, bool NT>
__global__ __launch_bounds__(kBlock) void pbas_step_kernel(PbasBatch<NB> b) {
    __shared__ PbasLds<NMAX> sh;
    const int w = (int)blockIdx.x;
    int i = 0;
#pragma unroll
    for (int j = 1; j < NB; ++j) i = w >= b.first[j] ? j : i;  // (first[j] is the grid size for j >= n)
    const int local = w - b.first[i], tiles_x = b.tiles_x[i];
    pbas_tile<NMAX, class_min(NMAX), NT>(b.a[i], local % tiles_x, local / tiles_x, sh);
}

// The state with the neighbour writes of the last processed frame (t_prev) applied: written back to
// the model (a flush, for fgs_get_state), or with EXPORT to the payload (samples[N], dhist[N], R[4],
// T[4] planes of 32 bits, S[4] of 16), with the model left as it is and its writes still pending:
// one launch and one pass over the samples, none of whose quads are written back a few bytes here
// and there.  Workgroups 0 .. tiles - 1 take the step's 64x4 tiles (the same scatter of the
// sources' writes into LDS, pbas_device.h); the others copy the D planes, which are the payload's
// as they are.  Bound by the bytes read and written: 123 MB at 640x480, N = 20, in 28.9 us
// (4.3 TB/s), where a flush, two transposes and a copy took 16.8 + 10.6 + 6.2 + 6.3 us; written
// back to the model as well, it took 37.5.  (The first four quads are read before the scatter, with
// the index clamped instead of a branch: with branches the reads went one at a time, 43.8 us.)
static_assert(kBlock == 256, "copy_block");
constexpr int kCopyWords = 256 * 4 * 4;  // words a block of 256 lanes copies, 4 x 16 bytes a lane
__device__ __forceinline__ void copy_block(uint32_t* __restrict__ dst, const uint32_t* __restrict__ src, int64_t words,
                                           int64_t block, int wide) {
    const int64_t first = block * kCopyWords;
    if (wide && first + kCopyWords <= words) {
        const uint4* s = reinterpret_cast<const uint4*>(src + first) + threadIdx.x;
        uint4* d = reinterpret_cast<uint4*>(dst + first) + threadIdx.x;
        const uint4 v0 = s[0], v1 = s[256], v2 = s[512], v3 = s[768];
        d[0] = v0;
        d[256] = v1;
        d[512] = v2;
        d[768] = v3;
        return;
    }
    const int64_t end = first + kCopyWords < words ? first + kCopyWords : words;
#pragma unroll 4
    for (int64_t j = first + threadIdx.x; j < end; j += 256) dst[j] = src[j];
}

// Quads q0 .. q0 + 3 of a pixel (the last one again where there are fewer).
struct QuadBatch {
    uint4 v[4];
};
__device__ __forceinline__ QuadBatch load_quads(const uint4* quads, int64_t n, int64_t p, int q0, int nq) {
    QuadBatch b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b.v[i] = quads[(int64_t)(q0 + i < nq ? q0 + i : nq - 1) * n + p];
    return b;
}

// The quad with `val` in place of the bytes whose bits are set.
__device__ __forceinline__ uint4 merge_quad(uint4 v, uint32_t val, uint32_t bits) {
    const uint32_t b0 = slot_byte_mask(bits, 0), b1 = slot_byte_mask(bits, 1), b2 = slot_byte_mask(bits, 2),
                   b3 = slot_byte_mask(bits, 3);
    return make_uint4((v.x & ~b0) | (val & b0), (v.y & ~b1) | (val & b1), (v.z & ~b2) | (val & b2),
                      (v.w & ~b3) | (val & b3));
}

// The writes into pixel p looked up by its own lane: each of its 8 neighbours that fired recomputes its
// draws and counts if it aimed the opposite way, 7 - d (the direction table is point symmetric).
__device__ __forceinline__ void pull_fired(PbasLds<64>& sh, const uint8_t* fire, int x, int y, int H, int W, int N,
                                           uint32_t t_prev, uint32_t k0, uint32_t k1) {
    for (int d = 0; d < 8; ++d) {
        const int qx = x + nb_dx(d), qy = y + nb_dy(d);
        if (qx < 0 || qx >= W || qy < 0 || qy >= H) continue;
        const uint32_t fb = fire[(int64_t)qy * W + qx] & 0xFu;  // (the high nibble: R flags)
        if (fb == 0u) continue;
        const U32x4 w1 = philox4x32_10((uint32_t)(qy * W + qx), t_prev, 1u, 0u, k0, k1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int dq, slot;
            intent_of(w1.v[j], N, dq, slot);
            if (((fb >> j) & 1u) && dq == 7 - d)
                sh.pend[(slot >> 3) * kBlock + threadIdx.x] |= 1u << (8 * j + (slot & 7));
        }
    }
}

// TILED: workgroups 0 .. tiles - 1 take the step's tiles; else 256 consecutive pixels each (frames
// that fill too little of their tiles, settle_of).
template <bool EXPORT, bool TILED>
__global__ __launch_bounds__(kBlock) void pbas_settle_kernel(PbasPlanes m, int H, int W, int N, int apply,
                                                             uint32_t t_prev, uint32_t k0, uint32_t k1, int tiles_x,
                                                             int tiles, uint32_t* __restrict__ out, int wide,
                                                             int has_header, StateWords header) {
    __shared__ PbasLds<64> sh;
    const int tid = threadIdx.x;
    const int64_t n = (int64_t)H * W;
    if (EXPORT) {
        write_header(out, has_header, header);
        if ((int)blockIdx.x >= tiles) {
            copy_block(out + n * N, m.dhist, n * N, (int64_t)blockIdx.x - tiles, wide);
            return;
        }
    }
    const int x0 = TILED ? ((int)blockIdx.x % tiles_x) * kTileW : 0, y0 = TILED ? ((int)blockIdx.x / tiles_x) * kTileH : 0;
    const int lx = tid % kTileW, ly = tid / kTileW;
    const int64_t first = TILED ? (int64_t)y0 * W + x0 : (int64_t)blockIdx.x * kBlock;
    const bool inside = TILED ? x0 + lx < W && y0 + ly < H : first + tid < n;
    const int64_t p = !inside ? first : TILED ? (int64_t)(y0 + ly) * W + x0 + lx : first + tid;
    const int nq = (N + 3) / 4;
    uint4* quads = reinterpret_cast<uint4*>(m.samples);
    QuadBatch b;
    if (EXPORT) b = load_quads(quads, n, p, 0, nq);  // on their way during the scatter
    uint32_t lastw = 0u;
    if (apply) {
        FireIn fin;
        if (TILED) fin = load_fire(m.fire[t_prev & 1u], x0, y0, H, W);
        lastw = m.last_in_pad ? *reinterpret_cast<const uint32_t*>(sample_byte(m.samples, n, N, (int)p, 0)) : m.last[p];
        for (int w = 0; w < (N + 7) / 8; ++w) sh.pend[w * kBlock + tid] = 0u;
        if (TILED) {
            __syncthreads();
            scatter_fired<64>(sh, fin, N, t_prev, k0, k1);
            __syncthreads();
        } else {  // (each lane its own words)
            const int y = (int)p / W;
            pull_fired(sh, m.fire[t_prev & 1u], (int)p - y * W, y, H, W, N, t_prev, k0, k1);
        }
    }
    if (!inside) return;
    const uint32_t keep = (lastw >> 24) != 0u ? 0xFFFFFFFFu : 0x00FFFFFFu;  // depth at t_prev?
    if (!EXPORT) {
        for (int q = 0; q < nq; ++q) {
            const uint32_t bits = apply ? (sh.pend[(q >> 1) * kBlock + tid] & keep) >> (4 * (q & 1)) & 0x0F0F0F0Fu : 0u;
            if (bits != 0u) quads[(int64_t)q * n + p] = merge_quad(quads[(int64_t)q * n + p], lastw, bits);
        }
        return;
    }
#pragma unroll 1
    for (int q0 = 0; q0 < nq; q0 += 4) {
        const QuadBatch next = load_quads(quads, n, p, q0 + 4, nq);
        uint32_t word[2] = {0u, 0u};  // (the second word is not there for the last odd pair: not used then)
        if (apply) {
            word[0] = sh.pend[(q0 >> 1) * kBlock + tid] & keep;
            if (q0 + 2 < nq) word[1] = sh.pend[((q0 >> 1) + 1) * kBlock + tid] & keep;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = merge_quad(b.v[i], lastw, word[i >> 1] >> (4 * (i & 1)) & 0x0F0F0F0Fu);
            uint32_t* o = out + (int64_t)(4 * (q0 + i)) * n + p;
            const int left = N - 4 * (q0 + i);
            if (left > 0) o[0] = v.x;
            if (left > 1) o[n] = v.y;
            if (left > 2) o[2 * n] = v.z;
            if (left > 3) o[3 * n] = v.w;
        }
        b = next;
    }
    const float4 r = m.R[p], t = m.T[p];
    const uint2 sv = m.S[p];
    float* rt = reinterpret_cast<float*>(out + 2 * n * N);
    uint16_t* s = reinterpret_cast<uint16_t*>(rt + 8 * n);
    rt[0 * n + p] = r.x; rt[1 * n + p] = r.y; rt[2 * n + p] = r.z; rt[3 * n + p] = r.w;
    rt[4 * n + p] = t.x; rt[5 * n + p] = t.y; rt[6 * n + p] = t.z; rt[7 * n + p] = t.w;
    s[0 * n + p] = (uint16_t)(sv.x & 0xFFFFu);
    s[1 * n + p] = (uint16_t)(sv.x >> 16);
    s[2 * n + p] = (uint16_t)(sv.y & 0xFFFFu);
    s[3 * n + p] = (uint16_t)(sv.y >> 16);
}

__global__ void pbas_init_state_kernel(PbasPlanes m, int npix, float4 Rl, float Tl) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    m.R[p] = Rl;
    m.T[p] = make_float4(Tl, Tl, Tl, Tl);
}

// Canonical slot-major sample planes (plane k = slot k of every pixel) <-> the
// device's quad planes.  Import writes the padding slots as zero.
__global__ void pbas_export_samples_kernel(const uint4* quads, uint32_t* out, int npix, int N) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    for (int q = 0; 4 * q < N; ++q) {
        const uint4 v = quads[q * n + p];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        for (int i = 0; i < 4 && 4 * q + i < N; ++i) out[(4 * q + i) * n + p] = w[i];
    }
}

__global__ void pbas_import_samples_kernel(uint4* quads, const uint32_t* in, int npix, int N, StateCheck check) {
    if (!header_matches(check)) return;
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    const int64_t n = npix;
    for (int q = 0; 4 * q < N; ++q) {
        uint32_t w[4];
        for (int i = 0; i < 4; ++i) w[i] = 4 * q + i < N ? in[(4 * q + i) * n + p] : 0u;
        quads[q * n + p] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// The payload into the model: workgroups 0 .. pixel_blocks - 1 a pixel per lane (samples, R, T, S),
// the others the D planes.  One launch (21.4 us for the 123 MB of 640x480, N = 20; as three 21.3 us,
// with a gap after each); see StateCheck for the header.
__global__ __launch_bounds__(256) void pbas_import_kernel(PbasPlanes m, int npix, int N, const uint32_t* __restrict__ in,
                                                          int pixel_blocks, int wide, StateCheck check) {
    if (!header_matches(check)) return;
    const int64_t n = npix;
    if ((int)blockIdx.x >= pixel_blocks) {
        copy_block(m.dhist, in + n * N, n * N, (int64_t)blockIdx.x - pixel_blocks, wide);
        return;
    }
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    uint4* quads = reinterpret_cast<uint4*>(m.samples);
#pragma unroll 4
    for (int q = 0; 4 * q < N; ++q) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = 4 * q + i < N ? in[(4 * q + i) * n + p] : 0u;
        quads[q * n + p] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    const float* rt = reinterpret_cast<const float*>(in + 2 * n * N);
    const uint16_t* s = reinterpret_cast<const uint16_t*>(rt + 8 * n);
    m.R[p] = make_float4(rt[0 * n + p], rt[1 * n + p], rt[2 * n + p], rt[3 * n + p]);
    m.T[p] = make_float4(rt[4 * n + p], rt[5 * n + p], rt[6 * n + p], rt[7 * n + p]);
    m.S[p] = make_uint2((uint32_t)s[0 * n + p] | ((uint32_t)s[1 * n + p] << 16),
                        (uint32_t)s[2 * n + p] | ((uint32_t)s[3 * n + p] << 16));
}

inline unsigned blocks1d(int n) { return (unsigned)((n + 255) / 256); }

template <int NB, int NMAX>
void launch_step_nt(const PbasBatch<NB>& b, dim3 grid, hipStream_t s) {
    if (b.a[0].streaming) hipLaunchKernelGGL((pbas_step_kernel<NB, NMAX, true>), grid, dim3(kBlock), 0, s, b);
    else hipLaunchKernelGGL((pbas_step_kernel<NB, NMAX, false>), grid, dim3(kBlock), 0, s, b);
}

// Register capacity for the N sample words: the smallest instantiated NMAX >= N
// (multiples of 4 up to 40, then 48, 56, 64), so that N >= class_min(NMAX).
int nmax_class(int N) {
    switch ((N + 3) / 4) {
        case 0: case 1: case 2: return 8;
        case 11: case 12: return 48;
        case 13: case 14: return 56;
        default: return (N + 3) / 4 <= 10 ? 4 * ((N + 3) / 4) : 64;
    }
}

template <int NB>
void launch_step_n(const PbasBatch<NB>& b, dim3 grid, hipStream_t s) {
    switch (nmax_class(b.a[0].c.N)) {
        case 8: launch_step_nt<NB, 8>(b, grid, s); break;
        case 12: launch_step_nt<NB, 12>(b, grid, s); break;
        case 16: launch_step_nt<NB, 16>(b, grid, s); break;
        case 20: launch_step_nt<NB, 20>(b, grid, s); break;
        case 24: launch_step_nt<NB, 24>(b, grid, s); break;
        case 28: launch_step_nt<NB, 28>(b, grid, s); break;
        case 32: launch_step_nt<NB, 32>(b, grid, s); break;
        case 36: launch_step_nt<NB, 36>(b, grid, s); break;
        case 40: launch_step_nt<NB, 40>(b, grid, s); break;
        case 48: launch_step_nt<NB, 48>(b, grid, s); break;
        case 56: launch_step_nt<NB, 56>(b, grid, s); break;
        default: launch_step_nt<NB, 64>(b, grid, s); break;
    }
}

template <int NB>
hipError_t launch_batch(const PbasStepArgs* a, int n, hipStream_t s) {
    PbasBatch<NB> b;
    std::memset(&b, 0, sizeof b);
    b.n = n;
    int64_t grid = 0;
    for (int i = 0; i < n; ++i) {
        b.a[i] = a[i];
        b.tiles_x[i] = (a[i].W + kTileW - 1) / kTileW;
        b.first[i] = (int32_t)grid;
        // ceil(W/64) * ceil(H/4) <= H*W/256 + W/64 + H/4 + 1 < 2^27 tiles for H*W <= 2^28
        grid += (int64_t)b.tiles_x[i] * ((a[i].H + kTileH - 1) / kTileH);
    }
    for (int i = n; i <= NB; ++i) b.first[i] = (int32_t)grid;
    for (int i = n; i < NB; ++i) b.tiles_x[i] = 1;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    launch_step_n(b, dim3((unsigned)grid), s);
    return hipGetLastError();
}

}  // namespace

hipError_t pbas_launch_init_state(const PbasPlanes& m, int npix, const PbasConsts& c,
                                  hipStream_t s) {
    hipLaunchKernelGGL(pbas_init_state_kernel, dim3(blocks1d(npix)), dim3(256), 0, s, m, npix,
                       make_float4(c.R_lower[0], c.R_lower[1], c.R_lower[2], c.R_lower[3]),
                       c.T_lower);
    return hipGetLastError();
}

int pbas_batch_key(const PbasStepArgs& a) {
    if ((int)a.t < a.c.N) return -1;
    return nmax_class(a.c.N) * 2 + (a.streaming ? 1 : 0);
}

hipError_t pbas_launch_step_batch(const PbasStepArgs* a, int n, hipStream_t s) {
    if (n < 1 || n > kBatchMax) return hipErrorInvalidValue;
    for (int i = 0; i < n; ++i) {
        const int key = pbas_batch_key(a[i]);
        if (key < 0 || key != pbas_batch_key(a[0])) return hipErrorInvalidValue;
    }
    return n == 1 ? launch_batch<1>(a, n, s) : launch_batch<kBatchMax>(a, n, s);
}

hipError_t pbas_launch_step(const PbasStepArgs& a, hipStream_t s) {
    if (pbas_batch_key(a) < 0) {
        hipLaunchKernelGGL(pbas_fill_kernel, dim3(blocks1d(a.npix)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    return pbas_launch_step_batch(&a, 1, s);
}

hipError_t pbas_launch_export_quads(const uint32_t* quads, int npix, int N, uint8_t* out, hipStream_t s) {
    hipLaunchKernelGGL(pbas_export_samples_kernel, dim3(blocks1d(npix)), dim3(256), 0, s,
                       reinterpret_cast<const uint4*>(quads), reinterpret_cast<uint32_t*>(out), npix, N);
    return hipGetLastError();
}

hipError_t pbas_launch_import_quads(uint32_t* quads, int npix, int N, const uint8_t* in, const StateCheck& check,
                                    hipStream_t s) {
    hipLaunchKernelGGL(pbas_import_samples_kernel, dim3(blocks1d(npix)), dim3(256), 0, s,
                       reinterpret_cast<uint4*>(quads), reinterpret_cast<const uint32_t*>(in), npix, N, check);
    return hipGetLastError();
}

namespace {

// Blocks that copy the D planes, and whether they may use 16-byte accesses.
int64_t copy_blocks(int64_t words) { return (words + kCopyWords - 1) / kCopyWords; }
bool wide_copy(const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; }

// Workgroups of a settle launch: tiles (each fire byte read once, an LDS scatter) where the frame fills
// at least 3/8 of them, else consecutive pixels (eight fire bytes each).  307,200 pixels, N = 20, export
// and flush in us with their calls, by tiles: 640 wide 30.1 and 26.0, 24 wide (3/8) 31.7 and 27.6, 16 wide
// 35.8 and 29.1, 5 wide 68.3 and 51.6; by pixels 31.9 to 32.4 and 28.7 to 29.2 at every width.
struct Settle {
    bool tiled;
    int tiles_x;
    int64_t groups;
};
Settle settle_of(int H, int W) {
    const int tiles_x = (W + kTileW - 1) / kTileW;
    const int64_t tiles = (int64_t)tiles_x * ((H + kTileH - 1) / kTileH), n = (int64_t)H * W;
    const bool tiled = 8 * n >= 3 * tiles * kTileW * kTileH;
    return Settle{tiled, tiles_x, tiled ? tiles : (n + kBlock - 1) / kBlock};
}

template <bool EXPORT>
hipError_t launch_settle(const PbasPlanes& m, int H, int W, bool apply, uint32_t t_prev, const PbasConsts& c, uint32_t* out,
                         int wide, const StateWords* header, hipStream_t s) {
    const Settle l = settle_of(H, W);
    const int64_t grid = l.groups + (EXPORT ? copy_blocks((int64_t)H * W * c.N) : 0);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    const StateWords h = header ? *header : StateWords();
    if (l.tiled)
        hipLaunchKernelGGL((pbas_settle_kernel<EXPORT, true>), dim3((unsigned)grid), dim3(kBlock), 0, s, m, H, W, c.N,
                           apply ? 1 : 0, t_prev, c.key0, c.key1, l.tiles_x, (int)l.groups, out, wide, header ? 1 : 0, h);
    else
        hipLaunchKernelGGL((pbas_settle_kernel<EXPORT, false>), dim3((unsigned)grid), dim3(kBlock), 0, s, m, H, W, c.N,
                           apply ? 1 : 0, t_prev, c.key0, c.key1, l.tiles_x, (int)l.groups, out, wide, header ? 1 : 0, h);
    return hipGetLastError();
}

}  // namespace

hipError_t pbas_launch_flush(const PbasPlanes& m, int H, int W, uint32_t t_prev, const PbasConsts& c,
                             hipStream_t s) {
    return launch_settle<false>(m, H, W, true, t_prev, c, nullptr, 0, nullptr, s);
}

// Canonical payload: samples[N] u32, dhist[N] u32, R[4] f32, T[4] f32, S[4] u16
// (out and in are 4-byte aligned device buffers).
hipError_t pbas_launch_export(const PbasPlanes& m, int H, int W, bool pending, uint32_t t_prev, const PbasConsts& c,
                              uint8_t* out, const StateWords* header, hipStream_t s) {
    uint32_t* o = reinterpret_cast<uint32_t*>(out);
    const bool wide = wide_copy(m.dhist, o + (int64_t)H * W * c.N);
    return launch_settle<true>(m, H, W, pending, t_prev, c, o, wide ? 1 : 0, header, s);
}

hipError_t pbas_launch_import(const PbasPlanes& m, int npix, int N, const uint8_t* in, const StateCheck& check,
                              hipStream_t s) {
    const int64_t words = (int64_t)npix * N, px = blocks1d(npix), grid = px + copy_blocks(words);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    const uint32_t* i = reinterpret_cast<const uint32_t*>(in);
    hipLaunchKernelGGL(pbas_import_kernel, dim3((unsigned)grid), dim3(256), 0, s, m, npix, N, i, (int)px,
                       wide_copy(m.dhist, i + words) ? 1 : 0, check);
    return hipGetLastError();
}

}  // namespace fgs
