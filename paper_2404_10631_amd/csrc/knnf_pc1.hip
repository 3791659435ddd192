// knnf_pc1.hip -- the one-band representation I of a hyperspectral cube (the
// PC1 projection step that feeds the KNN filter), for CDNA4 (gfx950).
//
// Method (PCA, Sec. II.C.2): centre every band by its average (step (i)) and
// project the centred image onto the first eigenvector (step (iv)); the GPU
// versions centre the cube and compute one matrix-vector product in double
// precision (Sec. III.A.2.a/d, III.B.2.a/d).  The covariance and eigenvector
// steps are not part of this library: band averages and eigenvector are
// inputs.  The KNN filter reads a normalised I (Sec. II.C.3); the reading
// taken here is min-max normalisation to [0, 1] over the frame.
//
//   I[p]  = sum_b (cube[p][b] - mean[b]) * vec[b]       binary64
//   I'[p] = (I[p] - min I) / (max I - min I)            binary64, 0 if constant
//   out[p] = binary32 rounding of I (or I')
//
// The step is HBM-bound (4 B per pixel and band, read once).  Lane layout of
// the projection kernel: a segment of S lanes covers one pixel, lane j of the
// segment reads bands 4j .. 4j+3 with one 16-byte load, so a wavefront reads
// 64/S whole pixels contiguously per load; the lane keeps its four averages
// and eigenvector entries in registers for the whole launch.  The segment sum
// is a butterfly over the S lanes.  A block takes one contiguous range of
// pixels, its four wavefronts side by side: with the wavefronts' reads spread
// over the cube in a grid-stride loop, a plain read reached 5.7 instead of 6.5
// TB/s (raw projection of 380 x 480 x 128: 18.2 and 17.2 us per call, about
// 2.3 us of each the launch).  Band counts that are no multiple of 4 and
// unaligned cubes take the same path (500 x 500 x 33: 13.0 us with the
// normalisation, 49.6 us with one thread per pixel); PC1_FEW_BANDS and fewer, and more
// than 256, have a thread per pixel.
// Normalisation needs min and max over the frame: each projection block stores
// its (min, max) pair, and every block of the second launch reduces those pairs
// before rescaling its pixels (no atomics on one address, no device-wide fence).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "../../include/knnf.h"
#include "knnf_device.h"

namespace knnf {
namespace {

constexpr int PC1_THREADS = 256;
constexpr int PC1_UNROLL = 4;  // loads of a wavefront in flight together (8: no faster)
// Projection grid: a block takes at least 32 KiB of the cube (500 x 500 x 33:
// 13.0 us, 15.2 us with blocks of 8 KiB, 14.5 with 64), and there are no more
// blocks than the normalisation's blocks can reduce the pairs of at once
// (1000 x 1000 x 100: 88.8 us, 91.2 with at most 1,024 blocks).
constexpr int PC1_MAX_BLOCKS = 4096;
constexpr int64_t PC1_BLOCK_BYTES = 32 * 1024;
// One thread per pixel for few bands, where a wavefront's rows share cache lines and no
// sum crosses lanes (700 x 800: 4 bands 12.1 against 23.3 us with segments, 9 bands 13.3 /
// 18.8, 10 bands 15.7 / 17.9, 11 bands 16.9 / 16.7; 1000 x 1500 x 10: 32.6 / 30.8), and
// beyond the 256 bands of a segment of 64 lanes.  There each thread's row is a stream of
// its own, and more than four blocks of them per CU evict each other's lines (500 x 800 x
// 300: 860 us with 1,024 blocks, 2,024 with 4,096).
constexpr int PC1_FEW_BANDS = 10;
constexpr int PC1_PIXEL_BLOCKS = 1024;

// Value of the partner lane for one butterfly step (64-bit through two
// 32-bit lane moves): DPP quad_perm xor 1 / xor 2, row_half_mirror (pairs the
// two quads of 8 lanes), row_mirror (the two halves of 16), and the
// permlane16 / permlane32 swaps (rows of 16, halves of 64).
template <int STEP>
__device__ __forceinline__ double partner(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    if constexpr (STEP < 4) {
        constexpr int ctrl = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : 0x140;
        lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, ctrl, 0xF, 0xF, false);
        hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, ctrl, 0xF, 0xF, false);
    } else if constexpr (STEP == 4) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        lo = (lane & 16) ? a[0] : a[1];
        hi = (lane & 16) ? b[0] : b[1];
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        lo = (lane & 32) ? a[0] : a[1];
        hi = (lane & 32) ? b[0] : b[1];
    }
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum over each aligned group of S lanes (S = 8, 16, 32, 64); every lane of the
// group ends with the same value (each step adds two equal-order partial sums,
// and binary64 addition is commutative).
template <int S>
__device__ __forceinline__ double seg_sum(double v) {
    v += partner<0>(v);
    v += partner<1>(v);
    v += partner<2>(v);
    if constexpr (S >= 16) v += partner<3>(v);
    if constexpr (S >= 32) v += partner<4>(v);
    if constexpr (S >= 64) v += partner<5>(v);
    return v;
}

// Block-wide min and max of per-thread values; thread 0 gets the result.
__device__ void block_minmax(double lo, double hi, double* out_lo, double* out_hi) {
    __shared__ double slo[PC1_THREADS / 64], shi[PC1_THREADS / 64];
    lo = fmin(lo, partner<0>(lo)), hi = fmax(hi, partner<0>(hi));
    lo = fmin(lo, partner<1>(lo)), hi = fmax(hi, partner<1>(hi));
    lo = fmin(lo, partner<2>(lo)), hi = fmax(hi, partner<2>(hi));
    lo = fmin(lo, partner<3>(lo)), hi = fmax(hi, partner<3>(hi));
    lo = fmin(lo, partner<4>(lo)), hi = fmax(hi, partner<4>(hi));
    lo = fmin(lo, partner<5>(lo)), hi = fmax(hi, partner<5>(hi));
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        slo[w] = lo;
        shi[w] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < PC1_THREADS / 64; ++k) {
            lo = fmin(lo, slo[k]);
            hi = fmax(hi, shi[k]);
        }
        *out_lo = lo;
        *out_hi = hi;
    }
}

// This block's min and max -> pairs[2 * blockIdx.x .. +1] (plain stores: the
// normalisation reads them in the next launch).
__device__ void publish_minmax(double lo, double hi, double* pairs) {
    __shared__ double blo, bhi;
    block_minmax(lo, hi, &blo, &bhi);
    if (threadIdx.x == 0) {
        pairs[2 * blockIdx.x] = blo;
        pairs[2 * blockIdx.x + 1] = bhi;
    }
}

// Four floats at a 4-byte aligned address, as one load.
__device__ __forceinline__ float4 load4(const float* p) {
    float4 v;
    memcpy(&v, __builtin_assume_aligned(p, 4), sizeof v);
    return v;
}

// Projection, 4 <= bands <= 4 * S, any 4-byte alignment.  Where bands is no
// multiple of 4, a pixel's last piece starts at bands - 4 and the bands that it
// repeats count as 0.  Block b takes the pixels [b * per, (b + 1) * per).
template <int S>
__global__ void __launch_bounds__(PC1_THREADS)
pc1_project_vec4(const float* __restrict__ cube, int64_t npix, int bands,
                 const double* __restrict__ mean, const double* __restrict__ vec,
                 float* __restrict__ out, double* __restrict__ ws, double* __restrict__ pairs,
                 int64_t per) {
    constexpr int PW = 64 / S;  // pixels per wavefront per load
    constexpr int STEP = PW * PC1_UNROLL, WAVES = PC1_THREADS / 64;
    const int lane = threadIdx.x & 63;
    const int j = lane % S;      // slot in the segment
    const int seg = lane / S;    // pixel of the segment within the wavefront group
    const int np = (bands + 3) >> 2;
    const bool act = j < np;
    const int b0 = j < np - 1 ? 4 * j : bands - 4;        // first band of the lane's piece
    const int rep = j == np - 1 ? 4 * np - bands : 0;     // its bands that the piece before covers
    const int64_t p1 = min(npix, (int64_t)(blockIdx.x + 1) * per);
    int64_t base = (int64_t)blockIdx.x * per + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * STEP;
    double mu[4], w[4];
    float4 x[PC1_UNROLL];
    // every lane loads (past the last pixel or band: a clamped address whose
    // value is dropped), so all loads are in flight together
    auto load = [&]() {
        const float* rp = cube + min(base, npix - 1) * (int64_t)bands;
        const uint32_t last = (uint32_t)min((int64_t)STEP, npix - 1 - min(base, npix - 1));
#pragma unroll
        for (int u = 0; u < PC1_UNROLL; ++u)
            x[u] = load4(rp + (min((uint32_t)(u * PW + seg), last) * (uint32_t)bands + (uint32_t)b0));
    };
    load();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool use = act && i >= rep;
        mu[i] = mean[b0 + i];
        w[i] = use ? vec[b0 + i] : 0.0;
    }
    double lo = __builtin_inf(), hi = -__builtin_inf();
    for (; base < p1; base += STEP * WAVES) {
        double t[PC1_UNROLL];
#pragma unroll
        for (int u = 0; u < PC1_UNROLL; ++u) {
            if (bands & 3) {
                x[u].x = rep > 0 ? 0.f : x[u].x;
                x[u].y = rep > 1 ? 0.f : x[u].y;
                x[u].z = rep > 2 ? 0.f : x[u].z;
            }
            double s = 0.0;
            s = fma((double)x[u].x - mu[0], w[0], s);
            s = fma((double)x[u].y - mu[1], w[1], s);
            s = fma((double)x[u].z - mu[2], w[2], s);
            s = fma((double)x[u].w - mu[3], w[3], s);
            t[u] = act ? s : 0.0;
        }
        const int64_t cur = base;
        if (base + STEP * WAVES < p1) {
            base += STEP * WAVES;
            load();  // the next step's loads, ahead of this one's sums
            base = cur;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < PC1_UNROLL; ++u) {
            const int64_t p = cur + u * PW + seg;
            const double s = seg_sum<S>(t[u]);
            if (p < p1) {
                lo = fmin(lo, s);
                hi = fmax(hi, s);
                if (j == 0) {
                    if (ws) ws[p] = s;
                    else out[p] = (float)s;
                }
            }
        }
    }
    if (ws) publish_minmax(lo, hi, pairs);
}

// Projection for few or for more than 256 bands: one thread per pixel.
__global__ void __launch_bounds__(PC1_THREADS)
pc1_project_scalar(const float* __restrict__ cube, int64_t npix, int bands,
                   const double* __restrict__ mean, const double* __restrict__ vec,
                   float* __restrict__ out, double* __restrict__ ws, double* __restrict__ pairs) {
    const int64_t nthreads = (int64_t)gridDim.x * PC1_THREADS;
    double lo = __builtin_inf(), hi = -__builtin_inf();
    for (int64_t p = (int64_t)blockIdx.x * PC1_THREADS + threadIdx.x; p < npix; p += nthreads) {
        const float* row = cube + p * (int64_t)bands;
        double t = 0.0;
        for (int b = 0; b < bands; ++b) t = fma((double)row[b] - mean[b], vec[b], t);
        lo = fmin(lo, t);
        hi = fmax(hi, t);
        if (ws) ws[p] = t;
        else out[p] = (float)t;
    }
    if (ws) publish_minmax(lo, hi, pairs);
}

__global__ void __launch_bounds__(PC1_THREADS)
pc1_normalise(const double* __restrict__ ws, int64_t npix, const double* __restrict__ pairs,
              int npairs, float* __restrict__ out) {
    // four pixels per thread and step, their loads issued together; the first
    // step's and the pairs' are in flight at once
    const int64_t nthreads = (int64_t)gridDim.x * PC1_THREADS;
    int64_t p = (int64_t)blockIdx.x * PC1_THREADS + threadIdx.x;
    double x[4];
    auto load = [&]() {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t pk = p + k * nthreads;
            x[k] = ws[pk < npix ? pk : npix - 1];
        }
    };
    load();
    // min and max over the frame from the projection blocks' pairs
    typedef double d2 __attribute__((ext_vector_type(2)));
    double l = __builtin_inf(), h = -__builtin_inf();
    for (int b = threadIdx.x; b < npairs; b += 4 * PC1_THREADS) {
        d2 q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = ((const d2*)pairs)[min(b + k * PC1_THREADS, npairs - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            l = fmin(l, q[k].x);
            h = fmax(h, q[k].y);
        }
    }
    __shared__ double pair[2];
    block_minmax(l, h, &pair[0], &pair[1]);
    __syncthreads();
    const double lo = pair[0], hi = pair[1];
    const bool flat = !(hi > lo);
    const double range = hi - lo;
    for (;;) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t pk = p + k * nthreads;
            if (pk < npix) out[pk] = flat ? 0.0f : (float)((x[k] - lo) / range);
        }
        p += 4 * nthreads;
        if (p >= npix) break;
        load();
    }
}

}  // namespace

int pc1_max_blocks() { return PC1_MAX_BLOCKS; }

int launch_pc1_normalise(const double* ws, int64_t npix, const double* pairs, int npairs,
                         float* out, int num_cu, void* stream) {
    const int64_t nb = (npix + PC1_THREADS - 1) / PC1_THREADS;
    const int nblocks = (int)(nb < (int64_t)num_cu ? nb : (int64_t)num_cu);
    hipLaunchKernelGGL(pc1_normalise, dim3(nblocks), dim3(PC1_THREADS), 0, (hipStream_t)stream, ws,
                       npix, pairs, npairs, out);
    return (int)hipGetLastError();
}

// ---- Static scratch of knnf_pc1_noalloc: the projection blocks' (min, max)
// pairs, then the binary64 projection of up to KNNF_PC1_NOALLOC_MAX_PIXELS
// pixels.  Each device holds its own copy for the life of the process; host
// code uses the device address hipGetSymbolAddress reports for it (the
// array's name is a host-side stand-in, not a device address).
constexpr size_t kScratchHead = 65536;
static_assert(2 * PC1_MAX_BLOCKS * sizeof(double) <= kScratchHead, "pairs fit the scratch head");
constexpr size_t kScratchBytes = kScratchHead + sizeof(double) * (size_t)KNNF_PC1_NOALLOC_MAX_PIXELS;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::once_flag g_scratch_once[kMaxDevices];
void* g_scratch_ptr[kMaxDevices];
hipError_t g_scratch_err[kMaxDevices];
}  // namespace

int pc1_scratch_init(int device, void** ptr) {
    *ptr = nullptr;
    if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
    // once per device, with that device current (the caller sets it)
    std::call_once(g_scratch_once[device], [device] {
        g_scratch_err[device] = hipGetSymbolAddress(&g_scratch_ptr[device], HIP_SYMBOL(scratch));
        if (g_scratch_err[device] != hipSuccess) g_scratch_ptr[device] = nullptr;
    });
    *ptr = g_scratch_ptr[device];
    return (int)g_scratch_err[device];
}

size_t pc1_scratch_head() { return kScratchHead; }

int launch_pc1(const float* cube, int64_t npix, int bands, const double* mean, const double* vec,
               float* out, double* ws, double* pairs, int num_cu, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    int blocks;
    if (bands > PC1_FEW_BANDS && bands <= 256) {
        const int S = bands <= 32 ? 8 : bands <= 64 ? 16 : bands <= 128 ? 32 : 64;
        // a block's step: PC1_UNROLL loads of each wavefront
        const int64_t step = (int64_t)(PC1_THREADS / 64) * (64 / S) * PC1_UNROLL;
        const int64_t steps = (npix + step - 1) / step;
        // steps per block: at least PC1_BLOCK_BYTES of the cube
        const int64_t some = (PC1_BLOCK_BYTES + step * bands * 4 - 1) / (step * bands * 4);
        const int64_t per = std::max<int64_t>(some, (steps + PC1_MAX_BLOCKS - 1) / PC1_MAX_BLOCKS);
        blocks = (int)((steps + per - 1) / per);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(PC1_THREADS), 0, st, cube, npix, bands,
                               mean, vec, out, ws, pairs, per * step);
        };
        if (S == 8) launch(pc1_project_vec4<8>);
        else if (S == 16) launch(pc1_project_vec4<16>);
        else if (S == 32) launch(pc1_project_vec4<32>);
        else launch(pc1_project_vec4<64>);
    } else {
        const int64_t want = (npix + PC1_THREADS - 1) / PC1_THREADS;
        blocks = (int)(want < PC1_PIXEL_BLOCKS ? want : PC1_PIXEL_BLOCKS);
        hipLaunchKernelGGL(pc1_project_scalar, dim3(blocks), dim3(PC1_THREADS), 0, st, cube, npix,
                           bands, mean, vec, out, ws, pairs);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !ws) return (int)e;
    return launch_pc1_normalise(ws, npix, pairs, blocks, out, num_cu, stream);
}

}  // namespace knnf
