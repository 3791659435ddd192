// knnf_svm.hip -- the SVM probability stage (the pixel-wise classifier whose
// probability maps the KNN filter averages), for CDNA4 (gfx950).
//
// Method (one-vs-one SVM, classification stage, Sec. II.C.1; GPU versions
// Sec. III.A.1 and III.B.1), per pixel x (a spectrum of `bands` values):
//   (i)   f[m] = sum_b w[m][b] x[b] + bias[m]  for every hyperplane m, one per
//         class pair (i, j), i < j, in lexicographic order;
//   (ii)  r[m] = 1 / (1 + exp(A[m] f[m] + B[m])), clamped to [1e-7, 1 - 1e-7]:
//         the probability of class i within the pair, 1 - r[m] that of j;
//   (iii) pairwise coupling (the second method of Wu, Lin and Weng, cited as
//         [30]): with Q[t][t] = sum_{s != t} r_st^2 and Q[t][j] = -r_jt r_tj,
//         sweep p[t] <- (p^T Q p - sum_{j != t} Q[t][j] p[j]) / Q[t][t], each
//         update followed by renormalising p, from the uniform p, until
//         max_t |(Q p)[t] - p^T Q p| < 0.005 / C or 100 sweeps.
// Every step is binary64; the probabilities are rounded once to binary32,
// pixel-major with the class fastest (the layout the filter reads).
//
// Work shape: the cube is read once (4 B per pixel and band); the rest is
// per-pixel binary64 arithmetic.  Step (i) is a matrix product, [pixels x
// bands] by [bands x M], on the binary64 matrix instruction
// (v_mfma_f64_4x4x4_4b: four blocks of 4 pixels x 4 bands x 4 hyperplanes).
// It is used for its operand layout, not for its rate: on this chip it takes 16
// cycles for 256 FMAs, the vector pipe's own binary64 rate, and does not
// overlap with that pipe.  But a lane-per-pixel dot product needs every weight
// in every lane, 8 bytes of LDS return bandwidth per FMA and lane (128 B/clk per
// CU: 45k of the 65k cycles that the fused call on the 380 x 480 x 128 cube
// took in that form); here a weight read from LDS serves 16 pixels.
//   * A wavefront owns a tile of 64 pixels and goes through it in items of 16
//     pixels x up to 128 bands: one contiguous span of memory, each cache line
//     requested once.  A load takes two pixel rows, 32 lanes of 16-byte pieces
//     (4 bands) each; up to 64, 32 and 16 bands, 4, 8
//     and 16 rows.  Any band count from 4 on
//     and any 4-byte alignment: the last piece of a pixel starts at bands - 4,
//     and the bands that it repeats count as 0.  The next item's loads are
//     issued before the current one is used.  (Two items in flight, persistent
//     blocks of two to five tiles per wavefront, and blocks of 64, 128 and 512
//     threads measured equal or slower.)
//   * The item goes through a wavefront-private LDS buffer into the matrix
//     operand layout (lane l: pixel l % 16 of a group of 16, piece l / 16 of a
//     k-step of 16 bands; component e of the piece is the operand of matrix
//     step e).  Loaded in that layout straight from memory, the lanes of a
//     quarter wavefront touch 16 cache lines, and the first-level cache held
//     the loads alone to 3.4 TB/s.
//   * The weights of up to 128 bands are staged in LDS once per block, in
//     operand order.
//   * The sums go through LDS to one lane per pixel for the sigmoids and the
//     coupling iteration, whose sweep count differs from pixel to pixel.
// The fused variant (PC1 = true) adds the PC1 projection, so the pipeline's two steps
// before the filter read the cube once.  Its terms are centred, so they can not be one
// more column of the product: each lane forms those of the operands that it has
// converted for the product, (x - average) times eigenvector entry, whose 16-byte pairs
// lie in LDS beside the weights (0 for the bands and slots that the product leaves out).
// (Uncentred, as a column of the product with one constant subtracted at the end, the
// error was that of the uncentred terms: sensor counts of 60,000 +- 2 came out up to 0.18
// of a binary32 ulp off at 128 bands, 1.1 at 4,096.  Formed as the pieces arrive, before
// the product, the terms cost a second conversion, an exchange through LDS and the work
// of idle lanes: 1000 x 1000, four classes, 100 bands 121 us a call, 111 in this form;
// 132 bands 172 and 149.)
// What bounds it: 1000 x 1000 x 100, four classes, 84.5 us (105 us with the
// lane-per-pixel product): the same kernel without its arithmetic takes 74 us
// (5.6 TB/s, the rate of a plain read of the cube), the vector pipe is busy
// for 50 us, and the two overlap only in part.  380 x 480 x 128 fused, 24.4 us
// of kernel (kernel trace), 15 of them the cube's read at that rate: all its blocks are
// resident at once, so they load together and then couple together.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string.h>

#include "knnf_device.h"

namespace knnf {
namespace {

constexpr int SVM_THREADS = 256;              // four wavefronts, a tile of 64 pixels each
constexpr int SVM_TILE = 64;
constexpr int SVM_SWEEPS = 100;
constexpr double SVM_CLAMP = 1e-7;

// Hyperplane of the pair (i, j), i < j, in the order (0,1), (0,2), ..., (C-2,C-1).
template <int C>
__device__ __forceinline__ constexpr int pair_index(int i, int j) {
    return i * C - i * (i + 1) / 2 + (j - i - 1);
}

// Block-wide (min, max) of per-thread values -> pairs[2 * blockIdx.x ..];
// lds: 2 NT / 64 doubles that no thread still uses.
template <int NT>
__device__ void svm_publish_minmax(double lo, double hi, double* pairs, double* lds) {
    double *slo = lds, *shi = lds + NT / 64;
    for (int m = 1; m < 64; m <<= 1) {
        lo = fmin(lo, __shfl_xor(lo, m));
        hi = fmax(hi, __shfl_xor(hi, m));
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        slo[wv] = lo;
        shi[wv] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < NT / 64; ++k) {
            lo = fmin(lo, slo[k]);
            hi = fmax(hi, shi[k]);
        }
        pairs[2 * blockIdx.x] = lo;
        pairs[2 * blockIdx.x + 1] = hi;
    }
}

// 1 / x in binary64 for the finite, normal x of the sigmoid and the coupling:
// the hardware reciprocal (relative error e below 2^-20) corrected by 1 + e +
// e^2 (an error of an ulp or so, far below the 1e-6 the probabilities are held
// to, for a third of the instructions of an IEEE division).
__device__ __forceinline__ double rcp64(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// exp(z) for |z| <= 700: z = k ln 2 + r with |r| <= ln 2 / 2 (ln 2 in two
// parts), and on that interval the truncated Chebyshev series of degree 11
// (relative error 1.6e-17 before rounding), by Horner's rule.  The sigmoid's argument is capped to that range, so the special cases
// of the library function (a third of its instructions) have no place.
__device__ __forceinline__ double exp_capped(double z) {
    const double k = __builtin_rint(z * 0x1.71547652b82fep+0);
    double r = fma(k, -0x1.62e42fefa39efp-1, z);
    r = fma(k, -0x1.abc9e3b39803fp-56, r);
    double p = 0x1.af785e0dfd450p-26;
    p = fma(p, r, 0x1.28b4063caeaedp-22);
    p = fma(p, r, 0x1.71dde76a2d404p-19);
    p = fma(p, r, 0x1.a01991aba4014p-16);
    p = fma(p, r, 0x1.a01a01b80266fp-13);
    p = fma(p, r, 0x1.6c16c187fc3f8p-10);
    p = fma(p, r, 0x1.111111110db75p-7);
    p = fma(p, r, 0x1.555555554f0ccp-5);
    p = fma(p, r, 0x1.5555555555562p-3);
    p = fma(p, r, 0x1.0000000000011p-1);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_ldexp(p, (int)k);
}

// Steps (ii) and (iii) for one pixel: sigmoids of the decision values f,
// then the coupling sweeps; writes the C probabilities to o.
template <int C>
__device__ __forceinline__ void svm_couple(const double (&f)[C * (C - 1) / 2],
                                           const double* __restrict__ bias,
                                           const double* __restrict__ A,
                                           const double* __restrict__ B, float* o) {
    constexpr int M = C * (C - 1) / 2;
    // (ii) binary probabilities; r[m] is that of the pair's first class (z is
    // capped where the clamp decides anyway, so exp(z) and 1 + exp(z) are
    // finite and normal)
    double r[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const double z = fmax(fmin(fma(f[m] + bias[m], A[m], B[m]), 700.0), -700.0);
        const double s = rcp64(1.0 + exp_capped(z));
        r[m] = fmin(fmax(s, SVM_CLAMP), 1.0 - SVM_CLAMP);
    }
    // (iii) coupling.  Q[t][t] sums r_st^2 over s in ascending order;
    // the off-diagonal Q[t][j] = -r_jt r_tj is the same for (t, j) and (j, t).
    double qtt[C];
#pragma unroll
    for (int t = 0; t < C; ++t) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < C; ++u) {
            if (u == t) continue;
            const double rut = u < t ? r[pair_index<C>(u, t)] : 1.0 - r[pair_index<C>(t, u)];
            s = s + rut * rut;
        }
        qtt[t] = s;
    }
    double qo[M];
#pragma unroll
    for (int m = 0; m < M; ++m) qo[m] = -((1.0 - r[m]) * r[m]);
    auto Q = [&](int t, int j) -> double {
        return t == j ? qtt[t] : t < j ? qo[pair_index<C>(t, j)] : qo[pair_index<C>(j, t)];
    };

    // The sweep keeps Q p and p^T Q p up to date instead of recomputing them:
    // the new p[t] equals p[t] + d with d = (p^T Q p - (Q p)[t]) / Q[t][t], by
    // which Q p gains d times column t of Q and p^T Q p gains d times the sum of
    // (Q p)[t] before and after.  Renormalising after each update is left to
    // the end of the sweep: with u = s p, s the sum of u, the same step is
    // u[t] += e, e = s d = (u^T Q u / s - (Q u)[t]) / Q[t][t], and s += e.  Same
    // fixed-point step as the plain form, O(C) per update instead of O(C^2).
    double p[C], qp[C], rq[C];
#pragma unroll
    for (int t = 0; t < C; ++t) {
        p[t] = 1.0 / C;
        rq[t] = rcp64(qtt[t]);
    }
    double pqp = 0.0;
#pragma unroll
    for (int t = 0; t < C; ++t) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < C; ++j) s = fma(Q(t, j), p[j], s);
        qp[t] = s;
        pqp = fma(p[t], s, pqp);
    }
    const double eps = 0.005 / C;
    for (int sweep = 0; sweep < SVM_SWEEPS; ++sweep) {
        double err = 0.0;
#pragma unroll
        for (int t = 0; t < C; ++t) err = fmax(err, fabs(qp[t] - pqp));
        if (!(err >= eps)) break;
        double s = 1.0, inv = 1.0;
#pragma unroll
        for (int t = 0; t < C; ++t) {
            const double q0 = qp[t];
            const double d = fma(pqp, inv, -q0) * rq[t];
#pragma unroll
            for (int j = 0; j < C; ++j) qp[j] = fma(d, Q(j, t), qp[j]);
            pqp = fma(d, q0 + qp[t], pqp);
            p[t] += d;
            s += d;
            inv = rcp64(s);
        }
#pragma unroll
        for (int t = 0; t < C; ++t) {
            qp[t] *= inv;
            p[t] *= inv;
        }
        pqp *= inv * inv;
    }
#pragma unroll
    for (int t = 0; t < C; ++t) o[t] = (float)p[t];
}

// Four floats at a 4-byte aligned address, as one load.
__device__ __forceinline__ float4 load4(const char* p) {
    float4 v;
    memcpy(&v, __builtin_assume_aligned(p, 4), sizeof v);
    return v;
}

// Columns of the product, the M hyperplanes, in groups of four.
template <int C>
struct SvmCols {
    static constexpr int M = C * (C - 1) / 2;
    static constexpr int NG = (M + 3) / 4;
    static constexpr int ST = 4 * NG + 1;  // exchange row (doubles): odd, so the rows' banks differ
    // pixels per exchange: a whole tile where its rows are short
    static constexpr int XP = NG <= 3 ? SVM_TILE : 16;
    static constexpr int WST = 4 * NG * 16;  // doubles of weights per k-step
};

// LDS traffic of one wavefront, in order.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// NL: 16-byte loads per lane and item, of up to 16 NL bands (1, 2, 4 or 8).
template <int C, bool PC1, int NL>
__global__ void __launch_bounds__(SVM_THREADS, C <= 4 ? 3 : C <= 6 ? 2 : 1)
svm_prob_kernel(const float* __restrict__ cube, int64_t npix, int bands,
                const double* __restrict__ w, const double* __restrict__ bias,
                const double* __restrict__ A, const double* __restrict__ B,
                float* __restrict__ out, const double* __restrict__ mean,
                const double* __restrict__ vec, float* __restrict__ band,
                double* __restrict__ ws, double* __restrict__ pairs) {
    using Cols = SvmCols<C>;
    constexpr int M = Cols::M, NG = Cols::NG, ST = Cols::ST, XP = Cols::XP;
    constexpr int G = SVM_TILE / 16;
    constexpr int MAXP = NL * 4;  // pieces per pixel of an item
    // weights[(4 s + e) / 2][group][k][n][e % 2]: lane (k, n) of matrix steps e
    // and e + 1 reads 16 bytes
    __shared__ __attribute__((aligned(16))) double wl[NL * Cols::WST];
    // an item's pieces, a row of MAXP per pixel and one of padding (bank
    // spread); after the tile's last item, its sums
    union Buf {
        float4 x[16 * (MAXP + 1)];
        double part[SVM_TILE / 16][64];
        double sum[XP * ST];
    };
    __shared__ __attribute__((aligned(16))) Buf buf[SVM_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int np = (bands + 3) >> 2;               // pieces per pixel
    const int nchunk = (np + MAXP - 1) / MAXP;     // items per 16 pixels, stagings of weights
    const int64_t tile0 = ((int64_t)blockIdx.x * (SVM_THREADS / 64) + wv) * SVM_TILE;  // first pixel

    // Item (group, chunk) of the tile: a load takes RPL pixels, MAXP lanes each
    // (lanes past the row's pieces load its last one and do not store it).
    constexpr int RPL = 64 / MAXP;
    const int lrow = lane / MAXP, lpc = lane % MAXP;
    const uint32_t b4 = (uint32_t)bands * 4u;
    float4 v[NL];
    auto load_item = [&](int g, int chunk) {
        // pixels past the cube repeat the last one
        const int64_t p0 = min(tile0 + 16 * g, npix - 1);
        const char* src = (const char*)(cube + p0 * (int64_t)bands);
        const uint32_t last = (uint32_t)min((int64_t)15, npix - 1 - p0);
        const int p = lpc + chunk * MAXP;
        const uint32_t po = (uint32_t)(p < np - 1 ? 4 * p : bands - 4) * 4u;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            v[i] = load4(src + (__umul24(min((uint32_t)(RPL * i + lrow), last), b4) + po));
    };
    // Weights of a chunk: fetched into registers, then stored to LDS.  Thread
    // tid takes column tid % (4 NG) of band slots SPT j + tid / (4 NG); the
    // last piece of a pixel starts at bands - 4 and has weight 0 for the bands
    // that it repeats, as have slots and columns past the end.
    constexpr int SPT = SVM_THREADS / (4 * NG), NSLOT = MAXP * 4;
    constexpr int NW = (NSLOT + SPT - 1) / SPT;
    const int wcol = tid % (4 * NG), wslot = tid / (4 * NG);
    const double* wsrc = w + (wcol < M ? wcol * bands : 0);
    double wr[NW];
    auto fetch_weights = [&](int chunk) {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const int slot = wslot + SPT * j + chunk * NSLOT, piece = slot >> 2;
            const int b = piece < np - 1 ? slot : bands - 4 + (slot & 3);
            const bool used = wcol < M && piece < np && b >= 4 * piece;
            const double x = wsrc[used ? b : 0];
            wr[j] = used ? x : 0.0;
        }
    };
    // (average, eigenvector entry) of the chunk's band slots, one a thread (PC1)
    typedef double d2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) d2 pl[PC1 ? NSLOT : 1];
    d2 pr = {0.0, 0.0};
    auto fetch_piece = [&](int chunk) {
        if constexpr (PC1) {
            const int slot = (tid & (NSLOT - 1)) + chunk * NSLOT, piece = slot >> 2;
            const int b = piece < np - 1 ? slot : bands - 4 + (slot & 3);
            const bool used = piece < np && b >= 4 * piece;
            const d2 x = {mean[used ? b : 0], vec[used ? b : 0]};
            pr = used ? x : d2{0.0, 0.0};
        }
    };
    auto store_weights = [&]() {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const int slot = wslot + SPT * j;
            const int s = slot >> 4, k = (slot >> 2) & 3, e = slot & 3;
            if (NSLOT % SPT == 0 || slot < NSLOT)
                wl[s * Cols::WST + (((e >> 1) * NG + (wcol >> 2)) * 16 + k * 4 + (wcol & 3)) * 2 + (e & 1)] = wr[j];
        }
        if (PC1 && tid < NSLOT) pl[tid] = pr;
    };
    load_item(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    fetch_weights(0);
    fetch_piece(0);
    store_weights();
    __syncthreads();

    char* xb = (char*)buf[wv].x;
    const double* wk = wl + ((lane >> 4) * 4 + (lane & 3)) * 2;
    double acc[G][NG];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int n = 0; n < NG; ++n) acc[g][n] = 0.0;
    double pj[G] = {};  // projection: pixel 16 g + lane % 16, pieces lane / 16, + 4, ...
    int chunk = 0;
    do {
        const int pc = min(MAXP, np - chunk * MAXP);
        const int ns = (pc + 3) >> 2;
        char* xw = xb + (lrow * (MAXP + 1) + lpc) * 16;
        const char* xr = xb + ((lane & 15) * (MAXP + 1) + (lane >> 4)) * 16;
        // slots past the row's pieces hold 0 (their weights are 0, but 0 times
        // an infinity is not)
        auto zero_slots = [&]() {
            if (lpc >= pc) {
#pragma unroll
                for (int i = 0; i < NL; ++i)
                    *(float4*)(xw + i * RPL * (MAXP + 1) * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        };
        zero_slots();
        // bands that the last piece repeats: 0 as well
        const int rep = lpc + chunk * MAXP == np - 1 ? 4 * np - bands : 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            wave_lds_sync();
            if (bands & 3) {
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    v[i].x = rep > 0 ? 0.f : v[i].x;
                    v[i].y = rep > 1 ? 0.f : v[i].y;
                    v[i].z = rep > 2 ? 0.f : v[i].z;
                }
            }
            if (lpc < pc) {
#pragma unroll
                for (int i = 0; i < NL; ++i) *(float4*)(xw + i * RPL * (MAXP + 1) * 16) = v[i];
            }
            wave_lds_sync();
            // the next item's loads
            if (g + 1 < G) load_item(g + 1, chunk);
            else if (chunk + 1 < nchunk) load_item(0, chunk + 1);
            __builtin_amdgcn_sched_barrier(0);
            for (int s = 0; s < ns; ++s) {
                const float4 x = *(const float4*)(xr + s * 64);
                const double xd[4] = {(double)x.x, (double)x.y, (double)x.z, (double)x.w};
                const double* wp = wk + s * Cols::WST;
                if constexpr (PC1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const d2 me = pl[16 * s + 4 * (lane >> 4) + e];
                        pj[g] = fma(xd[e] - me.x, me.y, pj[g]);
                    }
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    d2 wt[NG];
#pragma unroll
                    for (int n = 0; n < NG; ++n)
                        wt[n] = *(const d2*)(wp + (h * NG + n) * 32);
#pragma unroll
                    for (int n = 0; n < NG; ++n) 
                        acc[g][n] = __builtin_amdgcn_mfma_f64_4x4x4f64(xd[2 * h], wt[n].x, acc[g][n], 0, 0, 0);
#pragma unroll
                    for (int n = 0; n < NG; ++n) 
                        acc[g][n] = __builtin_amdgcn_mfma_f64_4x4x4f64(xd[2 * h + 1], wt[n].y, acc[g][n], 0, 0, 0);
                }
            }
        }
        if (++chunk < nchunk) {
            fetch_weights(chunk);
            fetch_piece(chunk);
            __syncthreads();
            store_weights();
            __syncthreads();
        }
    } while (chunk < nchunk);

    // sums to one lane per pixel: lane l of group g holds pixel
    // 16 g + 4 ((l / 4) % 4) + l / 16, column 4 n + l % 4
    double f[M];
    double* xr = buf[wv].sum;
    const int op = 4 * ((lane >> 2) & 3) + (lane >> 4), oc = lane & 3;
    wave_lds_sync();
    if constexpr (XP == SVM_TILE) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int n = 0; n < NG; ++n) xr[(16 * g + op) * ST + 4 * n + oc] = acc[g][n];
        wave_lds_sync();
#pragma unroll
        for (int m = 0; m < M; ++m) f[m] = xr[lane * ST + m];
    } else {
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int n = 0; n < NG; ++n) xr[op * ST + 4 * n + oc] = acc[g][n];
            wave_lds_sync();
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const double y = xr[(lane & 15) * ST + m];
                f[m] = g == 0 || lane >> 4 == g ? y : f[m];
            }
            wave_lds_sync();
        }
    }
    const int64_t pix = tile0 + lane;
    const bool in = pix < npix;
    if constexpr (PC1) {
        wave_lds_sync();
#pragma unroll
        for (int g = 0; g < G; ++g) buf[wv].part[g][lane] = pj[g];
        wave_lds_sync();
        double p = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) p += buf[wv].part[lane >> 4][16 * k + (lane & 15)];
        if (ws) {
            if (in) ws[pix] = p;
            __syncthreads();  // the buffers are free
            svm_publish_minmax<SVM_THREADS>(in ? p : __builtin_inf(), in ? p : -__builtin_inf(),
                                            pairs, buf[0].sum);
        } else if (in) {
            band[pix] = (float)p;
        }
    }
    if (in) svm_couple<C>(f, bias, A, B, out + pix * C);
}

// Fewer than four bands: one lane per pixel.
template <int C, bool PC1>
__global__ void __launch_bounds__(SVM_THREADS)
svm_prob_few_kernel(const float* __restrict__ cube, int64_t npix, int bands,
                    const double* __restrict__ w, const double* __restrict__ bias,
                    const double* __restrict__ A, const double* __restrict__ B,
                    float* __restrict__ out, const double* __restrict__ mean,
                    const double* __restrict__ vec, float* __restrict__ band,
                    double* __restrict__ ws, double* __restrict__ pairs) {
    constexpr int M = C * (C - 1) / 2;
    const int64_t nthreads = (int64_t)gridDim.x * SVM_THREADS;
    double lo = __builtin_inf(), hi = -__builtin_inf();
    for (int64_t pix = (int64_t)blockIdx.x * SVM_THREADS + threadIdx.x; pix < npix; pix += nthreads) {
        const float* row = cube + pix * (int64_t)bands;
        double f[M], pj = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m) f[m] = 0.0;
        for (int b = 0; b < bands; ++b) {
            const double x = (double)row[b];
#pragma unroll
            for (int m = 0; m < M; ++m) f[m] = fma(w[(int64_t)m * bands + b], x, f[m]);
            if constexpr (PC1) pj = fma(x - mean[b], vec[b], pj);
        }
        if constexpr (PC1) {
            if (ws) {
                ws[pix] = pj;
                lo = fmin(lo, pj);
                hi = fmax(hi, pj);
            } else {
                band[pix] = (float)pj;
            }
        }
        svm_couple<C>(f, bias, A, B, out + pix * C);
    }
    if constexpr (PC1) {
        __shared__ double lds[2 * SVM_THREADS / 64];
        if (ws) svm_publish_minmax<SVM_THREADS>(lo, hi, pairs, lds);
    }
}

struct SvmArgs {
    const float* cube;
    int64_t npix;
    int bands;
    const double *w, *bias, *A, *B, *mean, *vec;
    float *out, *band;
    double *ws, *pairs;
};

template <int C, bool PC1>
int launch_c(const SvmArgs& a, void* stream, int* nblocks) {
    const hipStream_t st = (hipStream_t)stream;
    const unsigned blocks = (unsigned)((a.npix + SVM_THREADS - 1) / SVM_THREADS);
    if (a.bands < 4)
        hipLaunchKernelGGL((svm_prob_few_kernel<C, PC1>), dim3(blocks), dim3(SVM_THREADS), 0, st,
                           a.cube, a.npix, a.bands, a.w, a.bias, a.A, a.B, a.out, a.mean, a.vec,
                           a.band, a.ws, a.pairs);
    else {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(SVM_THREADS), 0, st, a.cube, a.npix, a.bands, a.w,
                               a.bias, a.A, a.B, a.out, a.mean, a.vec, a.band, a.ws, a.pairs);
        };
        const int np = (a.bands + 3) / 4;
        // The least NL whose item holds the pixel's pieces: a lane past them loads
        // and stores nothing of use (us a call, 1000 x 1000, fused, two classes, NL 1
        // and 4: 16 bands 29.7 and 34; four classes 43.8 and 53).  Past 128 bands,
        // items of 64 where the last one of 128 would be half empty and rows start
        // at full cache lines (us, 380 x 480, four classes, NL 4 and 8: 160 bands
        // fused 31.1 and 34.7, 192 bands 33.8 and 37.7); where they do not, an item's
        // end cuts a line (1000 x 1000 x 132, two classes: 124 in halves, 102 whole).
        const bool halves = np > 32 && a.bands % 32 == 0 && (np - 1) % 32 < 16;
        if (np <= 4) launch(svm_prob_kernel<C, PC1, 1>);
        else if (np <= 8) launch(svm_prob_kernel<C, PC1, 2>);
        else if (np <= 16 || halves) launch(svm_prob_kernel<C, PC1, 4>);
        else launch(svm_prob_kernel<C, PC1, 8>);
    }
    if (nblocks) *nblocks = (int)blocks;
    return (int)hipGetLastError();
}

template <bool PC1>
int launch_classes(int classes, const SvmArgs& a, void* stream, int* nblocks) {
    switch (classes) {
        case 2: return launch_c<2, PC1>(a, stream, nblocks);
        case 3: return launch_c<3, PC1>(a, stream, nblocks);
        case 4: return launch_c<4, PC1>(a, stream, nblocks);
        case 5: return launch_c<5, PC1>(a, stream, nblocks);
        case 6: return launch_c<6, PC1>(a, stream, nblocks);
        case 7: return launch_c<7, PC1>(a, stream, nblocks);
        case 8: return launch_c<8, PC1>(a, stream, nblocks);
        default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace

int launch_svm(const float* cube, int64_t npix, int bands, int classes, const double* w,
               const double* bias, const double* A, const double* B, float* out, void* stream) {
    const SvmArgs a{cube, npix, bands, w, bias, A, B, nullptr, nullptr, out, nullptr, nullptr, nullptr};
    return launch_classes<false>(classes, a, stream, nullptr);
}

int svm_pixels_per_block() { return SVM_THREADS; }

int launch_svm_pc1(const float* cube, int64_t npix, int bands, int classes, const double* w,
                   const double* bias, const double* A, const double* B, const double* mean,
                   const double* vec, float* out, float* band, double* ws, double* pairs,
                   int* nblocks, void* stream) {
    const SvmArgs a{cube, npix, bands, w, bias, A, B, mean, vec, out, band, ws, pairs};
    return launch_classes<true>(classes, a, stream, nblocks);
}

}  // namespace knnf
