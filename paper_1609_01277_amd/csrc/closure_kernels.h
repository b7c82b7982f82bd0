// Kernels of the learned closure: box filter, channel statistics, standardise,
// BF16-MFMA implicit-GEMM 3x3x3 periodic convolution (forward, backward-data,
// backward-weight), bias gradient, MSE, Adam, weight packing, guard.
//
// Activation layout: channel-last [batch][point][channel] (point = (z*n + y)*n + x),
// channel count padded to a multiple of 8 so 8 consecutive channels are one
// 16-byte load.  The contraction index of a convolution is kk = tap*Cpad + c with
// tap = (dz+1)*9 + (dy+1)*3 + (dx+1).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace sbli {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int kNetLayers = 3;

__device__ __forceinline__ float gelu_f(float v) { return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float v) {
    return 0.5f * (1.0f + erff(v * 0.70710678118654752f)) + v * 0.39894228040143268f * expf(-0.5f * v * v);
}

__device__ __forceinline__ int wrapn(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// ---------------------------------------------------------------------------
// Box filter: separable centred trapezoid of width ratio*h (weights 1/(2 ratio)
// at +-ratio/2, 1/ratio in between), sampled at every ratio-th fine point.
// One thread per coarse output point and field.  With subtract != 0 the result
// is F(fine) - coarse (in place), e.g. F R_f - R_c for a closure target.
template <typename Tin>
__global__ void __launch_bounds__(256) box_filter_kernel(const Tin* __restrict__ fine, int nf, int nfields, int ratio,
                                                         float* __restrict__ coarse, int subtract) {
    const int nc = nf / ratio;
    const int64_t Pc = (int64_t)nc * nc * nc;
    const int64_t Pf = (int64_t)nf * nf * nf;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= Pc * nfields) return;
    const int f = (int)(id / Pc);
    const int64_t pc = id % Pc;
    const int xc = (int)(pc % nc), yc = (int)((pc / nc) % nc), zc = (int)(pc / ((int64_t)nc * nc));
    const int h = ratio / 2;
    const double wi = 1.0 / ratio, we = 0.5 / ratio;
    const Tin* src = fine + (int64_t)f * Pf;
    double acc = 0.0;
    for (int dz = -h; dz <= h; ++dz) {
        const double wz = (dz == -h || dz == h) ? we : wi;
        const int z = wrapn(zc * ratio + dz, nf);
        double accy = 0.0;
        for (int dy = -h; dy <= h; ++dy) {
            const double wy = (dy == -h || dy == h) ? we : wi;
            const int y = wrapn(yc * ratio + dy, nf);
            const Tin* row = src + ((int64_t)z * nf + y) * nf;
            double accx = 0.0;
            for (int dx = -h; dx <= h; ++dx) {
                const double wx = (dx == -h || dx == h) ? we : wi;
                accx += wx * (double)row[wrapn(xc * ratio + dx, nf)];
            }
            accy += wy * accx;
        }
        acc += wz * accy;
    }
    const int64_t o = (int64_t)f * Pc + pc;
    coarse[o] = subtract ? (float)(acc - (double)coarse[o]) : (float)acc;
}

// The same filter for ratio 2, 4 and 8 on 16-byte aligned rows.  The filter reads
// every fine value about once (1.25^2 times with ratio 4's shared end rows), so its
// time should be that of one pass over the fine fields; one thread per output point
// reading its (ratio + 1)^3 values one by one took 316 us for five 256^3 FP64 fields
// (671 MB), most of it in strided loads.  Here a lane loads the `ratio` consecutive
// values from its own point on (16-byte loads, a wavefront covers one contiguous run
// of a row) and takes the ratio/2 values to its left from the lane below; a thread
// marches zper output planes, and the z-plane two outputs share is reduced once.  The rows
// of one fine plane are requested together (three at a time for ratio 8), the planes one
// after the other: with several planes unrolled the registers leave two wavefronts a SIMD
// (ratio 4, FP64: 223 VGPRs, 171 us; 80 now) or spill (ratio 8).  133 us at 256^3, 5.0 TB/s
// (reads alone reach 5.9); 240^3 by 8: 264 -> 164 us; 200^3 by 2: 146 -> 90; 512^3 by 8:
// 3,859 -> 964.  The sums run in the order of box_filter_kernel, so the results are the
// same bits.
constexpr int kFilterZ = 4;      // output planes of a workgroup at most: 4 ratio + 1 fine planes
constexpr int kFilterWaves = 4;  // output rows of a workgroup
template <typename Tin, int RATIO>
__global__ void __launch_bounds__(64 * kFilterWaves)
    box_filter_rows_kernel(const Tin* __restrict__ fine, int nf, float* __restrict__ coarse, int subtract, int zper) {
    constexpr int H = RATIO / 2;
    constexpr int kRows = RATIO == 8 ? 3 : RATIO + 1;   // rows requested together
    constexpr int VL = 16 / (int)sizeof(Tin) < RATIO ? 16 / (int)sizeof(Tin) : RATIO;   // values of one load
    typedef Tin Vec __attribute__((ext_vector_type(VL)));
    const int nc = nf / RATIO;
    const int64_t Pc = (int64_t)nc * nc * nc, Pf = (int64_t)nf * nf * nf;
    const int lane = threadIdx.x & 63;
    const int xc = blockIdx.x * 64 + lane;
    const int yc = blockIdx.y * kFilterWaves + (threadIdx.x >> 6);
    const int nzb = (nc + zper - 1) / zper;
    const int f = blockIdx.z / nzb, zc0 = (blockIdx.z % nzb) * zper;
    if (yc >= nc) return;                              // a whole wavefront
    const int xl = xc < nc ? xc : nc - 1;              // lanes beyond the row repeat its last point
    const double wi = 1.0 / RATIO, we = 0.5 / RATIO;
    const Tin* src = fine + (int64_t)f * Pf;
    // x sum of fine row `row` at this lane's output point
    auto xsum = [&](const Tin* row) {
        Tin v[RATIO];
#pragma unroll
        for (int k = 0; k < RATIO; k += VL) {
            const Vec t = *(const Vec*)(row + xl * RATIO + k);
#pragma unroll
            for (int e = 0; e < VL; ++e) v[k + e] = t[e];
        }
        Tin left[H];
#pragma unroll
        for (int k = 0; k < H; ++k) left[k] = __shfl_up(v[RATIO - H + k], 1);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < H; ++k) left[k] = row[wrapn(xl * RATIO - H + k, nf)];
        }
        double acc = 0.0;
#pragma unroll
        for (int dx = -H; dx <= H; ++dx) {
            const double wx = (dx == -H || dx == H) ? we : wi;
            acc += wx * (double)(dx < 0 ? left[dx + H < 0 ? 0 : (dx + H < H ? dx + H : 0)] : v[dx < 0 ? 0 : dx]);
        }
        return acc;
    };
    // y sum of the x sums at fine plane z
    auto ysum = [&](int z) {
        const Tin* pz = src + (int64_t)wrapn(z, nf) * nf * nf;
        double acc = 0.0;
#pragma unroll kRows
        for (int dy = -H; dy <= H; ++dy) {
            const double wy = (dy == -H || dy == H) ? we : wi;
            acc += wy * xsum(pz + (int64_t)wrapn(yc * RATIO + dy, nf) * nf);
        }
        return acc;
    };
    const int zc1 = min(zc0 + zper, nc);
    double shared_plane = ysum(zc0 * RATIO - H);       // the plane this output shares with the one below
    for (int zc = zc0; zc < zc1; ++zc) {
        double acc = 0.0;
        acc += we * shared_plane;
#pragma unroll 1
        for (int dz = -H + 1; dz <= H; ++dz) {
            const double s = ysum(zc * RATIO + dz);
            acc += (dz == H ? we : wi) * s;
            if (dz == H) shared_plane = s;
        }
        if (xc < nc) {
            const int64_t o = (int64_t)f * Pc + ((int64_t)zc * nc + yc) * nc + xc;
            coarse[o] = subtract ? (float)(acc - (double)coarse[o]) : (float)acc;
        }
    }
}

// ---------------------------------------------------------------------------
// Per-channel mean, standard deviation (population statistics, FP64 sums) and
// largest magnitude of `count` planar [5][P] FP32 arrays.  One block per channel.
__global__ void __launch_bounds__(256) channel_stats_kernel(const float* __restrict__ data, int count, int64_t P,
                                                            float* __restrict__ mean_std /* [5] mean, [5] std */,
                                                            float* __restrict__ maxabs /* [5] */) {
    const int c = blockIdx.x;
    double s = 0.0, s2 = 0.0;
    float mx = 0.0f;
    for (int b = 0; b < count; ++b) {
        const float* src = data + ((int64_t)b * 5 + c) * P;
        for (int64_t i = threadIdx.x; i < P; i += blockDim.x) {
            const double v = src[i];
            s += v;
            s2 += v * v;
            mx = fmaxf(mx, fabsf(src[i]));
        }
    }
    __shared__ double ss[256], ss2[256];
    __shared__ float sm[256];
    ss[threadIdx.x] = s;
    ss2[threadIdx.x] = s2;
    sm[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            ss[threadIdx.x] += ss[threadIdx.x + w];
            ss2[threadIdx.x] += ss2[threadIdx.x + w];
            sm[threadIdx.x] = fmaxf(sm[threadIdx.x], sm[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double N = (double)count * (double)P;
        const double m = ss[0] / N;
        const double var = ss2[0] / N - m * m;
        mean_std[c] = (float)m;
        mean_std[5 + c] = (float)sqrt(var > 0.0 ? var : 0.0);
        maxabs[c] = sm[0];
    }
}

// Planar FP32 [B][5][P] -> standardised channel-last BF16 [B][P][8] (channels 5..7 zero).
__global__ void __launch_bounds__(256) standardize_kernel(const float* __restrict__ q, int64_t P, int B,
                                                          const float* __restrict__ mean_std,
                                                          __bf16* __restrict__ x) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)B * P) return;
    const int64_t b = id / P, p = id % P;
    bf16x8 v;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float f = 0.0f;
        if (c < 5) f = (q[(b * 5 + c) * P + p] - mean_std[c]) / mean_std[5 + c];
        v[c] = (__bf16)f;
    }
    *(bf16x8*)(x + id * 8) = v;
}

// Network output y [B][P][8] (standardised) -> closure term planar [B][5][P].
__global__ void __launch_bounds__(256) destandardize_kernel(const float* __restrict__ y, int64_t P, int B,
                                                            const float* __restrict__ mean_std,
                                                            float* __restrict__ out) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)B * P) return;
    const int64_t b = id / P, p = id % P;
#pragma unroll
    for (int c = 0; c < 5; ++c) out[(b * 5 + c) * P + p] = y[id * 8 + c] * mean_std[5 + c] + mean_std[c];
}

// Box mean of every (sample, field) plane of a planar [B][5][P] array, removed
// in place: the closure term then adds nothing to the box totals of mass,
// momentum and energy, as the exact closure term does (both residuals are
// conservative and the filter keeps totals).  Three steps, each in a fixed
// order, so the result is deterministic: FP64 partial sums of kBoxMeanChunk
// points per workgroup, one mean per (sample, field), the subtraction.
constexpr int kBoxMeanChunk = 4096;
__global__ void __launch_bounds__(256) box_mean_partial_kernel(const float* __restrict__ a, int64_t P, int nchunks,
                                                               double* __restrict__ part) {
    // one workgroup per (sample * 5 + field, chunk), chunks fastest
    const int chunk = (int)(blockIdx.x % (unsigned)nchunks);
    const int64_t bf = blockIdx.x / (unsigned)nchunks;
    const float* src = a + bf * P;
    const int64_t lo = (int64_t)chunk * kBoxMeanChunk;
    const int64_t hi = lo + kBoxMeanChunk < P ? lo + kBoxMeanChunk : P;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) s += (double)src[i];
    __shared__ double ss[256];
    ss[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) ss[threadIdx.x] += ss[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[bf * nchunks + chunk] = ss[0];
}
// one thread per (sample, field): the partials in chunk order
__global__ void __launch_bounds__(64) box_mean_final_kernel(const double* __restrict__ part, int nchunks, int nbf,
                                                            int64_t P, float* __restrict__ mean) {
    const int bf = blockIdx.x * blockDim.x + threadIdx.x;
    if (bf >= nbf) return;
    double s = 0.0;
    for (int k = 0; k < nchunks; ++k) s += part[(int64_t)bf * nchunks + k];
    mean[bf] = (float)(s / (double)P);
}
__global__ void __launch_bounds__(256) box_mean_subtract_kernel(float* __restrict__ a, int64_t P, int nbf,
                                                                const float* __restrict__ mean) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)nbf * P) return;
    a[id] -= mean[id / P];
}

// ---------------------------------------------------------------------------
// Implicit-GEMM convolution on MFMA (v_mfma_f32_32x32x16_bf16).
//   out[b][p][o] = sum_kk W[o][kk] * in[b][p + off(tap(kk))][c(kk)]
// A wave computes 2 tiles of 32 points x 32 output channels.  A operand
// (points x 16 kk): each lane reads 8 consecutive channels of one tap at one
// point (16 bytes); B operand (16 kk x 32 outputs): 8 consecutive kk of one
// output channel (16 bytes) from the packed weights Wp[32][Kpad] or, FRAG, from weights
// packed in operand order.
// Epilogues:
//   kEpiGelu   : v = acc + bias; pre[..][o] = v (FP32, 32 ch); act[..][o] = bf16(gelu v)
//   kEpiLinear : v = acc + bias; y[..][o] = v (FP32, ostride ch) for o < ocount
//   kEpiDGelu  : v = acc * gelu'(pre[..][o]); act[..][o] = bf16(v) (32 ch)
//   kEpiData   : out[..][o] = acc (FP32, 32 ch)
enum { kEpiGelu = 0, kEpiLinear = 1, kEpiDGelu = 2, kEpiData = 3 };

// The input is staged in LDS (grids with n % 32 == 0).  A workgroup owns 32
// x-points x 8 y-rows of one z-plane of one sample (256 points; wave w takes
// rows 2w and 2w + 1 as its two 32-point M tiles).  The
// 34 x 10 x 3 input points it reads (periodic halo of one point) are loaded
// once into LDS and every one of the 27 taps reads its A operands from there,
// instead of from global memory 27 times.  LDS point stride: cpad channels; for
// cpad = 32 (64 bytes) the four 16-byte groups of a point are rotated by its x (group ^
// (hx / 2) % 4), so that eight lanes' reads fall in distinct banks, and two workgroups fit
// a CU (65 KB; with 80-byte points one did).
// What bounds it: with weights by rows (Wp[32][Kpad]) a step's load touched 32 lines, and
// L1 was busy 78 % of the time, MFMA 17 %; in operand order it is one contiguous KB.  Then
// the chain of a step: its weights' and points' latency, hidden by requests 6 steps and 1
// step ahead.  4 x 64^3 points, 32 -> 32 channels with GELU: 145 -> 109 us (201 MB of
// outputs take 44, the MFMAs 27), 32 -> 5: 100 -> 69, backward data 32 -> 32: 147 -> 125;
// 8 -> 32: 62 -> 53.  The 8-channel forms have 14 steps and more workgroups a CU; there
// requests ahead cost registers (backward data 81 -> 103 us) and are left out, and the
// backward-data form with weights by rows, which holds its 32 pre-activations, takes two
// wavefronts a SIMD (with three it spills: 57 -> 62 us).
constexpr int kConvTx = 32, kConvTy = 8;
constexpr int kConvHx = kConvTx + 2, kConvHy = kConvTy + 2;

template <int EPI, int CPAD, bool FRAG>
__global__ void __launch_bounds__(256, CPAD == 8 && (FRAG || EPI != kEpiDGelu) ? 3 : 2) conv_mfma_lds_kernel(const __bf16* __restrict__ in, const __bf16* __restrict__ Wp,
                                                            int Kpad, const float* __restrict__ bias, int n,
                                                            float* __restrict__ fout, __bf16* __restrict__ bout,
                                                            const float* __restrict__ pre_in, int ocount, int ostride) {
    __shared__ __attribute__((aligned(16))) __bf16 sx[3 * kConvHy * kConvHx * CPAD];
    // element of channel group g (8 channels) of the point (hx, row hr = hz * kConvHy + hy)
    auto at = [](int hr, int hx, int g) {
        return (hr * kConvHx + hx) * CPAD + (CPAD == 32 ? (g ^ (hx >> 1 & 3)) * 8 : 0);
    };
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int row = lane & 31, half = lane >> 5;
    const int64_t P = (int64_t)n * n * n;
    // tile -> (sample, z, y0, x0)
    const int tx = n / kConvTx, ty = n / kConvTy;
    int t = blockIdx.x;
    const int x0 = (t % tx) * kConvTx;
    t /= tx;
    const int y0 = (t % ty) * kConvTy;
    t /= ty;
    const int z = t % n;
    const int64_t b = t / n;
    const __bf16* inb = in + b * P * CPAD;
    // stage the halo box: 3 x 10 rows of 34 points, CPAD / 8 16-byte loads each.  A
    // thread issues all of its loads before its first LDS store, so their latencies
    // overlap instead of adding up.  Row by row the 32 points of the tile (for CPAD = 32 a
    // row is the same for a whole wave, its address scalar), then the rows' two end points.
    constexpr int G = CPAD / 8, ROWS = 3 * kConvHy;
    constexpr int NM = ROWS * kConvTx * G, NE = ROWS * 2 * G;
    constexpr int IT = (NM + 255) / 256;
    static_assert(NE <= 256, "one end load per thread");
    auto row_base = [&](int hr) {                         // the row's first point
        const int hz = hr / kConvHy, hy = hr % kConvHy;
        return inb + ((int64_t)wrapn(z + hz - 1, n) * n + wrapn(y0 + hy - 1, n)) * n * CPAD;
    };
    auto row_of = [](int i) {
        const int r = i / (kConvTx * G);
        return kConvTx * G >= 64 ? __builtin_amdgcn_readfirstlane(r) : r;
    };
    bf16x8 sv[IT], se;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < NM) sv[k] = *(const bf16x8*)(row_base(row_of(i)) + x0 * CPAD + i % (kConvTx * G) * 8);
    }
    const int er = threadIdx.x / (2 * G), ex = threadIdx.x / G % 2 ? kConvHx - 1 : 0;
    if (threadIdx.x < NE) se = *(const bf16x8*)(row_base(er) + wrapn(x0 + ex - 1, n) * CPAD + threadIdx.x % G * 8);
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < NM) *(bf16x8*)(&sx[at(row_of(i), i / G % kConvTx + 1, i % G)]) = sv[k];
    }
    if (threadIdx.x < NE) *(bf16x8*)(&sx[at(er, ex, threadIdx.x % G)]) = se;
    const __bf16* wl = FRAG ? Wp + lane * 8 : Wp + (int64_t)row * Kpad + half * 8;
    constexpr int WS = FRAG ? 512 : 16;                   // elements from a step's operands to the next's
    constexpr int kAheadW = CPAD == 32 ? 6 : 0;
    bf16x8 wv[kAheadW + 1];
#pragma unroll
    for (int s = 0; s < kAheadW; ++s) wv[s] = *(const bf16x8*)(wl + s * WS);
    __syncthreads();
    floatx16 acc0 = {0}, acc1 = {0};
    const int ry0 = 2 * wave;                             // tile rows ry0, ry0 + 1 of the two M tiles
    // this lane's element in the box row ry0 (CPAD = 32: by dx and channel group), each tap a
    // constant from there.  (Elements, not pointers: a choice between two pointers loses that they
    // point to LDS, and its reads become flat loads, which cost the 8-channel forms a third of
    // their time.)
    const int lx8 = at(ry0, row, 0);
    int lx[3][2];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int c = 0; c < 2; ++c) lx[dx][c] = at(ry0, row + dx, 2 * c + half);
    constexpr int RS = kConvHx * CPAD;                    // from a box row to the next
    auto row_off = [](int t) { return ((t / 9) * kConvHy + (t / 3) % 3) * RS; };
    // The K loop runs over the packed width round_up(27 * CPAD, 16) (the value of
    // Kpad) and is unrolled completely, so every tap offset is a constant: a step
    // of 16 kk is one tap (channels c0 .. c0 + 15) for CPAD = 32, two taps (one
    // per half-wave) for CPAD = 8.
    constexpr int KP = (27 * CPAD + 15) / 16 * 16;
    // the backward-data epilogue's pre-activations are requested before the K
    // loop, so their latency is spent under the MFMAs
    float pre[2][16];
    if constexpr (EPI == kEpiDGelu) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int y = y0 + 2 * wave + tt;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int m = (j / 4) * 8 + half * 4 + (j & 3);
                const int64_t g = b * P + ((int64_t)z * n + y) * n + x0 + m;
                pre[tt][j] = pre_in[g * 32 + row];
            }
        }
    }
    // Operands are requested ahead, weights kAheadW steps (L2 latency), points one step (LDS).
    auto points = [&](int k0, bf16x8& a0, bf16x8& a1) {
        if (CPAD == 32 || k0 / CPAD + half < 27) {
            int a;
            if constexpr (CPAD == 32) {
                const int t = k0 / 32;
                a = lx[t % 3][k0 % 32 / 16] + row_off(t);
            } else {
                const int t = k0 / CPAD;
                a = lx8 + (half ? row_off(t + 1) + (t + 1) % 3 * CPAD : row_off(t) + t % 3 * CPAD);
            }
            a0 = *(const bf16x8*)&sx[a];
            a1 = *(const bf16x8*)&sx[a + RS];             // next row
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) { a0[j] = (__bf16)0.0f; a1[j] = (__bf16)0.0f; }
        }
    };
    if constexpr (CPAD == 32) {
        bf16x8 a0[2], a1[2];
        points(0, a0[0], a1[0]);
#pragma unroll
        for (int s = 0; s < KP / 16; ++s) {
            if (s + kAheadW < KP / 16) wv[(s + kAheadW) % (kAheadW + 1)] = *(const bf16x8*)(wl + (s + kAheadW) * WS);
            if (s + 1 < KP / 16) points(16 * (s + 1), a0[(s + 1) & 1], a1[(s + 1) & 1]);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[s & 1], wv[s % (kAheadW + 1)], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[s & 1], wv[s % (kAheadW + 1)], acc1, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int s = 0; s < KP / 16; ++s) {
            const bf16x8 w = *(const bf16x8*)(wl + s * WS);
            bf16x8 a0, a1;
            points(16 * s, a0, a1);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, w, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, w, acc1, 0, 0, 0);
        }
    }
    // D[m][o]: o = lane & 31, m = (j / 4) * 8 + (lane >> 5) * 4 + (j & 3); m = x within the row
    const int o = row;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        const floatx16 acc = tt == 0 ? acc0 : acc1;
        const int y = y0 + 2 * wave + tt;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int m = (j / 4) * 8 + half * 4 + (j & 3);
            const int64_t g = b * P + ((int64_t)z * n + y) * n + x0 + m;
            if (EPI == kEpiGelu) {
                const float v = acc[j] + bias[o];
                fout[g * 32 + o] = v;
                bout[g * 32 + o] = (__bf16)gelu_f(v);
            } else if (EPI == kEpiLinear) {
                if (o < ocount) fout[g * ostride + o] = acc[j] + bias[o];
            } else if (EPI == kEpiData) {
                fout[g * 32 + o] = acc[j];
            } else {
                bout[g * 32 + o] = (__bf16)(acc[j] * gelu_grad_f(pre[tt][j]));
            }
        }
    }
}

// Element-wise GELU backward: dx = bf16(g * gelu'(pre)), the arithmetic of the
// kEpiDGelu epilogue.
__global__ void __launch_bounds__(256) gelu_bwd_kernel(const float* __restrict__ g, const float* __restrict__ pre,
                                                       int64_t count, __bf16* __restrict__ dx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dx[i] = (__bf16)(g[i] * gelu_grad_f(pre[i]));
}

// ---------------------------------------------------------------------------
// Weight gradient on MFMA: dW[o][tap][c] = sum_p dout[p][o] * in[p + off(tap)][c]
//                                        = sum_p dout[p - off(tap)][o] * in[p][c].
// One of the two tensors is read at p (`a`, CA channels: the M side), the other at
// p + SIGN off(tap) (`b`, CB channels: the N side, a tile of 32 columns being one tap of
// 32 channels or four taps of 8).  a = dout, b = in, SIGN = 1, except for 8 output and 32
// input channels, where a = in, b = dout, SIGN = -1 leaves 7 tiles instead of 27 that are
// three quarters padding.  K runs over points, so both operands need 8 consecutive points
// of one channel in a lane, and the tensors are channel-last: ds_read_b64_tr_b16 makes
// that transpose on the way from LDS (16 lanes give the addresses of 4 rows of 16 values
// and get 4 points of one channel each), so a plane is staged as it lies in memory, once.
// The former kernel transposed in registers and wrote every tap's shifted copy to LDS
// for each block of 32 points: 218 us a call (64^3, batch 4, the three layers' mean), two
// thirds of it waiting.  This one: 44 us (83 us for 32 and 32 channels, 25 us with 8 on a side).
// A workgroup marches up a column of 32 x kWgradTy points in z.  LDS holds four planes of
// b with their halo (z - 1 .. z + 1 and the one being written) and two of a; the next
// planes are requested before the products of the present one: one barrier a plane.  Its
// bound is LDS: 4 reads of 4 cycles a product of 32 for one tile, 2.5 for four tiles.
// Results: per-workgroup partial sums part[wg][32][Kpad32] (FP32), rows the channels of a,
// columns tap * CB + channel of b.
constexpr int kWgradTy = 8;
constexpr int kWgradThreads = 512;
typedef short sbli_v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) sbli_v4s* sbli_lds_v4s;

// 8 consecutive points (rows `stride` elements apart) of one channel for the MFMA operand
// of this lane; p is this lane's address of the first 4 rows.
__device__ __forceinline__ bf16x8 read_points_tr(const __bf16* p, int stride) {
    const sbli_v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((sbli_lds_v4s)(p));
    const sbli_v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((sbli_lds_v4s)(p + 4 * stride));
    typedef short v8s __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (v8s)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int CA, int CB, int SIGN>
__global__ void __launch_bounds__(kWgradThreads, 2)
    conv_wgrad_kernel(const __bf16* __restrict__ a, const __bf16* __restrict__ b, int n, int64_t planes,
                      float* __restrict__ part) {
    constexpr int TX = 32, TY = kWgradTy, NT = kWgradThreads, NW = NT / 64;
    constexpr int HX = TX + 2, HY = TY + 2, HP = HX * HY;
    constexpr int LA = CA == 32 ? 40 : 8, LB = CB == 32 ? 40 : 8;   // LDS point strides (80 or 16 bytes)
    constexpr int TILES = CB == 32 ? 27 : 7, TPW = (TILES + NW - 1) / NW;
    constexpr int KP = TILES * 32;
    constexpr int NAC = TX * TY * CA / 8, NBC = HP * CB / 8;        // 16-byte pieces of a plane
    constexpr int ITA = (NAC + NT - 1) / NT, ITB = (NBC + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) __bf16 sa[2][TX * TY * LA];
    __shared__ __attribute__((aligned(16))) __bf16 sb[4][HP * LB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t P = (int64_t)n * n * n;
    const int ctx = n / TX, cty = n / TY;
    // this lane's address within 16 points: row (of 4) and first channel of its 8-byte piece;
    // lanes 0-15 / 16-31 serve columns 0-15 / 16-31, lanes 32-63 the upper 8 points
    const int r4 = (lane & 15) >> 2, c4 = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    const int row0 = (lane >> 5) * 8 + r4;
    const int laneA = row0 * LA + (CA == 32 ? c4 : c4 & 7);
    const bool a_valid = CA == 32 || (lane & 31) < 8;               // rows of a beyond its 8 channels are zero
    int laneB[TPW], dzB[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int tile = min(wave + NW * i, TILES - 1);
        const int tap = CB == 32 ? tile : min(4 * tile + c4 / 8, 26);   // the 28th tap's columns are never read back
        dzB[i] = SIGN * (tap / 9 - 1);
        laneB[i] = ((1 + SIGN * (tap / 3 % 3 - 1)) * HX + 1 + SIGN * (tap % 3 - 1) + row0) * LB +
                   (CB == 32 ? c4 : c4 & 7);
    }
    floatx16 acc[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.0f;
    const int64_t per = (planes + gridDim.x - 1) / gridDim.x;
    const int64_t u1 = min(((int64_t)blockIdx.x + 1) * per, planes);
    int64_t u = (int64_t)blockIdx.x * per;
    while (u < u1) {
        // planes z0 .. z1 - 1 of one column
        const int64_t colid = u / n;
        const int z0 = (int)(u % n);
        const int z1 = (int)min((int64_t)n, z0 + (u1 - u));
        u += z1 - z0;
        const int x0 = (int)(colid % ctx) * TX, y0 = (int)(colid / ctx % cty) * TY;
        const int64_t smp = colid / ctx / cty;
        const __bf16* as = a + smp * P * CA;
        const __bf16* bs = b + smp * P * CB;
        bf16x8 ra[ITA], rb[ITB];
        auto load_a = [&](int z) {
#pragma unroll
            for (int k = 0; k < ITA; ++k) {
                const int e = min(tid + NT * k, NAC - 1), pt = e / (CA / 8), g = e % (CA / 8);
                ra[k] = *(const bf16x8*)(as + (((int64_t)z * n + y0 + pt / TX) * n + x0 + pt % TX) * CA + g * 8);
            }
        };
        auto load_b = [&](int z) {
            const int64_t gz = (int64_t)wrapn(z, n) * n;
#pragma unroll
            for (int k = 0; k < ITB; ++k) {
                const int e = min(tid + NT * k, NBC - 1), pt = e / (CB / 8), g = e % (CB / 8);
                const int gy = wrapn(y0 + pt / HX - 1, n), gx = wrapn(x0 + pt % HX - 1, n);
                rb[k] = *(const bf16x8*)(bs + ((gz + gy) * n + gx) * CB + g * 8);
            }
        };
        auto store_a = [&](int buf) {
#pragma unroll
            for (int k = 0; k < ITA; ++k) {
                const int e = tid + NT * k;
                if (e < NAC) *(bf16x8*)(&sa[buf][e / (CA / 8) * LA + e % (CA / 8) * 8]) = ra[k];
            }
        };
        auto store_b = [&](int buf) {
#pragma unroll
            for (int k = 0; k < ITB; ++k) {
                const int e = tid + NT * k;
                if (e < NBC) *(bf16x8*)(&sb[buf][e / (CB / 8) * LB + e % (CB / 8) * 8]) = rb[k];
            }
        };
        __syncthreads();   // the previous column's products are done
        load_b(z0 - 1);
        store_b((z0 + 3) & 3);
        load_b(z0);
        store_b(z0 & 3);
        load_b(z0 + 1);
        load_a(z0);
        for (int z = z0; z < z1; ++z) {
            store_b((z + 1) & 3);
            store_a(z & 1);
            __syncthreads();
            if (z + 1 < z1) {
                load_b(z + 2);
                load_a(z + 1);
            }
            const __bf16* pa = &sa[z & 1][laneA];
            const __bf16* pb[TPW];
#pragma unroll
            for (int i = 0; i < TPW; ++i) pb[i] = &sb[(z + dzB[i]) & 3][laneB[i]];
#pragma unroll
            for (int y = 0; y < TY; ++y)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 av = read_points_tr(pa + (y * TX + ks * 16) * LA, LA);
                    if (CA == 8) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) av[j] = a_valid ? av[j] : (__bf16)0.0f;
                    }
#pragma unroll
                    for (int i = 0; i < TPW; ++i) {
                        if (wave + NW * i < TILES) {   // the same for a whole wavefront
                            const bf16x8 bv = read_points_tr(pb[i] + (y * HX + ks * 16) * LB, LB);
                            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[i], 0, 0, 0);
                        }
                    }
                }
        }
    }
    // D[m][kk]: kk = tile * 32 + (lane & 31), m = (j / 4) * 8 + (lane >> 5) * 4 + (j & 3)
    float* dst = part + (int64_t)blockIdx.x * 32 * KP;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int tile = wave + NW * i;
        if (tile >= TILES) continue;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int m = (j / 4) * 8 + (lane >> 5) * 4 + (j & 3);
            dst[(int64_t)m * KP + tile * 32 + (lane & 31)] = acc[i][j];
        }
    }
}

// Sums the per-workgroup partials in a fixed order and writes the gradient of
// a layer in the master layout dW[o][c][tap] (o < cout, c < cin).  Rows of a partial
// are output channels and its columns tap * cb + input channel, or (transposed) rows
// input channels and columns tap * cb + output channel.
__global__ void __launch_bounds__(256) wgrad_reduce_kernel(const float* __restrict__ part, int nwg, int Kpad32,
                                                           int cb, int cin, int cout, int transposed,
                                                           float* __restrict__ dW) {
    // one thread per (row, kk), kk fastest, so the partial rows
    // are read contiguously.  Four interleaved accumulators (partials w = 4i + j
    // into s_j) keep four loads in flight; they are combined in a fixed order,
    // so the result is deterministic.
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    const int kk = id % Kpad32;
    const int row = id / Kpad32;
    const int tap = kk / cb, ch = kk % cb;
    const int o = transposed ? ch : row, c = transposed ? row : ch;
    if (tap >= 27 || o >= cout || c >= cin) return;
    const float* p = part + (int64_t)row * Kpad32 + kk;
    const int64_t stride = (int64_t)32 * Kpad32;
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
    int w = 0;
    // unrolled so that many partials are in flight; each s_j still adds its
    // partials in order of w
#pragma unroll 8
    for (; w + 4 <= nwg; w += 4) {
        s0 += p[(w + 0) * stride];
        s1 += p[(w + 1) * stride];
        s2 += p[(w + 2) * stride];
        s3 += p[(w + 3) * stride];
    }
    for (; w < nwg; ++w) s0 += p[w * stride];
    dW[(o * cin + c) * 27 + tap] = (s0 + s1) + (s2 + s3);
}

// Bias gradient db[o] = sum_p dout[p][o], in two deterministic passes.
// Pass 1: workgroup w sums points [w * chunk, (w + 1) * chunk) into
// part[w][32]; each thread reads 8 channels of a point with one 16-byte load
// (opad / 8 threads per point, 256 / (opad / 8) point lanes), and the point
// lanes are combined in LDS in a fixed order.
constexpr int kBiasWg = 512;
__global__ void __launch_bounds__(256) bias_grad_kernel(const __bf16* __restrict__ dout, int opad, int64_t npts,
                                                        float* __restrict__ part) {
    const int groups = opad / 8;                     // 1 or 4
    const int cg = threadIdx.x % groups, pl = threadIdx.x / groups;
    const int lanes = 256 / groups;
    const int64_t chunk = (npts + gridDim.x - 1) / gridDim.x;
    const int64_t p0 = (int64_t)blockIdx.x * chunk;
    const int64_t p1 = p0 + chunk < npts ? p0 + chunk : npts;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t p = p0 + pl; p < p1; p += lanes) {
        const bf16x8 v = *(const bf16x8*)(dout + p * opad + cg * 8);
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] += (float)v[j];
    }
    __shared__ float ss[256][9];
#pragma unroll
    for (int j = 0; j < 8; ++j) ss[threadIdx.x][j] = s[j];
    __syncthreads();
    if ((int)threadIdx.x < opad) {
        const int c = threadIdx.x, g = c / 8, j = c % 8;
        float t = 0.0f;
        for (int l = 0; l < lanes; ++l) t += ss[l * groups + g][j];
        part[blockIdx.x * 32 + c] = t;
    }
}

// Pass 2: 256 threads = 32 channels x 8 slices; slice k sums partials
// w = k, k + 8, ...; the slices are combined in order.
__global__ void __launch_bounds__(256) bias_grad_final_kernel(const float* __restrict__ part, int nwg, int cout,
                                                              float* __restrict__ db) {
    const int o = threadIdx.x & 31, k = threadIdx.x >> 5;
    float s = 0.0f;
#pragma unroll 8
    for (int w = k; w < nwg; w += 8) s += part[w * 32 + o];   // in order of w
    __shared__ float ss[8][32];
    ss[k][o] = s;
    __syncthreads();
    if ((int)threadIdx.x < cout) {
        float t = 0.0f;
        for (int j = 0; j < 8; ++j) t += ss[j][threadIdx.x];
        db[threadIdx.x] = t;
    }
}

// MSE between the network output y [B][P][8] (5 used) and the standardised
// target (planar [B][5][P], standardised here): loss partial sums per block and
// the BF16 gradient dy = 2 (y - t) / (5 B P) into [B][P][8].
__global__ void __launch_bounds__(256) mse_grad_kernel(const float* __restrict__ y, const float* __restrict__ target,
                                                       int64_t P, int B, const float* __restrict__ mean_std,
                                                       __bf16* __restrict__ dy, double* __restrict__ loss_part) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double scale = 2.0 / (5.0 * (double)B * (double)P);
    double s = 0.0;
    if (id < (int64_t)B * P) {
        const int64_t b = id / P, p = id % P;
        bf16x8 g;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float gv = 0.0f;
            if (c < 5) {
                const float t = (target[(b * 5 + c) * P + p] - mean_std[c]) / mean_std[5 + c];
                const float d = y[id * 8 + c] - t;
                s += (double)d * d;
                gv = (float)(scale * d);
            }
            g[c] = (__bf16)gv;
        }
        *(bf16x8*)(dy + id * 8) = g;
    }
    __shared__ double ss[256];
    ss[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) ss[threadIdx.x] += ss[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = ss[0];
}

__global__ void __launch_bounds__(256) sum_doubles_kernel(const double* __restrict__ part, int n, double scale,
                                                          double* __restrict__ out) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
    __shared__ double ss[256];
    ss[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) ss[threadIdx.x] += ss[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = ss[0] * scale;
}

// Adam (Kingma & Ba) on a flat FP32 parameter vector; step t >= 1.
__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int n, float lr,
                                                   float beta1, float beta2, float eps, int t) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / (1.0f - powf(beta1, (float)t));
    const float vh = vi / (1.0f - powf(beta2, (float)t));
    p[i] -= lr * mh / (sqrtf(vh) + eps);
}

// Packs one layer's master weights W[o][c][tap] (FP32) into the MFMA layouts:
//   Wf[o][tap*cpad + c]  (32 x Kf, forward),  Wb[c][tap'*opad + o] (32 x Kb,
//   backward-data, tap' = 26 - tap mirrors the offset).  Padding entries are 0.
// frag: in the order of the MFMA operands instead, [kk / 16][kk / 8 % 2][row][kk % 8],
// 1 KB a step, which a wave loads as one contiguous piece.
__global__ void __launch_bounds__(256) pack_weights_kernel(const float* __restrict__ W, int cin, int cout, int cpad,
                                                           int opad, int Kf, int Kb, int frag, __bf16* __restrict__ Wf,
                                                           __bf16* __restrict__ Wb) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    auto at = [&](int row, int kk) { return (kk / 16 * 64 + kk / 8 % 2 * 32 + row) * 8 + kk % 8; };
    if (Wf != nullptr && id < 32 * Kf) {
        const int o = id / Kf, kk = id % Kf;
        const int tap = kk / cpad, c = kk % cpad;
        float v = 0.0f;
        if (o < cout && tap < 27 && c < cin) v = W[(o * cin + c) * 27 + tap];
        Wf[frag ? at(o, kk) : id] = (__bf16)v;
    }
    if (Wb != nullptr && id < 32 * Kb) {
        const int c = id / Kb, kk = id % Kb;
        const int tapm = kk / opad, o = kk % opad;
        float v = 0.0f;
        if (c < cin && tapm < 27 && o < cout) v = W[(o * cin + c) * 27 + (26 - tapm)];
        Wb[frag ? at(c, kk) : id] = (__bf16)v;
    }
}

// Closure guard: flag[0] = 1 if every closure value is finite and within
// +-limit[f] for its field, else 0; counters[0|1] count accepted / rejected.
// The check reads 5 P values, 5.2 MB at 64^3: the time is that of one pass of
// loads, so it wants many of them in flight on every CU.  A workgroup checks
// kGuardPer values; the last one to finish (a ticket counter) writes the verdict.
// At 64^3 one workgroup of 1,024 threads took 368 us, 320 workgroups of 4,096 values
// take about 8 us.
// state: workgroups done, and kGuardBad once one has seen a value out of bounds; 0 before
// the call and cleared by it.  It may be the word of `flag` itself, then cleared before.
constexpr int kGuardPer = 4096;   // divides P (a multiple of 32^3); at most 5 * 2^18 workgroups
constexpr unsigned kGuardBad = 1u << 30;
__global__ void guard_clear_kernel(int* __restrict__ flag) { flag[0] = 0; }
__global__ void __launch_bounds__(256) closure_guard_kernel(const float* __restrict__ C, int64_t P,
                                                            const float* __restrict__ limit,
                                                            unsigned* state, int* flag,
                                                            unsigned* __restrict__ counters) {
    const float* src = C + (int64_t)blockIdx.x * kGuardPer + threadIdx.x;
    const float L = limit[(int64_t)blockIdx.x * kGuardPer / P];   // kGuardPer divides P: one field per workgroup
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kGuardPer / 256; ++k) bad |= !(fabsf(src[256 * k]) <= L);
    const int any = __syncthreads_or(bad);
    if (threadIdx.x != 0) return;
    // one word, so a workgroup's verdict is there before its ticket
    if (any) atomicOr(state, kGuardBad);
    const unsigned seen = atomicAdd(state, 1u);
    if ((seen & ~kGuardBad) != gridDim.x - 1) return;
    const bool rejected = (seen & kGuardBad) != 0;
    atomicExch(state, 0u);
    atomicExch((unsigned*)flag, rejected ? 0u : 1u);
    atomicAdd(&counters[rejected ? 1 : 0], 1u);
}

}  // namespace sbli
