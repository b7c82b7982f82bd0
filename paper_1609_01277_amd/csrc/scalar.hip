// libsbli: scalar advection-diffusion on a periodic grid (include/sbli_scalar.h),
// the equation of the paper's 1D wave and 2D manufactured-solution cases, on the
// same central stencils (any even order 2..12) and the same low-storage RK3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "../../include/sbli.h"
#include "../../include/sbli_scalar.h"
#include "sbli_common.h"
#include "stencil_weights.h"

using namespace sbli;

namespace {

constexpr int kScalarMaxR = 6;

struct ScalarConst {
    int n[3];
    int64_t P;
    int r;
    int active[3];                  // axes with more than one point
    double da[3][kScalarMaxR];      // a_m / h
    double d2c0[3];                 // c_0 / h^2
    double d2c[3][kScalarMaxR];     // c_m / h^2
    double c[3];                    // advection velocity
    double k;                       // diffusivity
};

// Index of the neighbour m points away on a periodic axis of n points, for any m
// (a stencil may be wider than the grid: indices wrap modulo n).
__device__ __forceinline__ int64_t wrapped(int64_t id, int c, int m, int n, int64_t stride) {
    unsigned flip;
    const int cc = fold_index(c + m, n, 0, flip);
    return id + (int64_t)(cc - c) * stride;
}

// R = -sum_j c_j D_j phi + k sum_j D2_j phi - S, then (MODE != RHS) the 2N stage
// dq <- A dq + dt R, out <- phi + B dq.  One thread per point; neighbours through
// the caches (a scalar field needs no LDS staging to stay memory-bound).
template <int MODE>
__global__ void __launch_bounds__(256) scalar_stage_kernel(const double* __restrict__ phi,
                                                           const double* __restrict__ S, double* __restrict__ dq,
                                                           double* __restrict__ out, ScalarConst c, double dt,
                                                           double A, double B) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= c.P) return;
    const int i = (int)(id % c.n[0]);
    const int64_t t = id / c.n[0];
    const int j = (int)(t % c.n[1]);
    const int k = (int)(t / c.n[1]);
    const int coord[3] = {i, j, k};
    const int64_t stride[3] = {1, (int64_t)c.n[0], (int64_t)c.n[0] * c.n[1]};
    const double f0 = phi[id];
    double R = 0.0;
    for (int d = 0; d < 3; ++d) {
        if (!c.active[d]) continue;
        double s1 = 0.0, s2 = c.d2c0[d] * f0;
        for (int m = 1; m <= c.r; ++m) {
            const double fp = phi[wrapped(id, coord[d], m, c.n[d], stride[d])];
            const double fm = phi[wrapped(id, coord[d], -m, c.n[d], stride[d])];
            s1 += c.da[d][m - 1] * (fp - fm);
            s2 += c.d2c[d][m - 1] * (fp + fm);
        }
        R += c.k * s2 - c.c[d] * s1;
    }
    if (S) R -= S[id];
    if (MODE == kModeRHS) {
        out[id] = R;
    } else {
        double dn = dt * R;
        if (MODE != kModeStage1) dn += A * dq[id];
        if (MODE != kModeStage3) dq[id] = dn;
        out[id] = f0 + B * dn;
    }
}

// Many steps in one launch, the field in LDS.  A small grid's stage is a few hundred
// cycles of work, and a launch per stage costs 3.3 us of idle chip.  Here each point
// belongs to one thread, which keeps its value, its source and its dq in registers; a
// stage reads one LDS buffer and writes the other (one barrier), and what bounds it is
// that chain: LDS write, barrier, LDS read, the sums.  Per step, a launch a stage
// against this: 1000 points, order 8: 9.8 -> 0.9 us; 200,000 points: 14 -> 2.0; 32 x 32,
// order 4: 14 -> 1.8; 256 x 253: 16.5 -> 4.8; 1500 x 1497: 82 -> 31 (order 12: 134 ->
// 121).  The arithmetic is scalar_stage_kernel's, in its order.

// s1, s2 += the m-th pair of neighbours, and R of an axis from the sums.
__device__ __forceinline__ void pair_terms(double fm, double fp, double a, double b, double& s1, double& s2) {
    s1 += a * (fp - fm);
    s2 += b * (fp + fm);
}

// The 2N update of a point (stage k of a step); returns the new value.
__device__ __forceinline__ double stage_update(int k, double f0, double Rv, double dt, double& dq) {
    const double A = k == 0 ? 0.0 : (k == 1 ? -5.0 / 9.0 : -153.0 / 128.0);
    const double B = k == 0 ? 1.0 / 3.0 : (k == 1 ? 15.0 / 16.0 : 8.0 / 15.0);
    double dn = dt * Rv;
    if (k != 0) dn += A * dq;
    dq = dn;
    return f0 + B * dn;
}

// One axis.  RING: the whole field in one workgroup, its ends copied to ghost cells, any
// number of steps.  Otherwise a workgroup advances a tile `steps` steps from a copy that
// reaches H = 3 R steps points further on both sides, where the known part shrinks by R a
// stage; the field is read once and written once per launch.  A thread holds two adjacent
// points: their windows of 2 R + 2 values are R + 1 16-byte reads without bank conflicts.
constexpr int kTileThreads = 256;
constexpr int kTilePoints = 2 * kTileThreads;

template <int R, bool RING>
__global__ void __launch_bounds__(kTileThreads)
    scalar_march_kernel(const double* __restrict__ src, const double* __restrict__ S, double* __restrict__ dst,
                        ScalarConst c, int d, double dt, int steps) {
    constexpr int E = (R + 1) / 2 * 2;                      // ghost cells of a side, pairs aligned
    __shared__ double2 cells[2][kTileThreads + E];
    const int N = (int)c.P;
    const int H = RING ? 0 : 3 * R * steps;
    const int NB = RING ? N : kTilePoints;
    const int64_t base = RING ? 0 : (int64_t)blockIdx.x * (kTilePoints - 2 * H) - H;
    const int i0 = 2 * threadIdx.x;
    double f[2] = {0.0, 0.0}, dq[2] = {0.0, 0.0}, sv[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (i0 + j < NB) {
            int64_t g = (base + i0 + j) % N;
            if (g < 0) g += N;
            f[j] = src[g];
            if (S) sv[j] = S[g];
        }
    int b = 0, lo = 0;
    auto put = [&](double* o) {                             // the thread's points and their ghost copies
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = i0 + j;
            if (i < NB) {
                o[i] = f[j];
                if (RING) {
                    if (i < R) o[i + N] = f[j];
                    if (i >= N - R) o[i - N] = f[j];
                }
            }
        }
    };
    put(&cells[0][E / 2].x);
    __syncthreads();
    for (int st = 0; st < steps; ++st) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (!RING) lo += R;
            if (i0 + 1 >= lo && i0 < NB - lo) {
                double w[2 * E + 2];
#pragma unroll
                for (int m = 0; m <= E; ++m) {
                    const double2 v = cells[b][threadIdx.x + m];
                    w[2 * m] = v.x;
                    w[2 * m + 1] = v.y;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    double s1 = 0.0, s2 = c.d2c0[d] * f[j];
#pragma unroll
                    for (int m = 1; m <= R; ++m) pair_terms(w[E + j - m], w[E + j + m], c.da[d][m - 1], c.d2c[d][m - 1], s1, s2);
                    double Rv = 0.0;
                    Rv += c.k * s2 - c.c[d] * s1;
                    if (S) Rv -= sv[j];
                    f[j] = stage_update(k, f[j], Rv, dt, dq[j]);
                }
                put(&cells[b ^ 1][E / 2].x);
            }
            b ^= 1;
            __syncthreads();
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int i = i0 + j;
        if (i >= H && i < NB - H && base + i < N) dst[base + i] = f[j];
    }
}

// Two axes, ax and ay.  RING: the whole field in one workgroup (BX x BY its size);
// otherwise tiles of (BX - 2 H) x (BY - 2 H) points, as above.  A thread's points lie
// kPlaneThreads apart.
constexpr int kPlaneThreads = 1024;
constexpr int kPlanePpt = 4;
constexpr int kPlanePoints = kPlaneThreads * kPlanePpt;
constexpr int kRing2Points = 2304;
// Points and ghost cells of a ring: (nx + 2 R)(ny + 2 R) with nx ny <= kRing2Points and
// no axis under 2 R points is largest at ny = 2 R, R = kScalarMaxR.
constexpr int kRing2Cells = (kRing2Points / (2 * kScalarMaxR) + 2 * kScalarMaxR) * 4 * kScalarMaxR;

template <int R, bool RING>
__global__ void __launch_bounds__(kPlaneThreads)
    scalar_plane_kernel(const double* __restrict__ src, const double* __restrict__ S, double* __restrict__ dst,
                        ScalarConst c, int ax, int ay, double dt, int steps, int BX, int BY) {
    __shared__ double buf[2][RING ? kRing2Cells : kPlanePoints];
    const int nx = c.n[ax], ny = c.n[ay], B = BX * BY;
    const int G = RING ? R : 0, W = BX + 2 * G;
    const int H = RING ? 0 : 3 * R * steps;
    const int x0 = RING ? 0 : (int)blockIdx.x * (BX - 2 * H) - H;
    const int y0 = RING ? 0 : (int)blockIdx.y * (BY - 2 * H) - H;
    double f[kPlanePpt], dq[kPlanePpt], sv[kPlanePpt];
    int at[kPlanePpt], gx[kPlanePpt], gy[kPlanePpt];        // LDS cell of the point, offsets of its ghost copies
    int reach[kPlanePpt];                                   // stages (times R) for which the point is known
#pragma unroll
    for (int j = 0; j < kPlanePpt; ++j) {
        const int p = threadIdx.x + j * kPlaneThreads, y = p / BX, x = p - y * BX;
        f[j] = dq[j] = sv[j] = 0.0;
        at[j] = (y + G) * W + x + G;
        gx[j] = x < R ? nx : (x >= nx - R ? -nx : 0);
        gy[j] = y < R ? ny * W : (y >= ny - R ? -ny * W : 0);
        reach[j] = p < B ? (RING ? 0 : min(min(x, BX - 1 - x), min(y, BY - 1 - y))) : -1;
        if (p < B) {
            int X = RING ? x : (x0 + x) % nx, Y = RING ? y : (y0 + y) % ny;
            if (X < 0) X += nx;
            if (Y < 0) Y += ny;
            const int64_t g = (int64_t)Y * nx + X;
            f[j] = src[g];
            if (S) sv[j] = S[g];
        }
    }
    auto put = [&](double* o, int j) {
        o[0] = f[j];
        if (RING) {
            if (gx[j]) o[gx[j]] = f[j];
            if (gy[j]) o[gy[j]] = f[j];
        }
    };
#pragma unroll
    for (int j = 0; j < kPlanePpt; ++j)
        if (reach[j] >= 0) put(&buf[0][at[j]], j);
    __syncthreads();
    int b = 0, lo = 0;
    for (int st = 0; st < steps; ++st) {
#pragma unroll 1
        for (int k = 0; k < 3; ++k) {
            if (!RING) lo += R;
#pragma unroll
            for (int j = 0; j < kPlanePpt; ++j) {
                if (reach[j] >= lo) {
                    const double* q = &buf[b][at[j]];
                    double Rv = 0.0;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int d = e == 0 ? ax : ay, stride = e == 0 ? 1 : W;
                        double s1 = 0.0, s2 = c.d2c0[d] * f[j];
#pragma unroll
                        for (int m = 1; m <= R; ++m)
                            pair_terms(q[-m * stride], q[m * stride], c.da[d][m - 1], c.d2c[d][m - 1], s1, s2);
                        Rv += c.k * s2 - c.c[d] * s1;
                    }
                    if (S) Rv -= sv[j];
                    f[j] = stage_update(k, f[j], Rv, dt, dq[j]);
                    put(&buf[b ^ 1][at[j]], j);
                }
            }
            b ^= 1;
            __syncthreads();
        }
    }
#pragma unroll
    for (int j = 0; j < kPlanePpt; ++j) {
        const int p = threadIdx.x + j * kPlaneThreads, y = p / BX, x = p - y * BX;
        if (reach[j] >= H && x0 + x < nx && y0 + y < ny) dst[(int64_t)(y0 + y) * nx + x0 + x] = f[j];
    }
}

__global__ void __launch_bounds__(256) scalar_copy_kernel(const double* __restrict__ src, double* __restrict__ dst,
                                                          int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

thread_local std::string t_err;

int sfail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    t_err = buf;
    return code;
}

int make_const(const sbli_scalar_params* p, ScalarConst* c) {
    if (!p) return sfail(SBLI_ERR_ARG, "scalar: params is NULL");
    if (p->order < 2 || p->order > 2 * kScalarMaxR || p->order % 2)
        return sfail(SBLI_ERR_ARG, "scalar: order must be even in [2, %d] (got %d)", 2 * kScalarMaxR, p->order);
    const int r = p->order / 2;
    double a[kScalarMaxR], cc[kScalarMaxR], c0;
    central_weights(r, a, &c0, cc);
    c->r = r;
    c->P = 1;
    int nact = 0;
    for (int d = 0; d < 3; ++d) {
        const int n = p->n[d];
        if (n < 1) return sfail(SBLI_ERR_ARG, "scalar: n[%d] must be >= 1", d);
        c->n[d] = n;
        c->P *= n;
        c->active[d] = n > 1;
        nact += n > 1;
        if (n > 1 && !(p->length[d] > 0 && std::isfinite(p->length[d])))
            return sfail(SBLI_ERR_ARG, "scalar: length[%d] must be finite and > 0", d);
        const double h = n > 1 ? p->length[d] / n : 1.0;
        for (int m = 0; m < kScalarMaxR; ++m) {
            c->da[d][m] = m < r ? a[m] / h : 0.0;
            c->d2c[d][m] = m < r ? cc[m] / (h * h) : 0.0;
        }
        c->d2c0[d] = c0 / (h * h);
        c->c[d] = p->c[d];
        if (!std::isfinite(p->c[d])) return sfail(SBLI_ERR_ARG, "scalar: velocity must be finite");
    }
    if (nact == 0) return sfail(SBLI_ERR_ARG, "scalar: at least one axis needs more than one point");
    if (!(p->k >= 0 && std::isfinite(p->k))) return sfail(SBLI_ERR_ARG, "scalar: k must be finite and >= 0");
    c->k = p->k;
    return SBLI_OK;
}

const double kA[3] = {0.0, -5.0 / 9.0, -153.0 / 128.0};
const double kB[3] = {1.0 / 3.0, 15.0 / 16.0, 8.0 / 15.0};

// How sbli_scalar_rk3 advances a grid.
enum { kPerStage, kRing1, kTiles1, kRing2, kTiles2 };
struct Route {
    int kind;
    int ax, ay;    // the active axes of the marching forms
    int steps;     // steps of a launch at most
    int bx, by;    // buffer of a two-axis tile
};

constexpr int kRingSteps = 4096;                            // keeps a launch to some milliseconds
constexpr int kCus = 256;

// The buffer and the steps of a launch of two-axis tiles, by their modelled time: a
// launch's 4 us and, per step, 0.7 us and 2.2 + 0.6 R us for each 4096 cells; workgroups
// beyond one a CU queue, those of small buffers partly beside each other.  Measured from
// 48^2 to 1500^2 at orders 2 to 12: its choice is the fastest of the fifteen or within
// 15 % of it, which the other choices miss by up to 3 times.
Route plane_tiles(const ScalarConst& c, int ax, int ay, int nsteps, double* us_step) {
    static const struct { int x, y; double share; } bufs[] = {{64, 64, 1.0}, {64, 48, 1.0}, {48, 48, 1.0},
                                                              {64, 32, 0.85}, {32, 32, 0.75}};
    Route best{kPerStage, ax, ay, 1, 0, 0};
    double best_us = 0.0;
    for (const auto& b : bufs)
        for (int steps : {1, 2, 4}) {
            const int tx = b.x - 6 * c.r * steps, ty = b.y - 6 * c.r * steps;
            if (tx < 4 || ty < 4 || steps > std::max(nsteps, 1)) continue;
            const double gx = std::ceil((double)c.n[ax] / tx), gy = std::ceil((double)c.n[ay] / ty);
            if (gx > 65535.0 || gy > 65535.0) continue;
            const double step_us = 0.7 + b.x * b.y * (2.2 + 0.6 * c.r) / kPlanePoints;
            const double us = (1.0 + (3.0 + steps * step_us) * std::max(1.0, std::ceil(gx * gy / kCus) * b.share)) / steps;
            if (best.kind == kPerStage || us < best_us) {
                best = {kTiles2, ax, ay, steps, b.x, b.y};
                best_us = us;
            }
        }
    *us_step = best_us;
    return best;
}

// Modelled us a step of a launch a stage on two axes: three launches and, per point, the
// loads of the stencil.  Within 25 % of the measurements (1,024 x 1,024 to 8,192 x 8,192,
// 12 x 2^20, 2^20 x 12, 20 x 10^5, 65,536 x 64; orders 2 to 12).
double stage_model(const ScalarConst& c, int ax) {
    const double ps = (c.n[ax] < 64 ? 11.0 : 17.0) + 7.0 * c.r + (c.P > (1 << 23) ? 5.0 : 0.0);
    return 10.0 + c.P * ps * 1e-6;
}

// Measured, us a step.  One axis: a ring of 512 points 0.98 to 1.24 (orders 2 to 12),
// tiles 0.88 to 1.42; a tile no larger than gives every CU one, since its margin is then
// free (1000 points, order 8: 1.09 with T = 192, 1.26 with 320), and 320 points beyond
// (200,000 points: 1.96 with 320, 2.11 with 192).  Two axes: a ring of 48^2 points 2.5
// to 6.2, tiles 2.4 to 7.9; of 64^2 4.0 to 10.9, tiles 2.5 to 8.1.  A launch a stage
// (8 to 134) stays for three axes, for a stencil wider than the axis, whose ghost
// cells would hold a point more than once, and for thin grids at high orders, whose tiles
// are mostly margin (12 x 2^20, a launch a stage and tiles: order 2 330, 413; order 12 755,
// 1,497; 20 x 10^5: order 4 61, 58; order 8 88, 96; 65,536 x 64, order 12: 223, 299): where
// the modelled times say so.
Route choose_route(const ScalarConst& c, int nsteps) {
    int act[3], na = 0;
    for (int d = 0; d < 3; ++d)
        if (c.active[d]) {
            if (c.n[d] < 2 * c.r) return {kPerStage, 0, 0, 1, 0, 0};
            act[na++] = d;
        }
    if (na == 1) {
        if (c.P <= kTilePoints) return {kRing1, act[0], 0, kRingSteps, 0, 0};
        const int T = (int)std::min<int64_t>(std::max<int64_t>((c.P + kCus - 1) / kCus, 64), 320);
        return {kTiles1, act[0], 0, (kTilePoints - T) / (6 * c.r), 0, 0};
    }
    if (na == 2) {
        if (c.P <= kRing2Points) return {kRing2, act[0], act[1], kRingSteps, 0, 0};
        double us;
        const Route tiles = plane_tiles(c, act[0], act[1], nsteps, &us);
        if (tiles.kind == kPerStage || stage_model(c, act[0]) < 1.05 * us) return {kPerStage, 0, 0, 1, 0, 0};
        return tiles;
    }
    return {kPerStage, 0, 0, 1, 0, 0};
}

template <int R>
void march_launch_r(const Route& r, const ScalarConst& c, hipStream_t s, const double* src, const double* S,
                    double* dst, double dt, int steps) {
    if (r.kind == kRing1) {
        const int nt = (int)((c.P + 127) / 128 * 64);
        scalar_march_kernel<R, true><<<1, nt, 0, s>>>(src, S, dst, c, r.ax, dt, steps);
    } else if (r.kind == kTiles1) {
        const int T = kTilePoints - 6 * R * steps;
        scalar_march_kernel<R, false><<<(unsigned)((c.P + T - 1) / T), kTileThreads, 0, s>>>(src, S, dst, c, r.ax, dt,
                                                                                            steps);
    } else if (r.kind == kRing2) {
        scalar_plane_kernel<R, true><<<1, kPlaneThreads, 0, s>>>(src, S, dst, c, r.ax, r.ay, dt, steps, c.n[r.ax],
                                                                 c.n[r.ay]);
    } else {
        const int tx = r.bx - 6 * R * steps, ty = r.by - 6 * R * steps;
        const dim3 grid((c.n[r.ax] + tx - 1) / tx, (c.n[r.ay] + ty - 1) / ty);
        scalar_plane_kernel<R, false><<<grid, kPlaneThreads, 0, s>>>(src, S, dst, c, r.ax, r.ay, dt, steps, r.bx, r.by);
    }
}

void march_launch(const Route& r, const ScalarConst& c, hipStream_t s, const double* src, const double* S, double* dst,
                  double dt, int steps) {
    switch (c.r) {
        case 1: march_launch_r<1>(r, c, s, src, S, dst, dt, steps); break;
        case 2: march_launch_r<2>(r, c, s, src, S, dst, dt, steps); break;
        case 3: march_launch_r<3>(r, c, s, src, S, dst, dt, steps); break;
        case 4: march_launch_r<4>(r, c, s, src, S, dst, dt, steps); break;
        case 5: march_launch_r<5>(r, c, s, src, S, dst, dt, steps); break;
        default: march_launch_r<6>(r, c, s, src, S, dst, dt, steps); break;
    }
}

}  // namespace

extern "C" const char* sbli_scalar_last_error(void) { return t_err.c_str(); }

extern "C" int sbli_scalar_rhs(const sbli_scalar_params* p, const double* phi, const double* source, double* rhs,
                               void* hip_stream) {
    ScalarConst c;
    int rc = make_const(p, &c);
    if (rc != SBLI_OK) return rc;
    if (!phi || !rhs) return sfail(SBLI_ERR_ARG, "sbli_scalar_rhs: NULL pointer");
    if (phi == rhs) return sfail(SBLI_ERR_ARG, "sbli_scalar_rhs: phi and rhs must differ");
    const unsigned blocks = (unsigned)((c.P + 255) / 256);
    scalar_stage_kernel<kModeRHS><<<blocks, 256, 0, (hipStream_t)hip_stream>>>(phi, source, nullptr, rhs, c, 0.0,
                                                                              0.0, 0.0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sfail(SBLI_ERR_HIP, "sbli_scalar_rhs: %s", hipGetErrorString(e));
    return SBLI_OK;
}

extern "C" int sbli_scalar_rk3(const sbli_scalar_params* p, double* phi, double* phi_tmp, double* dphi,
                               const double* source, double dt, int nsteps, void* hip_stream) {
    ScalarConst c;
    int rc = make_const(p, &c);
    if (rc != SBLI_OK) return rc;
    if (!phi || !phi_tmp || !dphi) return sfail(SBLI_ERR_ARG, "sbli_scalar_rk3: NULL pointer");
    if (phi == phi_tmp || phi == dphi || phi_tmp == dphi)
        return sfail(SBLI_ERR_ARG, "sbli_scalar_rk3: phi, phi_tmp and dphi must be distinct");
    if (nsteps < 0 || !std::isfinite(dt)) return sfail(SBLI_ERR_ARG, "sbli_scalar_rk3: need nsteps >= 0, finite dt");
    hipStream_t s = (hipStream_t)hip_stream;
    const unsigned blocks = (unsigned)((c.P + 255) / 256);
    double* src = phi;
    double* dst = phi_tmp;
    const Route route = choose_route(c, nsteps);
    for (int st = 0; st < nsteps;) {
        if (route.kind != kPerStage) {
            const int k = std::min(nsteps - st, route.steps);
            march_launch(route, c, s, src, source, dst, dt, k);
            std::swap(src, dst);
            st += k;
            continue;
        }
        scalar_stage_kernel<kModeStage1><<<blocks, 256, 0, s>>>(src, source, dphi, dst, c, dt, kA[0], kB[0]);
        std::swap(src, dst);
        scalar_stage_kernel<kModeStage2><<<blocks, 256, 0, s>>>(src, source, dphi, dst, c, dt, kA[1], kB[1]);
        std::swap(src, dst);
        scalar_stage_kernel<kModeStage3><<<blocks, 256, 0, s>>>(src, source, dphi, dst, c, dt, kA[2], kB[2]);
        std::swap(src, dst);
        ++st;
    }
    if (src != phi) {
        const unsigned cb = (unsigned)std::min<int64_t>((c.P + 255) / 256, 65536);
        scalar_copy_kernel<<<cb, 256, 0, s>>>(src, phi, c.P);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sfail(SBLI_ERR_HIP, "sbli_scalar_rk3: %s", hipGetErrorString(e));
    return SBLI_OK;
}
