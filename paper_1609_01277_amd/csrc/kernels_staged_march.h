// The residual step of the staged form for large grids: workgroups march in z.
//
// staged_tiled_kernel forms one plane of a tile: each thread reads the 2R planes above
// and below from L2 and converts them again (make_pf) for every output plane.  At 256^3,
// FP64, order 8 that was 1,049 vector instructions and 11.7 GB through L2 a launch, and
// with 43 % VALU, 28 % L1, 25 % LDS and 2.5 TB/s nothing was busy: each plane is a chain of
// six waits for memory.  Here a workgroup owns a 16 x 16 tile and a run of planes; half
// of its wavefronts ("columns") keep the 2R + 1 planes of the z sums in a register window
// and do the update and the stores, the other half ("planes") stage a plane with its x
// and y arms in LDS and form the x and y sums, handed over as five partial sums a point.
// Each point is converted once per role, all loads but those of the plane that is written
// are requested a plane ahead, and the two kinds overlap on a SIMD.  One barrier a plane: a
// plane's LDS copy is double-buffered (written before barrier k, read after it), as are
// the partial sums (written after barrier k, read after barrier k + 1).
// FP64 at orders 10 and 12 would need more than the 256 VGPRs of two wavefronts a SIMD for
// its window (spills: 1,943 -> 2,221 us at order 12): there W_z, G_z and Th of the window
// are in LDS, which pays for it with single buffers and a second barrier a plane (A: the
// plane is staged, B: its sums are done), the columns passing A amid their z sums.
// There rho u_2 of the window is not held either but formed as rho u_2 + r from its remainder
// r = m - rho u_2, which is at most a rounding of m and needs no more than FP32: r's own
// rounding is 2^-24 of a unit in m's last place, so the sum rounds to m itself.
// The residual step at 256^3, FP64, order 8: 1,231 -> 880 us, 3.3 GB at 3.75 TB/s (a copy
// reaches 4.6), VALU 40 %, LDS 34 %; order 12: 1,619 -> 1,150.  (Both before the momentum along
// the axes was kept: a stage then takes 3 % and 6 % more.)
#pragma once

#include "kernels_staged.h"

namespace sbli {

// Fields of a staged plane over the tile and its arms: rho, rho E, Th, u_i, then the
// momentum where LDS keeps it, then p where the plain formulation needs it; and over the
// tile and the arms of one axis: W and G of that axis and the momentum along it (FP64).
template <typename T, bool PL>
constexpr int kMarchFields = (kMomentumInLds<T> ? 9 : 6) + (PL ? 1 : 0);
template <typename T>
constexpr int kMarchAxisFields = kMomentumInLds<T> ? 2 : 3;

// FP64 at orders 10 and 12: (W_z, G_z, Th) of the window in LDS, single buffers.
template <typename T, int R>
constexpr bool kMarchZLds = sizeof(T) == 8 && R >= 5;

// FP64 at orders 10 and 12: rho u_2 of the window from its remainder.
template <typename T, int R>
constexpr bool kMarchRem = sizeof(T) == 8 && R >= 5;

template <typename T, int R, bool PL>
struct MarchLds {
    static constexpr int TS = kStagedTile, SW = TS + 2 * R, NB = kMarchZLds<T, R> ? 1 : 2;
    // zr first: an LDS instruction's offset reaches 64 KB
    static constexpr int ZS = kMarchZLds<T, R> ? TS : 1;
    T zr[kMarchZLds<T, R> ? 2 * R + 1 : 1][3][ZS][ZS];
    static constexpr int RS = kMarchRem<T, R> ? TS : 1;
    float rem[kMarchRem<T, R> ? 2 * R + 1 : 1][RS][RS];
    T part[NB][5][TS][TS];
    T f[NB][kMarchFields<T, PL>][SW][SW];
    T w[NB][2][kMarchAxisFields<T>][TS * SW];   // x axis: rows of SW points; y axis: of TS
};

template <typename T, int R, int MODE>
__device__ __forceinline__ void march_columns(MarchLds<T, R, kPlain<T, MODE>>& lds, const T* __restrict__ q,
                                              const T* __restrict__ nf, T* __restrict__ dq, T* __restrict__ out,
                                              const BoxConst<T>& c, T dt, T A, T B, const T* __restrict__ clos,
                                              const int* __restrict__ cflag, int x0, int y0, int z0, int run) {
    constexpr int TS = kStagedTile, W = 2 * R + 1;
    constexpr bool PL = kPlain<T, MODE>, DQ = MODE == kModeStage2 || MODE == kModeStage3;
    constexpr bool ZU = kMomentumFromU<T, R>;
    const int nx = c.n[0], ny = c.n[1], nz = c.n[2];
    const int64_t P = c.P, plane = (int64_t)nx * ny;
    const int cx = threadIdx.x % TS, cy = threadIdx.x / TS;
    const bool store = x0 + cx < nx && y0 + cy < ny;
    unsigned fxo, fyo;
    const int64_t col = (int64_t)fold_index(y0 + cy, ny, c.sym[1], fyo) * nx + fold_index(x0 + cx, nx, c.sym[0], fxo);
    const bool wide = (int64_t)TS * nx * (int64_t)sizeof(T) >= kBufferBytes;
    const int soff = store && !wide ? (cy * nx + cx) * (int)sizeof(T) : kDropOff;
    const int64_t dcol = store ? col : (int64_t)y0 * nx + x0;
    constexpr int NB = MarchLds<T, R, PL>::NB;
    constexpr bool ZL = kMarchZLds<T, R>;
    PF<T> win[W];
    T Wz[W], Gz[W];
    T p0, p1, p2, p3, p4, pv, pt;
    unsigned pf;
    auto issue = [&](int z) {
        const int64_t i = (int64_t)map_index(z, nz, c.sym[2], pf) * plane + col;
        p0 = q[i];
        p1 = q[P + i];
        p2 = q[2 * P + i];
        p3 = q[3 * P + i];
        p4 = q[4 * P + i];
        pv = nf[2 * P + i];
        pt = nf[5 * P + i];
    };
    auto enter = [&](int k) {                      // the requested plane, converted
        PF<T>& s = win[k];
        s = make_pf<T, PL>(p0, p1, p2, flip_sign(p3, pf), p4, c);
        const T w = nested_W<PL>(flip_sign(pv, pf), s, s.u2, c), g = nested_G<PL>(pt, s, c);
        if constexpr (kMarchRem<T, R>) lds.rem[k][cy][cx] = (float)fmaT(-s.rho, s.u2, s.m2);
        if constexpr (ZL) {
            lds.zr[k][0][cy][cx] = w;
            lds.zr[k][1][cy][cx] = g;
            lds.zr[k][2][cy][cx] = s.Th;
        } else {
            Wz[k] = w;
            Gz[k] = g;
        }
    };
    auto W_at = [&](int k) { return ZL ? lds.zr[k][0][cy][cx] : Wz[k]; };
    auto G_at = [&](int k) { return ZL ? lds.zr[k][1][cy][cx] : Gz[k]; };
    auto plane_of = [&](int k) {                   // point of the window for the z sums
        PF<T> s = win[k];
        if constexpr (ZL) s.Th = lds.zr[k][2][cy][cx];
        if constexpr (kMarchRem<T, R>) s.m2 = fmaT(s.rho, s.u2, (T)lds.rem[k][cy][cx]);
        return z_point<T, R>(with_pressure<PL>(s, c));
    };
    T pd[5] = {0, 0, 0, 0, 0}, pm[2] = {0, 0};
    auto issue_own = [&](int z) {                  // dq, rho u_0 and rho u_1 of an output plane
        const int64_t i = (int64_t)z * plane + dcol;
        if constexpr (DQ) {
#pragma unroll
            for (int f = 0; f < 5; ++f) pd[f] = __builtin_nontemporal_load(&dq[f * P + i]);
        }
        if constexpr (ZU && MODE != kModeRHS) {
#pragma unroll
            for (int f = 0; f < 2; ++f) pm[f] = q[(1 + f) * P + i];
        }
    };
    issue(z0 - R);
    static_for<2 * R>([&](auto k) {
        constexpr int K = decltype(k)::value;
        enter(K);
        issue(z0 - R + K + 1);
        __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
    rotating_loop<W>(run, [&](auto ph, const int j) {
        constexpr int PH = decltype(ph)::value;
        auto slot = [](int k) { return (k + PH) % W; };
        const int z = z0 + j;
        enter(slot(2 * R));
        issue_own(z);
        if (j + 1 < run) issue(z + R + 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        const auto& pp = lds.part[NB == 2 ? j & 1 : 0];
        ResidualSums<T, PL> rs;
        rs.set({pp[0][cy][cx], pp[1][cy][cx], pp[2][cy][cx], pp[3][cy][cx], pp[4][cy][cx]});
        rs.begin();
        const PF<T> s = plane_of(slot(R));
#pragma unroll
        for (int m = 1; m <= R; ++m) {
            if (NB == 1 && m == 3 && j + 1 < run) __syncthreads();   // the next plane is staged
            rs.template add<2>(s, plane_of(slot(R + m)), W_at(slot(R + m)), G_at(slot(R + m)), plane_of(slot(R - m)),
                               W_at(slot(R - m)), G_at(slot(R - m)), c, m - 1);
        }
        rs.template end<2>(s, c);
        T Rv[5];
        rs.result(Rv);
        if (clos != nullptr && __builtin_amdgcn_readfirstlane(cflag[0]) != 0) {
            const int64_t id = (int64_t)z * plane + col;
#pragma unroll
            for (int f = 0; f < 5; ++f) Rv[f] += clos[f * P + id];
        }
        const PF<T>& w0 = win[slot(R)];
        const T qv[5] = {w0.rho, ZU ? pm[0] : w0.m0, ZU ? pm[1] : w0.m1, ZU ? s.m2 : w0.m2, w0.E};
        T dn[5], qn[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            dn[f] = MODE == kModeRHS ? Rv[f] : dt * Rv[f];
            if (DQ) dn[f] = fmaT(A, pd[f], dn[f]);
            if (MODE != kModeRHS) qn[f] = fmaT(B, dn[f], qv[f]);
        }
        if (wide && store) {
            const int64_t id = (int64_t)z * plane + col;
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                if (MODE == kModeStage1 || MODE == kModeStage2) dq[f * P + id] = dn[f];
                out[f * P + id] = MODE == kModeRHS ? dn[f] : qn[f];
            }
        }
        const int64_t org = (int64_t)z * plane + (int64_t)y0 * nx + x0;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            if (MODE == kModeRHS) {
                buffer_store_nt(dn[f], out + f * P + org, soff);
            } else {
                if (MODE != kModeStage3) buffer_store_nt(dn[f], dq + f * P + org, soff);
                buffer_store_nt(qn[f], out + f * P + org, soff);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

template <typename T, int R, int MODE>
__device__ __forceinline__ void march_planes(MarchLds<T, R, kPlain<T, MODE>>& lds, const T* __restrict__ q,
                                             const T* __restrict__ nf, const BoxConst<T>& c, int x0, int y0, int z0,
                                             int run) {
    constexpr int TS = kStagedTile, NT = TS * TS;
    constexpr int NB = MarchLds<T, R, kPlain<T, MODE>>::NB;
    constexpr int SW = TS + 2 * R;
    constexpr int NARM = 4 * R * TS, APT = (NARM + NT - 1) / NT;
    constexpr bool PL = kPlain<T, MODE>;
    const int nx = c.n[0], ny = c.n[1];
    const int64_t P = c.P, plane = (int64_t)nx * ny;
    const int t = threadIdx.x - NT;
    const int cx = t % TS, cy = t / TS;
    unsigned fxo, fyo;
    const int64_t col = (int64_t)fold_index(y0 + cy, ny, c.sym[1], fyo) * nx + fold_index(x0 + cx, nx, c.sym[0], fxo);
    // arm points: LDS position, column, mirror flags, axis of the arm
    int ax[APT], ay[APT], pair[APT];
    int64_t acol[APT], anf[APT];
    unsigned afx[APT], afy[APT];
#pragma unroll
    for (int k = 0; k < APT; ++k) {
        const int a = t + k * NT;
        ax[k] = ay[k] = -1;
        pair[k] = 0;
        acol[k] = col;       // a thread without this arm point requests its own (unused)
        afx[k] = afy[k] = 0u;
        if (a < NARM) {
            const int side = a / (R * TS), r = a % (R * TS);
            if (side < 2) {
                ay[k] = R + r / R;
                ax[k] = (side == 0 ? 0 : R + TS) + r % R;
            } else {
                ax[k] = R + r % TS;
                ay[k] = (side == 2 ? 0 : R + TS) + r / TS;
                pair[k] = 1;
            }
            acol[k] = (int64_t)fold_index(y0 - R + ay[k], ny, c.sym[1], afy[k]) * nx +
                      fold_index(x0 - R + ax[k], nx, c.sym[0], afx[k]);
        }
        anf[k] = acol[k] + pair[k] * P;
    }
    T po[9], pa[APT][7];
    auto issue = [&](int z) {
        const int64_t i = (int64_t)z * plane + col;
#pragma unroll
        for (int f = 0; f < 5; ++f) po[f] = q[f * P + i];
        po[5] = nf[i];
        po[6] = nf[3 * P + i];
        po[7] = nf[P + i];
        po[8] = nf[4 * P + i];
#pragma unroll
        for (int k = 0; k < APT; ++k) {
            const int64_t e = (int64_t)z * plane;
#pragma unroll
            for (int f = 0; f < 5; ++f) pa[k][f] = q[f * P + e + acol[k]];
            pa[k][5] = nf[e + anf[k]];
            pa[k][6] = nf[3 * P + e + anf[k]];
        }
    };
    auto put = [&](int b, int y, int x, const PF<T>& p, unsigned fx, unsigned fy) {
        auto& f = lds.f[b];
        f[0][y][x] = p.rho;
        f[1][y][x] = p.E;
        f[2][y][x] = p.Th;
        f[3][y][x] = flip_sign(p.u0, fx);
        f[4][y][x] = flip_sign(p.u1, fy);
        f[5][y][x] = p.u2;
        if constexpr (kMomentumInLds<T>) {
            f[6][y][x] = flip_sign(p.m0, fx);
            f[7][y][x] = flip_sign(p.m1, fy);
            f[8][y][x] = p.m2;
        }
        if constexpr (PL) f[kMarchFields<T, PL> - 1][y][x] = p.pk;
    };
    // the fields of one axis (0: x, 1: y) at element i of their rows
    auto put_axis = [&](int b, int axis, int i, const PF<T>& p, T V, T t, unsigned fx, unsigned fy) {
        T* w = &lds.w[b][axis][0][i];
        // W is odd under a mirror of its axis, and so is the momentum along it
        w[0] = flip_sign(nested_W<PL>(V, p, axis ? p.u1 : p.u0, c), axis ? fy : fx);
        w[TS * SW] = nested_G<PL>(t, p, c);
        if constexpr (!kMomentumInLds<T>) w[2 * TS * SW] = axis ? flip_sign(p.m1, fy) : flip_sign(p.m0, fx);
    };
    issue(z0);
    for (int it = 0; it < run; ++it) {
        const int b = NB == 2 ? it & 1 : 0;
        auto& f = lds.f[b];
        const PF<T> s0 = make_pf<T, PL>(po[0], po[1], po[2], po[3], po[4], c);
        put(b, R + cy, R + cx, s0, fxo, fyo);
        put_axis(b, 0, cy * SW + R + cx, s0, po[5], po[6], fxo, fyo);
        put_axis(b, 1, (R + cy) * TS + cx, s0, po[7], po[8], fxo, fyo);
#pragma unroll
        for (int k = 0; k < APT; ++k) {
            if (ax[k] >= 0) {
                const PF<T> p = make_pf<T, PL>(pa[k][0], pa[k][1], pa[k][2], pa[k][3], pa[k][4], c);
                put(b, ay[k], ax[k], p, afx[k], afy[k]);
                put_axis(b, pair[k], pair[k] ? ay[k] * TS + ax[k] - R : (ay[k] - R) * SW + ax[k], p, pa[k][5], pa[k][6],
                         afx[k], afy[k]);
            }
        }
        if (it + 1 < run) issue(z0 + it + 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        const auto& wx = lds.w[b][0];
        const auto& wy = lds.w[b][1];
        auto ld = [&](auto axis, int y, int x) {
            constexpr int D = decltype(axis)::value;
            PF<T> p;
            p.rho = f[0][y][x];
            p.E = f[1][y][x];
            p.Th = f[2][y][x];
            p.u0 = f[3][y][x];
            p.u1 = f[4][y][x];
            p.u2 = f[5][y][x];
            p.pk = 0;
            if constexpr (PL) p.pk = f[kMarchFields<T, PL> - 1][y][x];
            if constexpr (kMomentumInLds<T>) {
                p.m0 = f[6][y][x];
                p.m1 = f[7][y][x];
                p.m2 = f[8][y][x];
            } else if constexpr (D == 0) {
                p.m0 = wx[2][(y - R) * SW + x];
            } else {
                p.m1 = wy[2][y * TS + x - R];
            }
            return point_along<D>(p);
        };
        constexpr std::integral_constant<int, 0> along_x{};
        constexpr std::integral_constant<int, 1> along_y{};
        const int ly = cy + R, lx = cx + R;
        const int ix = cy * SW + lx, iy = ly * TS + cx;
        auto one_pair = [] {   // at orders 10 and 12 the threads spill without (7 to 22 registers)
            if constexpr (sizeof(T) == 8 && R >= 5) pair_fence();
        };
        const PF<T> sx = point_along<0>(s0);
        ResidualSums<T, PL> rs;
        rs.start(s0, c);
        rs.begin();
#pragma unroll
        for (int m = 1; m <= R; ++m) {
            one_pair();
            rs.template add<0>(sx, ld(along_x, ly, lx + m), wx[0][ix + m], wx[1][ix + m], ld(along_x, ly, lx - m),
                               wx[0][ix - m], wx[1][ix - m], c, m - 1);
        }
        rs.template end<0>(sx, c);
        const PF<T> sy = point_along<1>(s0);
        rs.begin();
#pragma unroll
        for (int m = 1; m <= R; ++m) {
            one_pair();
            rs.template add<1>(sy, ld(along_y, ly + m, lx), wy[0][iy + m * TS], wy[1][iy + m * TS],
                               ld(along_y, ly - m, lx), wy[0][iy - m * TS], wy[1][iy - m * TS], c, m - 1);
        }
        rs.template end<1>(sy, c);
        T sums[5];
        rs.get(sums);
#pragma unroll
        for (int k = 0; k < 5; ++k) lds.part[b][k][cy][cx] = sums[k];
        if (NB == 1) __syncthreads();   // the sums have been read
        __builtin_amdgcn_sched_barrier(0);
    }
    if (NB == 2) __syncthreads();
}

// FP32 at order 8: two workgroups a CU (128 VGPRs, 12 spilled) 776 us a stage at 256^3, one
// 807; the residual alone would spill 53.
template <typename T, int R, int MODE>
__global__ void __launch_bounds__(2 * kStagedTile * kStagedTile,
                                  (sizeof(T) == 4 && R == 4 && MODE != kModeRHS) ? 4 : 2)
    staged_march_kernel(const T* __restrict__ q, const T* __restrict__ nf, T* __restrict__ dq, T* __restrict__ out,
                        const BoxConst<T> c, T dt, T A, T B, const T* __restrict__ clos, const int* __restrict__ cflag,
                        int tiles_x, int tiles_y, int zchunk) {
    __shared__ MarchLds<T, R, kPlain<T, MODE>> lds;
    // XCDs and tiles as in fused_stage_kernel
    const int total = gridDim.x, w = blockIdx.x, xcd = w % 8, per = total / 8, extra = total % 8;
    const int lam = xcd * per + min(xcd, extra) + w / 8;
    const int tile = lam % (tiles_x * tiles_y), chunk = lam / (tiles_x * tiles_y);
    const int strip = tile / (kStripRows * tiles_x), in_strip = tile % (kStripRows * tiles_x);
    const int rows = min(kStripRows, tiles_y - strip * kStripRows);
    const int x0 = in_strip / rows * kStagedTile, y0 = (strip * kStripRows + in_strip % rows) * kStagedTile;
    const int z0 = chunk * zchunk, run = min(zchunk, c.n[2] - z0);
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) < kStagedTile * kStagedTile)   // whole wavefronts
        march_columns<T, R, MODE>(lds, q, nf, dq, out, c, dt, A, B, clos, cflag, x0, y0, z0, run);
    else
        march_planes<T, R, MODE>(lds, q, nf, c, x0, y0, z0, run);
}

}  // namespace sbli
