// Fused residual + RK3-stage kernel: one launch per stage, the state read once
// and written once per point (plus dq).
//
// Data flow (per workgroup): a TX x TY tile of (x, y) columns marches along z.
// The nested terms of the residual (viscous work D_j(u_i tau_ij) and the
// grad-div part D_i(D_k u_k), paper Sec. "Expanding": inner derivative first)
// need the velocity gradient on a ring of R columns around the tile and R
// planes ahead of the output plane, so every stage is a pipeline per z-plane:
//   1. each column thread loads the state R planes ahead of the gradient plane
//      and keeps a register window of 3R+1 planes of point fields; the gradient
//      plane's fields go to LDS (u over the tile + 2R ring, the others over the
//      tile + R ring);
//   2. the gradient plane a: velocity gradient by x/y stencils over that LDS
//      plane and z stencils over the register window, reduced at once to the six
//      fields the outer derivatives act on (nested_terms): the x/y pairs go to
//      LDS, the z pair to a ring of the thread's own column;
//   3. the x and y sums of the residual on the newest plane whose nested fields
//      are in LDS: the same LDS plane serves the gradient and these sums, so u is
//      stored once, and five partial residuals per column wait for the z sums;
//   4. the output plane o = a - R: the z sums from the register window and the
//      ring, and the RK update written straight to HBM.
// Columns of the R-ring around the tile are handled by extra "halo" threads
// (whole wavefronts apart from the interior ones); the 2R-ring of u needed only
// for the x/y gradient stencils of halo columns is loaded directly.
//
// Two barrier schedules.  DB = 0: step 1 | barrier | step 2 | barrier | steps 3
// (on plane a) and 4; two buffers of the LDS plane, one of the nested pairs.
// DB = 1: step 3 runs one plane behind the gradient (on plane a - 1), so nothing
// it reads was written by another thread since the last barrier: step 1 | barrier
// | steps 2, 3 and 4 in any order; three buffers of the LDS plane (a - 1, a and
// the next one, which a fast wavefront may already store) and two of the nested
// pairs.  Periodic
// wrap (or, on a symmetry axis, the mirror image with the normal momentum
// negated) is folded into the column and plane coordinates, so ragged tiles and
// boundaries need no special case beyond masking the stores.
#pragma once

#include <type_traits>
#include <utility>

#include "sbli_common.h"

namespace sbli {

template <int R, int TX, int TY>
struct FusedShape {
    static constexpr int NI = TX * TY;              // interior columns
    static constexpr int NHX = 2 * R * TY;          // x-ring columns
    static constexpr int NHY = 2 * R * TX;          // y-ring columns
    static constexpr int NE1 = NI + NHX + NHY;      // columns with a register window
    static constexpr int NT = (NE1 + 63) / 64 * 64; // threads per workgroup
    // LDS boxes of the point fields and of u.  Rows are padded to an odd length: the
    // x-ring's threads walk down a column, and an even stride puts them on a few banks
    // (420 of 2,630 LDS cycles a plane at 16 x 16, FP64 order 4, before the padding).
    static constexpr int BX1 = TX + 2 * R + 1, BY1 = TY + 2 * R;
    static constexpr int BX2 = TX + 4 * R + 1, BY2 = TY + 4 * R;
    static constexpr int NOUT = 2 * R * TY + 2 * R * TX + 4 * R * R;  // u-only ring points
    static_assert(NI % 64 == 0, "interior columns must fill whole wavefronts");
    static_assert(NOUT <= NT, "one u-ring point per thread at most");
};

// Point fields kept per plane and per column.
template <typename T>
struct PF {
    // pk = -(gamma - 1) rho u_j u_j, so 2p = 2 (gamma - 1) rho E + pk; Th = (gamma / Pr) times
    // the internal energy, the temperature scaled so that the heat flux is (1/Re) grad Th.
    // (kPlain: p and T.)
    T rho, m0, m1, m2, E, u0, u1, u2, pk, Th;
};

// 1/x from the hardware reciprocal refined by Newton steps (two in FP64, one in
// FP32): within an ulp of the quotient, at a third of the instructions of the
// IEEE division sequence.
__device__ __forceinline__ double fast_recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float fast_recip(float x) {
    float r = __builtin_amdgcn_rcpf(x);
    const float e = __builtin_fmaf(-x, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}

// a*b + c with one rounding.  The residual arithmetic spells out its fused
// multiply-adds (the library is built with contraction limited to single
// expressions), so every launch variant rounds every point identically.
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// The residual itself in FP32 (sbli_rhs) keeps the sums of the plain formulation: there
// the result is the residual, and in a nearly incompressible state the FP32 rounding of
// the pressure gradient is a visible part of it (2e-4 of the momentum residual at 48^3,
// 2 % of a closure target, which subtracts two residuals).  Another order of operations
// rounds as well but differently, and results that are compared or trained on would
// change by that much.  Everything else uses the shorter sums (see ResidualSums).
template <typename T, int MODE>
constexpr bool kPlain = sizeof(T) == 4 && MODE == kModeRHS;

// Velocity component m / rho, rr = fast_recip(rho).  Every field's residual inherits the
// rounding of u, so outside the plain formulation one residual step makes it the rounded
// quotient: two operations a component, for an error of the mass residual of 0.8 times
// (FP64, order 4) and of the energy residual of 0.65 times that of the plain formulation
// (1.02 and 0.86 without the step).
template <bool PLAIN, typename T>
__device__ __forceinline__ T velocity(T m, T rho, T rr) {
    const T u = m * rr;
    if constexpr (PLAIN) return u;
    else return fmaT(fmaT(-rho, u, m), rr, u);
}

template <typename T, bool PLAIN>
__device__ __forceinline__ PF<T> make_pf(T rho, T m0, T m1, T m2, T E, const BoxConst<T>& c) {
    PF<T> s;
    s.rho = rho;
    s.m0 = m0;
    s.m1 = m1;
    s.m2 = m2;
    s.E = E;
    const T rr = fast_recip(rho);
    s.u0 = velocity<PLAIN>(m0, rho, rr);
    s.u1 = velocity<PLAIN>(m1, rho, rr);
    s.u2 = velocity<PLAIN>(m2, rho, rr);
    const T ke2 = fmaT(m2, s.u2, fmaT(m1, s.u1, m0 * s.u0));    // 2 x kinetic energy
    if constexpr (PLAIN) {
        s.pk = c.gm1 * fmaT(T(-0.5), ke2, E);
        s.Th = c.gM2 * s.pk * rr;
    } else {
        s.pk = -(c.gm1 * ke2);
        s.Th = c.gPr * fmaT(T(-0.5), ke2, E) * rr;
    }
    return s;
}

// The pressure of a point of the plain formulation, formed again from the other fields
// (the same operations as in make_pf): the register windows need not hold it.
template <bool PLAIN, typename T>
__device__ __forceinline__ PF<T> with_pressure(PF<T> s, const BoxConst<T>& c) {
    if constexpr (PLAIN) s.pk = c.gm1 * fmaT(T(-0.5), fmaT(s.m2, s.u2, fmaT(s.m1, s.u1, s.m0 * s.u0)), s.E);
    return s;
}

// Calls f(integral_constant<int, 0>), ..., f(integral_constant<int, N-1>).
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Stores through a raw buffer descriptor.  `off` is the byte offset from the
// descriptor's base; one beyond its size drops the store, so lanes without an
// output take part in the instruction and no branch surrounds it.
constexpr int kBufferWord3 = 0x00020000;   // descriptor word 3 of a raw (untyped) buffer
constexpr int kBufferBytes = 0x40000000;   // descriptor size
constexpr int kDropOff = 0x40000000;       // first offset that is dropped
constexpr int kAuxNt = 2;                  // non-temporal
typedef int sbli_v2i __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ void buffer_store_nt(T v, T* base, int off) {
    const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(base, 0, kBufferBytes, kBufferWord3);
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(sbli_v2i, v), d, off, 0, kAuxNt);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), d, off, 0, kAuxNt);
}
// N stores that are all dropped (at distinct offsets: equal ones would be merged):
// they keep the count of memory operations equal on both sides of a uniform branch.
template <int N, typename T>
__device__ __forceinline__ void dropped_stores(T* any) {
#pragma unroll
    for (int k = 0; k < N; ++k) buffer_store_nt(T(0), any, kDropOff + 16 * k);
}

__device__ __forceinline__ int wrap_mod(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// Whether the momentum of a point is kept in LDS beside rho and u.  In FP64 the LDS
// pipe is the busier one (44 % against 34 % for the VALU at order 4, 512^3), and
// x and y neighbours form the momentum across the axis as rho u_i again; in FP32, with
// half the bytes, the VALU is.  The momentum along the axis is always the state's own: in
// the mass residual D_j (rho u_j) carries the rounding of rho u_j in full, and with rho
// times the rounded u_j that residual's error was 1.7 to 2.0 times the plain formulation's.
template <typename T>
constexpr bool kMomentumInLds = sizeof(T) == 4;
// LDS fields of a plane beside u: rho, rho E, Th, the momentum where it is kept, and the
// pressure where it is not part of the nested fields.
template <typename T, bool PLAIN>
constexpr int kPlFields = (kMomentumInLds<T> ? 6 : 3) + (PLAIN ? 1 : 0);
// Fields of a plane below the output plane in LDS (ZL; FP64 only): rho, rho u_i, rho E, u_i, Th.
constexpr int kZtFields = 9;

// A point of the sums along axis d: s.m_d is the state's, the others are formed from u
// (the centre point like its neighbours).
template <int d, typename T>
__device__ __forceinline__ PF<T> point_along(PF<T> s) {
    if constexpr (!kMomentumInLds<T>) {
        if constexpr (d != 0) s.m0 = s.rho * s.u0;
        if constexpr (d != 1) s.m1 = s.rho * s.u1;
        if constexpr (d != 2) s.m2 = s.rho * s.u2;
    }
    return s;
}

// FP64 at orders 6 and up: the z sums form the momentum across the axis likewise, so that
// a register window of 2R + 1 planes need not hold it.
template <typename T, int R>
constexpr bool kMomentumFromU = !kMomentumInLds<T> && R >= 3;
template <typename T, int R>
__device__ __forceinline__ PF<T> z_point(PF<T> s) {
    if constexpr (kMomentumFromU<T, R>) return point_along<2>(s);
    return s;
}

// The nested terms of axis j act on V_j = Re u_i tau_ij and t_j = 2 (g_jj - theta) / (3 Re)
// (g_ij = D_j u_i, theta = g_kk).  With the point's pressure they become the two
// fields whose first derivatives enter the residual:
//   W_j = 2 (u_i tau_ij - p u_j)  (energy)    G_j = 2 p - 2 (theta - g_jj) / (3 Re)  (momentum j)
// so the pressure terms cost a stencil nothing.  2p is taken from rho E and pk each time, so
// G is rounded once at the size of 2p where p from the internal energy is rounded twice: the
// momentum residual's error is 0.6 to 0.8 times the plain formulation's.
// PLAIN: V_j = u_i tau_ij and t_j = theta - g_jj themselves, W = V, G = t.
template <bool PLAIN, typename T>
__device__ __forceinline__ void nested_terms(const T (&g)[3][3], T u0, T u1, T u2, const BoxConst<T>& c, T (&V)[3],
                                             T (&t)[3]) {
    const T theta = g[0][0] + g[1][1] + g[2][2];
    if constexpr (PLAIN) {
        const T uc[3] = {u0, u1, u2};
#pragma unroll
        for (int jj = 0; jj < 3; ++jj) {
            T v = 0;
#pragma unroll
            for (int ii = 0; ii < 3; ++ii) {
                T tau = c.inv_Re * (g[ii][jj] + g[jj][ii]);
                if (ii == jj) tau = fmaT(-c.inv_Re23, theta, tau);
                v = fmaT(uc[ii], tau, v);
            }
            V[jj] = v;
            t[jj] = theta - g[jj][jj];
        }
    } else {
        const T th23 = T(2.0 / 3.0) * theta;
        const T s01 = g[0][1] + g[1][0], s02 = g[0][2] + g[2][0], s12 = g[1][2] + g[2][1];
        V[0] = fmaT(u2, s02, fmaT(u1, s01, u0 * fmaT(T(2), g[0][0], -th23)));
        V[1] = fmaT(u2, s12, fmaT(u1, fmaT(T(2), g[1][1], -th23), u0 * s01));
        V[2] = fmaT(u2, fmaT(T(2), g[2][2], -th23), fmaT(u1, s12, u0 * s02));
#pragma unroll
        for (int j = 0; j < 3; ++j) t[j] = c.inv_3Re2 * (g[j][j] - theta);
    }
}
template <bool PLAIN, typename T>
__device__ __forceinline__ T nested_W(T V, const PF<T>& s, T u, const BoxConst<T>& c) {
    return PLAIN ? V : fmaT(c.inv_Re2, V, -(fmaT(c.gm1x2, s.E, s.pk) * u));
}
template <bool PLAIN, typename T>
__device__ __forceinline__ T nested_G(T t, const PF<T>& s, const BoxConst<T>& c) {
    return PLAIN ? t : fmaT(c.gm1x2, s.E, s.pk + t);
}

// -2 times the residual of one point, summed neighbour pair by neighbour pair.
//
// Convection in the skew-symmetric form is, for Q in (rho, rho u_i, rho E) and by
// linearity of D, -1/2 [D(Q u) + Q D u + u D Q] = -1/2 sum_m a_m/h [(Q + Q+)(u + u+) -
// (Q + Q-)(u + u-)], and each bracket is (Q + Q+)(u+ - u-) + (Q+ - Q-)(u + u-): differences
// of neighbours are taken before any product, and the three terms of every field cost two
// additions and two fused multiply-adds a pair.  For Q = rho, Q u is the momentum itself, an
// input: there the pair's term is (rho u+ - rho u-) + u (Q+ - Q-) + Q (u+ - u-), in which u's
// rounding enters once (in the bracket, where Q u is formed from u, twice).  Every sum goes
// straight into the residual (the weights hold the coefficients), so a direction ends
// without a combining step: 38 operations a pair, where separate sums of the derivatives of
// Q, Q u, u, p, theta and V took 41 a pair and 27 a direction.  The factor -2 is exact and
// saves a second set of weights.  RMS error against 113-bit arithmetic over that of those
// separate sums, orders 2 to 12, both types: mass 0.76 to 0.86, momentum 0.60 to 0.81,
// energy 0.64 to 0.70; with the bracket in the mass row, too, u = m rr and p from the internal
// energy: 1.73 to 1.97, 1.00 to 1.02, 0.85 to 0.92.  The difference costs 3 to 4 % of a launch
// at FP64 order 4 (512^3), 3 % at order 8, 5 to 6 % at order 12 and 1 % at FP32 order 4.
template <typename T, bool PLAIN>
struct ResidualSums {
    T Rr, R0, R1, R2, RE;
    // the five sums so far, handed from the x and y sums to the z sums
    __device__ __forceinline__ void get(T (&p)[5]) const {
        p[0] = Rr;
        p[1] = R0;
        p[2] = R1;
        p[3] = R2;
        p[4] = RE;
    }
    __device__ __forceinline__ void set(const T (&p)[5]) {
        Rr = p[0];
        R0 = p[1];
        R1 = p[2];
        R2 = p[3];
        RE = p[4];
    }
    __device__ __forceinline__ void begin() {}
    template <int d>
    __device__ __forceinline__ void end(const PF<T>&, const BoxConst<T>&) {}
    // the centre point's part of the viscous terms
    __device__ __forceinline__ void start(const PF<T>& s, const BoxConst<T>& c) {
        Rr = RE = 0;
        R0 = c.v0[0] * s.u0;
        R1 = c.v0[1] * s.u1;
        R2 = c.v0[2] * s.u2;
    }
    // Adds the pair a = +m, b = -m along axis d (mi = m - 1); s is the centre point.
    template <int d>
    __device__ __forceinline__ void add(const PF<T>& s, const PF<T>& a, T Wa, T Ga, const PF<T>& b, T Wb, T Gb,
                                        const BoxConst<T>& c, int mi) {
        const T uc = d == 0 ? s.u0 : (d == 1 ? s.u1 : s.u2);
        const T ua = d == 0 ? a.u0 : (d == 1 ? a.u1 : a.u2);
        const T ub = d == 0 ? b.u0 : (d == 1 ? b.u1 : b.u2);
        const T w = c.da[d][mi], v = c.v2[d][mi], vn = c.v2n[d][mi];
        const T ma = d == 0 ? a.m0 : (d == 1 ? a.m1 : a.m2);
        const T mb = d == 0 ? b.m0 : (d == 1 ? b.m1 : b.m2);
        const T du = ua - ub, wd = w * du, ws = w * (uc + ub);
        auto conv = [&](T qc, T qa, T qb, T r) { return fmaT(qa - qb, ws, fmaT(qc + qa, wd, r)); };
        Rr = fmaT(w, fmaT(s.rho, du, fmaT(uc, a.rho - b.rho, ma - mb)), Rr);
        R0 = conv(s.m0, a.m0, b.m0, R0);
        R1 = conv(s.m1, a.m1, b.m1, R1);
        R2 = conv(s.m2, a.m2, b.m2, R2);
        RE = conv(s.E, a.E, b.E, RE);
        T& Rd = d == 0 ? R0 : (d == 1 ? R1 : R2);
        Rd = fmaT(w, Ga - Gb, Rd);
        RE = fmaT(w, Wb - Wa, RE);
        R0 = fmaT(d == 0 ? vn : v, a.u0 + b.u0, R0);
        R1 = fmaT(d == 1 ? vn : v, a.u1 + b.u1, R1);
        R2 = fmaT(d == 2 ? vn : v, a.u2 + b.u2, R2);
        RE = fmaT(v, fmaT(T(-2), s.Th, a.Th + b.Th), RE);
    }
    // dq/dt of the five fields
    __device__ __forceinline__ void result(T (&R)[5]) const {
        R[0] = T(-0.5) * Rr;
        R[1] = T(-0.5) * R0;
        R[2] = T(-0.5) * R1;
        R[3] = T(-0.5) * R2;
        R[4] = T(-0.5) * RE;
    }
};

// The plain formulation: accumulates, for one direction d, the derivative sums of the
// residual from a neighbour pair (a = +m, b = -m) with weights w (first) and w2 (second).
template <typename T>
struct DirSums {
    T dRho, dM0, dM1, dM2, dF0, dF1, dF2, dE, dH, dU, dTh, d2U0, d2U1, d2U2, d2T;
    __device__ __forceinline__ void zero() {
        dRho = dM0 = dM1 = dM2 = dF0 = dF1 = dF2 = dE = dH = dU = dTh = 0;
        d2U0 = d2U1 = d2U2 = d2T = 0;
    }
    // d is the direction (0, 1, 2): selects u_d and which momentum gets 2p.
    template <int d>
    __device__ __forceinline__ void add(const PF<T>& a, T Va, T Tha, const PF<T>& b, T Vb, T Thb, T w, T w2) {
        const T ua = d == 0 ? a.u0 : (d == 1 ? a.u1 : a.u2);
        const T ub = d == 0 ? b.u0 : (d == 1 ? b.u1 : b.u2);
        dRho = fmaT(w, a.rho - b.rho, dRho);
        dM0 = fmaT(w, a.m0 - b.m0, dM0);
        dM1 = fmaT(w, a.m1 - b.m1, dM1);
        dM2 = fmaT(w, a.m2 - b.m2, dM2);
        // momentum fluxes rho u_i u_d (+ 2p for i = d): differences a - b
        const T pa2 = T(2) * (a.pk - b.pk);
        const T f0 = d == 0 ? fmaT(a.m0, ua, pa2 - b.m0 * ub) : fmaT(a.m0, ua, -(b.m0 * ub));
        const T f1 = d == 1 ? fmaT(a.m1, ua, pa2 - b.m1 * ub) : fmaT(a.m1, ua, -(b.m1 * ub));
        const T f2 = d == 2 ? fmaT(a.m2, ua, pa2 - b.m2 * ub) : fmaT(a.m2, ua, -(b.m2 * ub));
        dF0 = fmaT(w, f0, dF0);
        dF1 = fmaT(w, f1, dF1);
        dF2 = fmaT(w, f2, dF2);
        dE = fmaT(w, a.E - b.E, dE);
        // energy flux (rho E + 2p) u_d - 2 V_d: difference a - b
        const T hb = fmaT(fmaT(T(2), b.pk, b.E), ub, T(-2) * Vb);
        const T fh = fmaT(fmaT(T(2), a.pk, a.E), ua, fmaT(T(-2), Va, -hb));
        dH = fmaT(w, fh, dH);
        dU = fmaT(w, ua - ub, dU);
        dTh = fmaT(w, Tha - Thb, dTh);
        d2U0 = fmaT(w2, a.u0 + b.u0, d2U0);
        d2U1 = fmaT(w2, a.u1 + b.u1, d2U1);
        d2U2 = fmaT(w2, a.u2 + b.u2, d2U2);
        d2T = fmaT(w2, a.Th + b.Th, d2T);
    }
    // Adds this direction's part of the residual (paper eq. mass, momentum,
    // energy in the skew-symmetric form, regrouped by linearity) at point s.
    template <int d>
    __device__ __forceinline__ void finish(const PF<T>& s, T c0, const BoxConst<T>& c, T& Rr, T& R0, T& R1, T& R2,
                                           T& RE) {
        const T ud = d == 0 ? s.u0 : (d == 1 ? s.u1 : s.u2);
        const T e0 = fmaT(c0, s.u0, d2U0);
        const T e1 = fmaT(c0, s.u1, d2U1);
        const T e2 = fmaT(c0, s.u2, d2U2);
        const T eT = fmaT(c0, s.Th, d2T);
        const T dMd = d == 0 ? dM0 : (d == 1 ? dM1 : dM2);
        const T h = T(-0.5);
        Rr = fmaT(h, dMd + fmaT(ud, dRho, s.rho * dU), Rr);
        R0 = fmaT(c.inv_Re, e0, fmaT(h, dF0 + fmaT(ud, dM0, s.m0 * dU), R0));
        R1 = fmaT(c.inv_Re, e1, fmaT(h, dF1 + fmaT(ud, dM1, s.m1 * dU), R1));
        R2 = fmaT(c.inv_Re, e2, fmaT(h, dF2 + fmaT(ud, dM2, s.m2 * dU), R2));
        const T ed = d == 0 ? e0 : (d == 1 ? e1 : e2);
        if (d == 0) R0 = fmaT(c.inv_3Re, ed + dTh, R0);
        if (d == 1) R1 = fmaT(c.inv_3Re, ed + dTh, R1);
        if (d == 2) R2 = fmaT(c.inv_3Re, ed + dTh, R2);
        RE = fmaT(c.kappa, eT, fmaT(h, dH + fmaT(ud, dE, s.E * dU), RE));
    }
};

template <typename T>
struct ResidualSums<T, true> {
    T Rr, R0, R1, R2, RE;
    DirSums<T> ds;
    __device__ __forceinline__ void get(T (&p)[5]) const {
        p[0] = Rr;
        p[1] = R0;
        p[2] = R1;
        p[3] = R2;
        p[4] = RE;
    }
    __device__ __forceinline__ void set(const T (&p)[5]) {
        Rr = p[0];
        R0 = p[1];
        R1 = p[2];
        R2 = p[3];
        RE = p[4];
    }
    __device__ __forceinline__ void start(const PF<T>&, const BoxConst<T>&) { Rr = R0 = R1 = R2 = RE = 0; }
    __device__ __forceinline__ void begin() { ds.zero(); }
    template <int d>
    __device__ __forceinline__ void add(const PF<T>&, const PF<T>& a, T Va, T Tha, const PF<T>& b, T Vb, T Thb,
                                        const BoxConst<T>& c, int mi) {
        ds.template add<d>(a, Va, Tha, b, Vb, Thb, c.da[d][mi], c.d2c[d][mi]);
    }
    template <int d>
    __device__ __forceinline__ void end(const PF<T>& s, const BoxConst<T>& c) {
        ds.template finish<d>(s, c.d2c0[d], c, Rr, R0, R1, R2, RE);
    }
    __device__ __forceinline__ void result(T (&R)[5]) const {
        R[0] = Rr;
        R[1] = R0;
        R[2] = R1;
        R[3] = R2;
        R[4] = RE;
    }
};

// The scheduler keeps to one neighbour pair of the sums at a time.  Left alone, in FP64 it
// requests every pair's LDS reads first, and the threads of fused_stage_body spill 27 to 92
// registers (their window takes about 130 of 256); the plane wavefronts of the split form
// spill none either way, but their residual alone takes 545 us instead of 527 (256^3, order 4).
__device__ __forceinline__ void pair_fence() {
    __builtin_amdgcn_sched_barrier(0x100);   // LDS reads may cross
}

// One workgroup = one (x, y) tile and one z-chunk [z0, z0 + zc).
// PRE: whether the state of the entering plane and of the u-ring point is
// requested one iteration ahead (1) or in the iteration itself (0).  RT = 1
// rotates the register window instead of shifting it (for windows of at most 7
// planes).
// clos (may be null): a closure term with the state's planar layout, added to
// the residual when *cflag != 0.
template <typename T, int R, int TX, int TY, int MODE, int PRE, int RT, int SYM, int DB, int ZL>
__device__ __forceinline__ void fused_stage_body(const T* __restrict__ q, T* __restrict__ dq, T* __restrict__ out,
                                                 const BoxConst<T>& c, int x0, int y0, int z0, int zc, T dt, T A,
                                                 T B, const T* __restrict__ clos, const int* __restrict__ cflag) {
    using S = FusedShape<R, TX, TY>;
    constexpr bool PL = kPlain<T, MODE>;
    constexpr int NP = DB ? 3 : 2;     // buffers of the gradient plane's point fields
    constexpr int NW = DB ? 2 : 1;     // buffers of its nested pairs
    __shared__ T s_u[NP][3][S::BY2][S::BX2];
    __shared__ T s_pl[NP][kPlFields<T, PL>][S::BY1][S::BX1];
    // FP64: rho u_0 of the tile's rows and rho u_1 of its columns, with their R-ring
    __shared__ T s_mx[kMomentumInLds<T> ? 1 : NP][kMomentumInLds<T> ? 1 : TY][kMomentumInLds<T> ? 1 : TX + 2 * R];
    __shared__ T s_my[kMomentumInLds<T> ? 1 : NP][kMomentumInLds<T> ? 1 : TY + 2 * R][kMomentumInLds<T> ? 1 : TX];
    // (W_x, G_x, W_y, G_y) of a gradient plane over the tile and its R-ring
    __shared__ T s_xy[NW][4][S::BY1][S::BX1];
    // (W_z, G_z) of the last 2R+1 gradient planes over the tile, indexed by iteration
    __shared__ T s_az[2 * R + 1][2][TY][TX];
    // ZL: the point fields of the R planes below the output plane (own column,
    // stored when a plane leaves the centre of the window) are kept in LDS
    // instead of the register window, which then needs 2R + 1 live planes.
    __shared__ T s_zt[ZL ? R : 1][ZL ? kZtFields : 1][ZL ? TY : 1][ZL ? TX : 1];

    const int nx = c.n[0], ny = c.n[1], nz = c.n[2];
    const int64_t P = c.P;
    const int64_t plane = (int64_t)nx * ny;
    const int tid = threadIdx.x;
    constexpr bool DQ = MODE == kModeStage2 || MODE == kModeStage3;

    // ---- column role and coordinates ----
    int cx = 0, cy = 0;
    const bool e1 = tid < S::NE1;
    const bool interior = __builtin_amdgcn_readfirstlane(tid) < S::NI;   // whole wavefronts
    if (tid < S::NI) {
        cx = tid % TX;
        cy = tid / TX;
    } else if (tid < S::NI + S::NHX) {
        const int t = tid - S::NI;
        const int side = t / (R * TY);
        const int t2 = t % (R * TY);
        cy = t2 / R;
        const int k = t2 % R;
        cx = side ? TX + k : -R + k;
    } else if (tid < S::NE1) {
        const int t = tid - S::NI - S::NHX;
        const int side = t / (R * TX);
        const int t2 = t % (R * TX);
        const int k = t2 / TX;
        cx = t2 % TX;
        cy = side ? TY + k : -R + k;
    }
    // Periodic axes wrap; symmetry axes mirror, and a mirrored column carries the
    // sign-bit mask of the momentum component normal to that boundary.
    // SYM = 0 compiles the periodic case only (no masks, no sign flips).
    const int symx = SYM ? c.sym[0] : 0, symy = SYM ? c.sym[1] : 0, symz = SYM ? c.sym[2] : 0;
    unsigned fcx, fcy;
    const int64_t col = (int64_t)fold_index(y0 + cy, ny, symy, fcy) * nx + fold_index(x0 + cx, nx, symx, fcx);
    const bool store = interior && (x0 + cx < nx) && (y0 + cy < ny);

    // u-only ring point of this thread (if any): E2 minus E1.
    int ox = 0, oy = 0;
    const bool has_out = tid < S::NOUT;
    if (has_out) {
        int t = tid;
        if (t < 2 * R * TY) {                       // left / right, interior rows
            const int side = t / (R * TY);
            const int t2 = t % (R * TY);
            oy = t2 / R;
            const int k = t2 % R;
            ox = side ? TX + R + k : -2 * R + k;
        } else if ((t -= 2 * R * TY) < 2 * R * TX) {  // bottom / top, interior columns
            const int side = t / (R * TX);
            const int t2 = t % (R * TX);
            const int k = t2 / TX;
            ox = t2 % TX;
            oy = side ? TY + R + k : -2 * R + k;
        } else {                                    // the four R x R corners
            t -= 2 * R * TX;
            const int corner = t / (R * R);
            const int t2 = t % (R * R);
            const int ky = t2 / R, kx = t2 % R;
            ox = (corner & 1) ? TX + kx : -R + kx;
            oy = (corner & 2) ? TY + ky : -R + ky;
        }
    }
    unsigned fox, foy;
    const int64_t ocol = (int64_t)fold_index(y0 + oy, ny, symy, foy) * nx + fold_index(x0 + ox, nx, symx, fox);

    // ---- register windows ----
    constexpr int W = 3 * R + 1;
    constexpr bool ROT = RT && W <= 7;  // rotate instead of shifting (code size grows W-fold)
    PF<T> Qb[W];                  // point fields, planes L-3R .. L (logical index 3R = newest)
#pragma unroll
    for (int s = 0; s <= 3 * R; ++s) Qb[s] = PF<T>{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    // x/y sums waiting for their z sums: planes o .. o + NQ - 1
    constexpr int NQ = DB ? R - 1 : R;
    T part[NQ > 0 ? NQ : 1][5];
#pragma unroll
    for (int k = 0; k < NQ; ++k)
#pragma unroll
        for (int f = 0; f < 5; ++f) part[k][f] = 0;

    const int iters = zc + 4 * R;
    // With PRE = 1 the loads of iteration it+1 are issued before the work of
    // iteration it starts, and consumed one iteration later.
    T pq0 = 0, pq1 = 0, pq2 = 0, pq3 = 0, pq4 = 0;   // next q (own column)
    T pr0 = 1, pr1 = 0, pr2 = 0, pr3 = 0;            // next ring point (rho, rho u_i)
    T pd[5] = {0, 0, 0, 0, 0};                       // next output point's dq
    // byte offset of the output column from the tile's first column; lanes without one
    // drop their stores.  Rows so long that a tile passes the descriptor's size take
    // plain stores instead.
    const bool wide = (int64_t)TY * nx * (int64_t)sizeof(T) >= kBufferBytes;
    const int soff = store && !wide ? (cy * nx + cx) * (int)sizeof(T) : kDropOff;
    const int64_t dcol = store ? col : (int64_t)y0 * nx + x0;   // lanes without an output read the tile's first column
    // Sign-bit masks of the z-momentum of the planes just requested (mirror
    // images beyond a z symmetry boundary).  The loaded values stay untouched
    // until they are used, so a prefetch never waits for its data.
    unsigned pqz = 0u, prz = 0u;
    // planes stay within [-2R, nz + 2R): one mirror or wrap at most.  Every lane
    // loads in every iteration, from an in-range point (a lane without a column
    // reads the tile's first column; its values are unused).
    auto issue = [&](int it) {
        const int L = z0 - 2 * R + it;
        {
            const T* b = q + (int64_t)map_index(L, nz, symz, pqz) * plane + col;
            pq0 = b[0];
            pq1 = b[P];
            pq2 = b[2 * P];
            pq3 = b[3 * P];
            pq4 = b[4 * P];
        }
        {
            // the ring plane L - R is needed from the first gradient plane on
            const T* b = q + (int64_t)map_index(it >= 2 * R ? L - R : L, nz, symz, prz) * plane + ocol;
            pr0 = b[0];
            pr1 = b[P];
            pr2 = b[2 * P];
            pr3 = b[3 * P];
        }
        if constexpr (DQ) {
            const T* b = dq + (int64_t)(z0 + max(it - 4 * R, 0)) * plane + dcol;
#pragma unroll
            for (int f = 0; f < 5; ++f) pd[f] = __builtin_nontemporal_load(&b[f * P]);
        }
    };
    if (PRE > 0) issue(0);
    // One z-iteration.  With ROT the window is never shifted: logical plane k of
    // the window lives in register slot (k + PH) % W, and the loop is unrolled W
    // times so every slot index is a compile-time constant.
    auto body = [&](auto ph, const int it) {
        constexpr int PH = decltype(ph)::value;
        auto slot = [](int k) { return ROT ? (k + PH) % W : k; };
            const int L = z0 - 2 * R + it;           // plane loaded this iteration
            const int bp = it % NP;                  // LDS buffer of this iteration's gradient plane
            if (PRE == 0) issue(it);
            const T cq0 = pq0, cq1 = flip_sign(pq1, fcx), cq2 = flip_sign(pq2, fcy), cq3 = flip_sign(pq3, pqz),
                    cq4 = pq4;
            const T cr0 = pr0, cr1 = flip_sign(pr1, fox), cr2 = flip_sign(pr2, foy), cr3 = flip_sign(pr3, prz);
            T cd[5];
#pragma unroll
            for (int f = 0; f < 5; ++f) cd[f] = pd[f];
            if (PRE > 0 && it + 1 < iters) issue(it + 1);
            __builtin_amdgcn_sched_barrier(0);
            // 1. plane L enters the window
            if (e1) {
                const PF<T> f = make_pf<T, kPlain<T, MODE>>(cq0, cq1, cq2, cq3, cq4, c);
                if (!ROT) {
    #pragma unroll
                    for (int s = 0; s < 3 * R; ++s) Qb[slot(s)] = Qb[slot(s + 1)];
                }
                Qb[slot(3 * R)] = f;
            }
            const bool do_grad = it >= 2 * R;
            const bool do_out = it >= 4 * R;
            // LDS plane of the gradient plane a = L - R
            if (do_grad) {
                if (e1) {
                    const PF<T>& f = Qb[slot(2 * R)];
                    s_u[bp][0][cy + 2 * R][cx + 2 * R] = f.u0;
                    s_u[bp][1][cy + 2 * R][cx + 2 * R] = f.u1;
                    s_u[bp][2][cy + 2 * R][cx + 2 * R] = f.u2;
                    s_pl[bp][0][cy + R][cx + R] = f.rho;
                    s_pl[bp][1][cy + R][cx + R] = f.E;
                    s_pl[bp][2][cy + R][cx + R] = f.Th;
                    if constexpr (kMomentumInLds<T>) {
                        s_pl[bp][3][cy + R][cx + R] = f.m0;
                        s_pl[bp][4][cy + R][cx + R] = f.m1;
                        s_pl[bp][5][cy + R][cx + R] = f.m2;
                    } else {
                        if (cy >= 0 && cy < TY) s_mx[bp][cy][cx + R] = f.m0;
                        if (cx >= 0 && cx < TX) s_my[bp][cy + R][cx] = f.m1;
                    }
                    if constexpr (PL) s_pl[bp][kPlFields<T, PL> - 1][cy + R][cx + R] = with_pressure<PL>(f, c).pk;
                }
                if (has_out) {
                    const T rr = fast_recip(cr0);
                    s_u[bp][0][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr1, cr0, rr);
                    s_u[bp][1][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr2, cr0, rr);
                    s_u[bp][2][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr3, cr0, rr);
                }
            }
            __syncthreads();
            // 2. velocity gradient at plane a -> nested fields
            if (do_grad && e1) {
                T g[3][3];
    #pragma unroll
                for (int b = 0; b < 3; ++b) {
                    T sx = 0, sy = 0, sz = 0;
    #pragma unroll
                    for (int m = 1; m <= R; ++m) {
                        sx = fmaT(c.da[0][m - 1],
                                  s_u[bp][b][cy + 2 * R][cx + 2 * R + m] - s_u[bp][b][cy + 2 * R][cx + 2 * R - m], sx);
                        sy = fmaT(c.da[1][m - 1],
                                  s_u[bp][b][cy + 2 * R + m][cx + 2 * R] - s_u[bp][b][cy + 2 * R - m][cx + 2 * R], sy);
                        const T up = b == 0 ? Qb[slot(2 * R + m)].u0 : (b == 1 ? Qb[slot(2 * R + m)].u1 : Qb[slot(2 * R + m)].u2);
                        const T um = b == 0 ? Qb[slot(2 * R - m)].u0 : (b == 1 ? Qb[slot(2 * R - m)].u1 : Qb[slot(2 * R - m)].u2);
                        sz = fmaT(c.da[2][m - 1], up - um, sz);
                    }
                    g[b][0] = sx;
                    g[b][1] = sy;
                    g[b][2] = sz;
                }
                const PF<T>& f = Qb[slot(2 * R)];
                T V[3], t[3];
                nested_terms<PL>(g, f.u0, f.u1, f.u2, c, V, t);
                T (&w)[4][S::BY1][S::BX1] = s_xy[it % NW];
                w[0][cy + R][cx + R] = nested_W<PL>(V[0], f, f.u0, c);
                w[1][cy + R][cx + R] = nested_G<PL>(t[0], f, c);
                w[2][cy + R][cx + R] = nested_W<PL>(V[1], f, f.u1, c);
                w[3][cy + R][cx + R] = nested_G<PL>(t[1], f, c);
                if (interior) {
                    const int sz = it % (2 * R + 1);
                    // read back only by this thread
                    s_az[sz][0][cy][cx] = nested_W<PL>(V[2], f, f.u2, c);
                    s_az[sz][1][cy][cx] = nested_G<PL>(t[2], f, c);
                }
            }
            constexpr int NST = (MODE == kModeRHS || MODE == kModeStage3) ? 5 : 10;
            // 3. x and y sums at plane b = a (DB = 0) or a - 1 (DB = 1)
            auto sums_xy = [&](T (&to)[5]) {
                const int pb = (it - DB) % NP, wb = (it - DB) % NW;
                const int ly = cy + R, lx = cx + R;
                const PF<T>& s = Qb[slot(2 * R - DB)];
                const PF<T> sx = point_along<0>(s), sy = point_along<1>(s);
                auto ld = [&](auto axis, int yy, int xx) {   // a neighbour along the axis
                    constexpr int D = decltype(axis)::value;
                    PF<T> f;
                    f.rho = s_pl[pb][0][yy][xx];
                    f.E = s_pl[pb][1][yy][xx];
                    f.pk = 0;
                    if constexpr (PL) f.pk = s_pl[pb][kPlFields<T, PL> - 1][yy][xx];
                    f.Th = s_pl[pb][2][yy][xx];
                    f.u0 = s_u[pb][0][yy + R][xx + R];
                    f.u1 = s_u[pb][1][yy + R][xx + R];
                    f.u2 = s_u[pb][2][yy + R][xx + R];
                    if constexpr (kMomentumInLds<T>) {
                        f.m0 = s_pl[pb][3][yy][xx];
                        f.m1 = s_pl[pb][4][yy][xx];
                        f.m2 = s_pl[pb][5][yy][xx];
                    } else {
                        if constexpr (D == 0) f.m0 = s_mx[pb][yy - R][xx];
                        else f.m1 = s_my[pb][yy][xx - R];
                    }
                    return point_along<D>(f);
                };
                constexpr std::integral_constant<int, 0> along_x{};
                constexpr std::integral_constant<int, 1> along_y{};
                T (&w)[4][S::BY1][S::BX1] = s_xy[wb];
                ResidualSums<T, PL> rs;
                rs.start(s, c);
                rs.begin();
    #pragma unroll
                for (int m = 1; m <= R; ++m) {
                    pair_fence();
                    rs.template add<0>(sx, ld(along_x, ly, lx + m), w[0][ly][lx + m], w[1][ly][lx + m],
                                       ld(along_x, ly, lx - m), w[0][ly][lx - m], w[1][ly][lx - m], c, m - 1);
                }
                rs.template end<0>(sx, c);
                rs.begin();
    #pragma unroll
                for (int m = 1; m <= R; ++m) {
                    pair_fence();
                    rs.template add<1>(sy, ld(along_y, ly + m, lx), w[2][ly + m][lx], w[3][ly + m][lx],
                                       ld(along_y, ly - m, lx), w[2][ly - m][lx], w[3][ly - m][lx], c, m - 1);
                }
                rs.template end<1>(sy, c);
                rs.get(to);
            };
            const bool xy_here = it >= 3 * R + DB && it < zc + 3 * R + DB && interior;
            if constexpr (NQ == 0) {
                if (xy_here) sums_xy(part[0]);
            }
            // 4. z sums and RK update at the output plane o = L - 2R.
            // The counter a wave waits on for its loads also counts its stores, in order.
            // This step's stores come after the next plane's loads; with as many stores on
            // every path (dropped ones where there is no output plane, and for lanes of a
            // ragged tile) the wait for those loads leaves the stores in flight.
            T dn[5], qn[5];
            if (do_out && interior) {
                const PF<T>& s = Qb[slot(R)];
                const PF<T> sz = z_point<T, R>(s);
                auto below = [&](int m) -> PF<T> {         // point fields of plane o - m
                    if constexpr (ZL) {
                        const int k = (it - m) % R;
                        PF<T> f;
                        f.rho = s_zt[k][0][cy][cx];
                        f.m0 = s_zt[k][1][cy][cx];
                        f.m1 = s_zt[k][2][cy][cx];
                        f.m2 = s_zt[k][3][cy][cx];
                        f.E = s_zt[k][4][cy][cx];
                        f.u0 = s_zt[k][5][cy][cx];
                        f.u1 = s_zt[k][6][cy][cx];
                        f.u2 = s_zt[k][7][cy][cx];
                        f.pk = 0;
                        f.Th = s_zt[k][8][cy][cx];
                        return f;
                    } else {
                        return Qb[slot(R - m)];
                    }
                };
                ResidualSums<T, PL> rs;
                rs.set(part[0]);
                rs.begin();
    #pragma unroll
                for (int m = 1; m <= R; ++m) {
                    pair_fence();
                    rs.template add<2>(sz, z_point<T, R>(with_pressure<PL>(Qb[slot(R + m)], c)),
                                       s_az[(it + m - R) % (2 * R + 1)][0][cy][cx],
                                       s_az[(it + m - R) % (2 * R + 1)][1][cy][cx],
                                       z_point<T, R>(with_pressure<PL>(below(m), c)),
                                       s_az[(it - m - R) % (2 * R + 1)][0][cy][cx],
                                       s_az[(it - m - R) % (2 * R + 1)][1][cy][cx], c, m - 1);
                }
                rs.template end<2>(sz, c);
                T Rv[5];
                rs.result(Rv);
                if (clos != nullptr && __builtin_amdgcn_readfirstlane(cflag[0]) != 0) {   // a uniform branch
                    const int64_t idx = (int64_t)(L - 2 * R) * plane + col;
    #pragma unroll
                    for (int f = 0; f < 5; ++f) Rv[f] += clos[f * P + idx];
                }
                const T qv[5] = {s.rho, s.m0, s.m1, s.m2, s.E};
    #pragma unroll
                for (int f = 0; f < 5; ++f) {
                    dn[f] = MODE == kModeRHS ? Rv[f] : dt * Rv[f];
                    if (DQ) dn[f] = fmaT(A, cd[f], dn[f]);
                    if (MODE != kModeRHS) qn[f] = fmaT(B, dn[f], qv[f]);
                }
            }
            // dq and the new state are streamed: nothing reads them again in
            // this launch, so they need not displace the state in L2
            {
                if (wide && do_out && store) {
                    const int64_t idx = (int64_t)(L - 2 * R) * plane + col;
    #pragma unroll
                    for (int f = 0; f < 5; ++f) {
                        if (MODE == kModeStage1 || MODE == kModeStage2) dq[f * P + idx] = dn[f];
                        out[f * P + idx] = MODE == kModeRHS ? dn[f] : qn[f];
                    }
                }
                const int off = do_out ? soff : kDropOff;
                const int64_t org = (int64_t)(do_out ? L - 2 * R : z0) * plane + (int64_t)y0 * nx + x0;
    #pragma unroll
                for (int f = 0; f < 5; ++f) {
                    if (MODE == kModeRHS) {
                        buffer_store_nt(dn[f], out + f * P + org, off);
                    } else {
                        if (MODE != kModeStage3) buffer_store_nt(dn[f], dq + f * P + org, off);
                        buffer_store_nt(qn[f], out + f * P + org, off);
                    }
                }
            }
            if (!DB) __syncthreads();
            if constexpr (NQ > 0) {
#pragma unroll
                for (int k = 0; k + 1 < NQ; ++k)
#pragma unroll
                    for (int f = 0; f < 5; ++f) part[k][f] = part[k + 1][f];
                if (xy_here) sums_xy(part[NQ - 1]);
            }
            if constexpr (ZL) {
                // plane o leaves the centre of the window; only this thread reads it
                // back, as plane o' - m of the next R output planes
                if (interior && it >= 2 * R) {
                    const PF<T>& f = Qb[slot(R)];
                    const int k = it % R;
                    s_zt[k][0][cy][cx] = f.rho;
                    s_zt[k][1][cy][cx] = f.m0;
                    s_zt[k][2][cy][cx] = f.m1;
                    s_zt[k][3][cy][cx] = f.m2;
                    s_zt[k][4][cy][cx] = f.E;
                    s_zt[k][5][cy][cx] = f.u0;
                    s_zt[k][6][cy][cx] = f.u1;
                    s_zt[k][7][cy][cx] = f.u2;
                    s_zt[k][8][cy][cx] = f.Th;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (ROT) {
        for (int it0 = 0; it0 < iters; it0 += W) {
            static_for<W>([&](auto ph) {
                const int it = it0 + decltype(ph)::value;
                if (it < iters) body(ph, it);
            });
        }
    } else {
        for (int it = 0; it < iters; ++it) body(std::integral_constant<int, 0>{}, it);
    }
}

// The same tile and pipeline with the work of a plane split between two kinds of
// wavefronts (schedule 2).  NI / 64 "column" wavefronts own the tile's columns: state
// loads, register window, gradient, z sums, update and stores.  As many "plane"
// wavefronts work from LDS: they load and convert the R-ring columns and the 2R-ring of
// u, form the ring's gradients, and sum x and y on plane a - 1 for the column wavefronts,
// which read the five partial residuals one barrier later.  A SIMD then runs one wavefront
// of each kind: the VALU and LDS work of a plane, which one wavefront could only do in
// turn, overlap, and the ring's work is spread over all SIMDs.
// What bounds it: at 512^3, FP64, order 4 a launch moved 20.7 GB at 3.5 TB/s (a copy
// reaches 4.6) while neither VALU (34 %) nor LDS (44 %) was busy: with schedule 1 a SIMD
// had one output wavefront, whose LDS reads, arithmetic and waits for the next plane
// followed each other.  Per launch: 5.96 ms with the former sums and order of steps,
// 5.43 with the bracket sums, x and y summed on the gradient's LDS plane and the loads a
// full step ahead, 4.66 in this form (bare tile alone on the chip: 2.17 -> 1.92 us a
// plane, 2.24 in contention), 4.83 with the momentum along the axes in LDS (see
// ResidualSums).  FP32, order 6, 256^3: 823 -> 614 us.  FP32 at order 4
// stays with 32 x 16 tiles and schedule 1 (2.60 ms; 16 x 16 or 32 x 12 here 4.00, 2.98):
// it is bound by VALU issue, and there the larger tile has less ring work a point.
// One barrier a plane, as schedule 1: what is read between two barriers was written
// before the first.  (Step it: the planes of u and the point fields are written before
// barrier it; the nested pairs of plane a after it; x and y sums of a - 1 read the pairs
// written after barrier it - 1 and the point fields written before it; partial sums
// written after barrier it are read after it + R - 1.)  R >= 2: the output plane a - R
// needs its partial sums one barrier after step a - R + 1.
template <typename T, int R, int TX, int TY, bool PL>
struct SplitLds {
    using S = FusedShape<R, TX, TY>;
    T u[3][3][S::BY2][S::BX2];                    // three planes: a - 1, a and the next one
    T pl[3][kPlFields<T, PL>][S::BY1][S::BX1];
    // FP64: rho u_0 of the tile's rows, rho u_1 of its columns (rows of even length: with
    // these two 16 x 8 workgroups just fit a CU)
    T mx[kMomentumInLds<T> ? 1 : 3][kMomentumInLds<T> ? 1 : TY][kMomentumInLds<T> ? 1 : TX + 2 * R];
    T my[kMomentumInLds<T> ? 1 : 3][kMomentumInLds<T> ? 1 : TY + 2 * R][kMomentumInLds<T> ? 1 : TX];
    T xy[2][4][S::BY1][S::BX1];                   // (W_x, G_x, W_y, G_y) of planes a - 1, a
    T part[R][5][TY][TX];                         // partial residuals
};

// Velocity gradient at LDS position (cy, cx) of the tile, plane buffer u; the z
// derivative from the window, whose slot k planes above the gradient plane is w(k).
template <typename T, int R, typename LU, typename WIN>
__device__ __forceinline__ void plane_gradient(const LU& u, int yy, int xx, const WIN& w, const BoxConst<T>& c,
                                               T (&g)[3][3]) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        T sx = 0, sy = 0, sz = 0;
#pragma unroll
        for (int m = 1; m <= R; ++m) {
            sx = fmaT(c.da[0][m - 1], u[b][yy][xx + m] - u[b][yy][xx - m], sx);
            sy = fmaT(c.da[1][m - 1], u[b][yy + m][xx] - u[b][yy - m][xx], sy);
            const PF<T>&p = w(m), &n = w(-m);
            const T up = b == 0 ? p.u0 : (b == 1 ? p.u1 : p.u2);
            const T un = b == 0 ? n.u0 : (b == 1 ? n.u1 : n.u2);
            sz = fmaT(c.da[2][m - 1], up - un, sz);
        }
        g[b][0] = sx;
        g[b][1] = sy;
        g[b][2] = sz;
    }
}

template <typename T, int R, bool PL, typename LDS>
__device__ __forceinline__ void store_plane(LDS& lds, int bp, int yy, int xx, const PF<T>& f) {
    lds.u[bp][0][yy + 2 * R][xx + 2 * R] = f.u0;
    lds.u[bp][1][yy + 2 * R][xx + 2 * R] = f.u1;
    lds.u[bp][2][yy + 2 * R][xx + 2 * R] = f.u2;
    lds.pl[bp][0][yy + R][xx + R] = f.rho;
    lds.pl[bp][1][yy + R][xx + R] = f.E;
    lds.pl[bp][2][yy + R][xx + R] = f.Th;
    if constexpr (kMomentumInLds<T>) {
        lds.pl[bp][3][yy + R][xx + R] = f.m0;
        lds.pl[bp][4][yy + R][xx + R] = f.m1;
        lds.pl[bp][5][yy + R][xx + R] = f.m2;
    }
    if constexpr (PL) lds.pl[bp][kPlFields<T, PL> - 1][yy + R][xx + R] = f.pk;
}

// Runs body(phase, it) for it = 0 .. iters - 1, phase = it % W a constant: register slots
// indexed by it + k are then fixed registers.
template <int W, typename F>
__device__ __forceinline__ void rotating_loop(int iters, F&& body) {
    for (int it0 = 0; it0 < iters; it0 += W) {
        static_for<W>([&](auto ph) {
            const int it = it0 + decltype(ph)::value;
            if (it < iters) body(ph, it);
        });
    }
}

template <typename T, int R, int TX, int TY, int MODE, int SYM, bool PL>
__device__ __forceinline__ void split_columns(SplitLds<T, R, TX, TY, PL>& lds, const T* __restrict__ q, T* __restrict__ dq,
                                              T* __restrict__ out, const BoxConst<T>& c, int x0, int y0, int z0,
                                              int zc, T dt, T A, T B, const T* __restrict__ clos,
                                              const int* __restrict__ cflag) {
    const int nx = c.n[0], ny = c.n[1], nz = c.n[2];
    const int64_t P = c.P, plane = (int64_t)nx * ny;
    const int cx = threadIdx.x % TX, cy = threadIdx.x / TX;
    const int symx = SYM ? c.sym[0] : 0, symy = SYM ? c.sym[1] : 0, symz = SYM ? c.sym[2] : 0;
    unsigned fcx, fcy;
    const int64_t col = (int64_t)fold_index(y0 + cy, ny, symy, fcy) * nx + fold_index(x0 + cx, nx, symx, fcx);
    const bool store = (x0 + cx < nx) && (y0 + cy < ny);
    constexpr bool DQ = MODE == kModeStage2 || MODE == kModeStage3;
    // (see fused_stage_body)
    const bool wide = (int64_t)TY * nx * (int64_t)sizeof(T) >= kBufferBytes;
    const int soff = store && !wide ? (cy * nx + cx) * (int)sizeof(T) : kDropOff;
    const int64_t dcol = store ? col : (int64_t)y0 * nx + x0;
    constexpr int W = 3 * R + 1;
    PF<T> Qb[W];
#pragma unroll
    for (int s = 0; s < W; ++s) Qb[s] = PF<T>{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    T Wz[W], Gz[W];
#pragma unroll
    for (int s = 0; s < W; ++s) Wz[s] = Gz[s] = 0;
    const int iters = zc + 4 * R;
    T pq0, pq1, pq2, pq3, pq4, pd[5] = {0, 0, 0, 0, 0};
    unsigned pqz = 0u;
    auto issue = [&](int it) {
        const T* b = q + (int64_t)map_index(z0 - 2 * R + it, nz, symz, pqz) * plane + col;
        pq0 = b[0];
        pq1 = b[P];
        pq2 = b[2 * P];
        pq3 = b[3 * P];
        pq4 = b[4 * P];
        if constexpr (DQ) {
            const T* d = dq + (int64_t)(z0 + max(it - 4 * R, 0)) * plane + dcol;
#pragma unroll
            for (int f = 0; f < 5; ++f) pd[f] = __builtin_nontemporal_load(&d[f * P]);
        }
    };
    issue(0);
    rotating_loop<W>(iters, [&](auto ph, const int it) {
        constexpr int PH = decltype(ph)::value;
        auto slot = [](int k) { return (k + PH) % W; };
        const int L = z0 - 2 * R + it;
        const int bp = it % 3;
        const T cq0 = pq0, cq1 = flip_sign(pq1, fcx), cq2 = flip_sign(pq2, fcy), cq3 = flip_sign(pq3, pqz), cq4 = pq4;
        T cd[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) cd[f] = pd[f];
        if (it + 1 < iters) issue(it + 1);
        __builtin_amdgcn_sched_barrier(0);
        Qb[slot(3 * R)] = make_pf<T, kPlain<T, MODE>>(cq0, cq1, cq2, cq3, cq4, c);
        const bool do_grad = it >= 2 * R, do_out = it >= 4 * R;
        if (do_grad) {
            store_plane<T, R, PL>(lds, bp, cy, cx, Qb[slot(2 * R)]);
            if constexpr (!kMomentumInLds<T>) {
                lds.mx[bp][cy][cx + R] = Qb[slot(2 * R)].m0;
                lds.my[bp][cy + R][cx] = Qb[slot(2 * R)].m1;
            }
        }
        __syncthreads();
        if (do_grad) {
            T g[3][3], V[3], t[3];
            plane_gradient<T, R>(lds.u[bp], cy + 2 * R, cx + 2 * R,
                                 [&](int k) -> const PF<T>& { return Qb[slot(2 * R + k)]; }, c, g);
            const PF<T>& f = Qb[slot(2 * R)];
            nested_terms<PL>(g, f.u0, f.u1, f.u2, c, V, t);
            auto& w = lds.xy[it & 1];
            w[0][cy + R][cx + R] = nested_W<PL>(V[0], f, f.u0, c);
            w[1][cy + R][cx + R] = nested_G<PL>(t[0], f, c);
            w[2][cy + R][cx + R] = nested_W<PL>(V[1], f, f.u1, c);
            w[3][cy + R][cx + R] = nested_G<PL>(t[1], f, c);
            Wz[slot(2 * R)] = nested_W<PL>(V[2], f, f.u2, c);
            Gz[slot(2 * R)] = nested_G<PL>(t[2], f, c);
        }
        T dn[5], qn[5];
        if (do_out) {
            const PF<T>& s = Qb[slot(R)];
            ResidualSums<T, PL> rs;
            const auto& pp = lds.part[(it + 1) % R];
            rs.set({pp[0][cy][cx], pp[1][cy][cx], pp[2][cy][cx], pp[3][cy][cx], pp[4][cy][cx]});
            rs.begin();
#pragma unroll
            for (int m = 1; m <= R; ++m)
                rs.template add<2>(s, Qb[slot(R + m)], Wz[slot(R + m)],
                                   Gz[slot(R + m)], Qb[slot(R - m)],
                                   Wz[slot(R - m)],
                                   Gz[slot(R - m)], c, m - 1);
            rs.template end<2>(s, c);
            T Rv[5];
            rs.result(Rv);
            if (clos != nullptr && __builtin_amdgcn_readfirstlane(cflag[0]) != 0) {
                const int64_t idx = (int64_t)(L - 2 * R) * plane + col;
#pragma unroll
                for (int f = 0; f < 5; ++f) Rv[f] += clos[f * P + idx];
            }
            const T qv[5] = {s.rho, s.m0, s.m1, s.m2, s.E};
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                dn[f] = MODE == kModeRHS ? Rv[f] : dt * Rv[f];
                if (DQ) dn[f] = fmaT(A, cd[f], dn[f]);
                if (MODE != kModeRHS) qn[f] = fmaT(B, dn[f], qv[f]);
            }
        }
        if (wide && do_out && store) {
            const int64_t idx = (int64_t)(L - 2 * R) * plane + col;
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                if (MODE == kModeStage1 || MODE == kModeStage2) dq[f * P + idx] = dn[f];
                out[f * P + idx] = MODE == kModeRHS ? dn[f] : qn[f];
            }
        }
        const int off = do_out ? soff : kDropOff;
        const int64_t org = (int64_t)(do_out ? L - 2 * R : z0) * plane + (int64_t)y0 * nx + x0;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            if (MODE == kModeRHS) {
                buffer_store_nt(dn[f], out + f * P + org, off);
            } else {
                if (MODE != kModeStage3) buffer_store_nt(dn[f], dq + f * P + org, off);
                buffer_store_nt(qn[f], out + f * P + org, off);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

template <typename T, int R, int TX, int TY, int MODE, int SYM, bool PL>
__device__ __forceinline__ void split_planes(SplitLds<T, R, TX, TY, PL>& lds, const T* __restrict__ q,
                                             const BoxConst<T>& c, int x0, int y0, int z0, int zc) {
    using S = FusedShape<R, TX, TY>;
    static_assert(S::NHX + S::NHY <= S::NI && S::NOUT <= S::NI, "one ring column and one ring point per thread at most");
    const int nx = c.n[0], ny = c.n[1], nz = c.n[2];
    const int64_t P = c.P, plane = (int64_t)nx * ny;
    const int t = threadIdx.x - S::NI;
    const int cx = t % TX, cy = t / TX;     // the column whose x and y sums this thread forms
    const int symx = SYM ? c.sym[0] : 0, symy = SYM ? c.sym[1] : 0, symz = SYM ? c.sym[2] : 0;
    // R-ring column (threads 0 .. NHX + NHY - 1) and u-ring point (the last NOUT threads)
    const bool has_col = t < S::NHX + S::NHY, has_out = t >= S::NI - S::NOUT;
    int hx = 0, hy = 0, ox = 0, oy = 0;
    if (t < S::NHX) {
        const int side = t / (R * TY), r = t % (R * TY);
        hy = r / R;
        hx = side ? TX + r % R : -R + r % R;
    } else if (has_col) {
        const int e = t - S::NHX, side = e / (R * TX), r = e % (R * TX);
        hx = r % TX;
        hy = side ? TY + r / TX : -R + r / TX;
    }
    if (has_out) {
        int e = S::NI - 1 - t;
        if (e < 2 * R * TY) {                         // left / right, interior rows
            const int side = e / (R * TY), r = e % (R * TY);
            oy = r / R;
            ox = side ? TX + R + r % R : -2 * R + r % R;
        } else if ((e -= 2 * R * TY) < 2 * R * TX) {  // bottom / top, interior columns
            const int side = e / (R * TX), r = e % (R * TX);
            ox = r % TX;
            oy = side ? TY + R + r / TX : -2 * R + r / TX;
        } else {                                      // the four R x R corners
            e -= 2 * R * TX;
            const int corner = e / (R * R), r = e % (R * R);
            ox = (corner & 1) ? TX + r % R : -R + r % R;
            oy = (corner & 2) ? TY + r / R : -R + r / R;
        }
    }
    unsigned fhx, fhy, fox, foy;
    // a thread without a ring column or point reads the tile's first column
    const int64_t hcol = (int64_t)fold_index(y0 + hy, ny, symy, fhy) * nx + fold_index(x0 + hx, nx, symx, fhx);
    const int64_t ocol = (int64_t)fold_index(y0 + oy, ny, symy, foy) * nx + fold_index(x0 + ox, nx, symx, fox);
    // window of the ring column, planes L - 2R .. L (only what the gradient plane needs)
    constexpr int W = 3 * R + 1;
    PF<T> Hb[W];
#pragma unroll
    for (int s = 0; s < W; ++s) Hb[s] = PF<T>{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int iters = zc + 4 * R;
    T pq0, pq1, pq2, pq3, pq4, pr0, pr1, pr2, pr3;
    unsigned pqz = 0u, prz = 0u;
    auto issue = [&](int it) {
        const int L = z0 - 2 * R + it;
        const T* b = q + (int64_t)map_index(L, nz, symz, pqz) * plane + hcol;
        pq0 = b[0];
        pq1 = b[P];
        pq2 = b[2 * P];
        pq3 = b[3 * P];
        pq4 = b[4 * P];
        // the ring plane L - R is needed from the first gradient plane on
        const T* r = q + (int64_t)map_index(it >= 2 * R ? L - R : L, nz, symz, prz) * plane + ocol;
        pr0 = r[0];
        pr1 = r[P];
        pr2 = r[2 * P];
        pr3 = r[3 * P];
    };
    issue(0);
    rotating_loop<W>(iters, [&](auto ph, const int it) {
        constexpr int PH = decltype(ph)::value;
        auto slot = [](int k) { return (k + PH) % W; };
        const int bp = it % 3;
        const T cq0 = pq0, cq1 = flip_sign(pq1, fhx), cq2 = flip_sign(pq2, fhy), cq3 = flip_sign(pq3, pqz), cq4 = pq4;
        const T cr0 = pr0, cr1 = flip_sign(pr1, fox), cr2 = flip_sign(pr2, foy), cr3 = flip_sign(pr3, prz);
        if (it + 1 < iters) issue(it + 1);
        __builtin_amdgcn_sched_barrier(0);
        const bool do_grad = it >= 2 * R;
        if (has_col) {
            Hb[slot(3 * R)] = make_pf<T, kPlain<T, MODE>>(cq0, cq1, cq2, cq3, cq4, c);
            // FP64: the window holds one momentum component, along the ring column's axis
            if constexpr (!kMomentumInLds<T>) Hb[slot(3 * R)].m0 = t < S::NHX ? cq1 : cq2;
            if (do_grad) {
                store_plane<T, R, PL>(lds, bp, hy, hx, Hb[slot(2 * R)]);
                if constexpr (!kMomentumInLds<T>)
                    *(t < S::NHX ? &lds.mx[bp][hy][hx + R] : &lds.my[bp][hy + R][hx]) = Hb[slot(2 * R)].m0;
            }
        }
        if (do_grad && has_out) {
            const T rr = fast_recip(cr0);
            lds.u[bp][0][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr1, cr0, rr);
            lds.u[bp][1][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr2, cr0, rr);
            lds.u[bp][2][oy + 2 * R][ox + 2 * R] = velocity<PL>(cr3, cr0, rr);
        }
        __syncthreads();
        if (do_grad && has_col) {
            T g[3][3], V[3], tt[3];
            plane_gradient<T, R>(lds.u[bp], hy + 2 * R, hx + 2 * R,
                                 [&](int k) -> const PF<T>& { return Hb[slot(2 * R + k)]; }, c, g);
            const PF<T>& f = Hb[slot(2 * R)];
            nested_terms<PL>(g, f.u0, f.u1, f.u2, c, V, tt);
            auto& w = lds.xy[it & 1];
            w[0][hy + R][hx + R] = nested_W<PL>(V[0], f, f.u0, c);
            w[1][hy + R][hx + R] = nested_G<PL>(tt[0], f, c);
            w[2][hy + R][hx + R] = nested_W<PL>(V[1], f, f.u1, c);
            w[3][hy + R][hx + R] = nested_G<PL>(tt[1], f, c);
        }
        // x and y sums of plane a - 1
        if (it >= 3 * R + 1 && it < zc + 3 * R + 1) {
            const int pb = (it - 1) % 3;
            const auto& w = lds.xy[(it - 1) & 1];
            const int ly = cy + R, lx = cx + R;
            auto ld = [&](auto axis, int yy, int xx) {   // a point of the sums along the axis
                constexpr int D = decltype(axis)::value;
                PF<T> f;
                f.rho = lds.pl[pb][0][yy][xx];
                f.E = lds.pl[pb][1][yy][xx];
                f.pk = 0;
                if constexpr (PL) f.pk = lds.pl[pb][kPlFields<T, PL> - 1][yy][xx];
                f.Th = lds.pl[pb][2][yy][xx];
                f.u0 = lds.u[pb][0][yy + R][xx + R];
                f.u1 = lds.u[pb][1][yy + R][xx + R];
                f.u2 = lds.u[pb][2][yy + R][xx + R];
                if constexpr (kMomentumInLds<T>) {
                    f.m0 = lds.pl[pb][3][yy][xx];
                    f.m1 = lds.pl[pb][4][yy][xx];
                    f.m2 = lds.pl[pb][5][yy][xx];
                } else {
                    if constexpr (D == 0) f.m0 = lds.mx[pb][yy - R][xx];
                    else f.m1 = lds.my[pb][yy][xx - R];
                }
                return point_along<D>(f);
            };
            constexpr std::integral_constant<int, 0> along_x{};
            constexpr std::integral_constant<int, 1> along_y{};
            const PF<T> sx = ld(along_x, ly, lx);
            ResidualSums<T, PL> rs;
            rs.start(sx, c);
            rs.begin();
#pragma unroll
            for (int m = 1; m <= R; ++m) {
                pair_fence();
                rs.template add<0>(sx, ld(along_x, ly, lx + m), w[0][ly][lx + m], w[1][ly][lx + m],
                                   ld(along_x, ly, lx - m), w[0][ly][lx - m], w[1][ly][lx - m], c, m - 1);
            }
            rs.template end<0>(sx, c);
            const PF<T> sy = ld(along_y, ly, lx);
            rs.begin();
#pragma unroll
            for (int m = 1; m <= R; ++m) {
                pair_fence();
                rs.template add<1>(sy, ld(along_y, ly + m, lx), w[2][ly + m][lx], w[3][ly + m][lx],
                                   ld(along_y, ly - m, lx), w[2][ly - m][lx], w[3][ly - m][lx], c, m - 1);
            }
            rs.template end<1>(sy, c);
            auto& pp = lds.part[it % R];
            T sums[5];
            rs.get(sums);
#pragma unroll
            for (int f = 0; f < 5; ++f) pp[f][cy][cx] = sums[f];
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

// One periodic box of a launch: its constants, where its state starts in the
// packed buffers, its time step and its share of the launch grid.
template <typename T>
struct BoxInst {
    BoxConst<T> c;
    int64_t offset;    // element offset of the box's state in q, dq and out
    T dt;              // time step (multiplied by the launch's dt_scale)
    int tiles_x, tiles_y, zchunk;
    int first_wg;      // first logical workgroup of this box
    int num_wg;        // tiles_x * tiles_y * ceil(nz / zchunk)
    const T* closure;  // closure term of this box (planar, 5 fields) or null
    const int* cflag;  // the closure is added only while *cflag != 0
};

constexpr int kStripRows = 4;   // tile rows of a strip (see fused_stage_kernel)
constexpr int kXcdPiece = 16;   // workgroups of an ensemble dealt to an XCD at a time

// Threads of a workgroup: schedule 2 has as many plane threads as column threads.
template <int R, int TX, int TY, int DB>
constexpr int fused_threads() {
    return DB == 2 ? 2 * TX * TY : FusedShape<R, TX, TY>::NT;
}

// One launch covers `ninst` boxes (one for a single solver, many for an
// ensemble): a 1D grid whose logical workgroup ids are split between the boxes
// by first_wg.  Workgroups are handed to the 8 XCDs round-robin by id; the id is
// remapped so that each XCD (with its own L2) walks a contiguous run of
// neighbouring tiles, whose halos then hit in that L2.
// MINW: the fewest wavefronts per SIMD the register allocation must allow
// (2 caps a thread at 256 VGPRs, so two 4-wavefront workgroups share a CU).
// SYM: 1 for boxes with a symmetry axis, 0 for periodic boxes.
// DB: barrier schedule; ZL: lower planes of the window in LDS (see fused_stage_body).
template <typename T, int R, int TX, int TY, int MODE, int PRE, int RT, int MINW, int SYM, int DB, int ZL>
__global__ void __launch_bounds__((fused_threads<R, TX, TY, DB>()), MINW)
    fused_stage_kernel(const T* __restrict__ q, T* __restrict__ dq, T* __restrict__ out,
                       const BoxInst<T>* __restrict__ inst, int ninst, T dt_scale, T A, T B) {
    const int total = gridDim.x;
    const int w = blockIdx.x;
    const int xcd = w % 8;
    // An ensemble's workgroups differ in length: its XCDs take turns in pieces of kXcdPiece
    // neighbours, and only what is left over goes in eighths.
    const int dealt = ninst > 1 ? total / (8 * kXcdPiece) * (8 * kXcdPiece) : 0;
    const int per = (total - dealt) / 8, extra = total % 8;      // the first `extra` XCDs take one more
    const int turn = w / 8;
    const int lam = w < dealt ? (turn / kXcdPiece * 8 + xcd) * kXcdPiece + turn % kXcdPiece
                              : dealt + xcd * per + min(xcd, extra) + (turn - dealt / 8);
    int lo = 0, hi = ninst - 1;     // last box with first_wg <= lam
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (inst[mid].first_wg <= lam) lo = mid;
        else hi = mid - 1;
    }
    const BoxInst<T>& b = inst[lo];
    const int local = lam - b.first_wg;
    const int tile = local % (b.tiles_x * b.tiles_y);
    const int chunk = local / (b.tiles_x * b.tiles_y);
    // Tiles go strip by strip of kStripRows tile rows, column by column within a strip,
    // so the 32 workgroups an XCD runs at a time form a block and find each other's
    // x and y halos in its L2.
    const int strip = tile / (kStripRows * b.tiles_x), in_strip = tile % (kStripRows * b.tiles_x);
    const int rows = min(kStripRows, b.tiles_y - strip * kStripRows);
    const int tx = in_strip / rows;
    const int ty = strip * kStripRows + in_strip % rows;
    const int z0 = chunk * b.zchunk;
    const int zc = min(b.zchunk, b.c.n[2] - z0);
    T* dqb = dq ? dq + b.offset : nullptr;
    if constexpr (DB == 2) {
        constexpr bool PL = kPlain<T, MODE>;
        __shared__ SplitLds<T, R, TX, TY, PL> lds;
        if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) < TX * TY)   // whole wavefronts
            split_columns<T, R, TX, TY, MODE, SYM, PL>(lds, q + b.offset, dqb, out + b.offset, b.c, tx * TX, ty * TY, z0, zc,
                                                   b.dt * dt_scale, A, B, b.closure, b.cflag);
        else
            split_planes<T, R, TX, TY, MODE, SYM, PL>(lds, q + b.offset, b.c, tx * TX, ty * TY, z0, zc);
    } else {
        fused_stage_body<T, R, TX, TY, MODE, PRE, RT, SYM, DB, ZL>(q + b.offset, dqb, out + b.offset, b.c, tx * TX,
                                                                   ty * TY, z0, zc, b.dt * dt_scale, A, B, b.closure,
                                                                   b.cflag);
    }
}

}  // namespace sbli
