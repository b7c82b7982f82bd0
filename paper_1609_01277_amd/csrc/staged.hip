// Launches of the staged form of the stage kernel (kernels_staged.h, kernels_staged_march.h) for every
// element type, radius 1..6 and mode; compiled in a translation unit of its own.
#include "kernels_staged_march.h"
#include "staged.h"

#include <algorithm>

namespace sbli {

// Planes per run of a kernel that marches in z.  A workgroup (a tile and a run) fills a CU
// and the plane loop is one chain, so few long runs leave the chip idle (96^3 in 32x32
// tiles and runs of 64 planes: 18 workgroups), a number of them just over a multiple of
// the CUs costs a further round, and each run begins with 2R planes of its own columns,
// worth `fill` planes of the loop.  So: the run that makes *cost = rounds x (planes + fill)
// least, up to 160 planes (runs of 32, 64 and 128 measure the same at 512^3).
static int run_planes(int tiles, int nz, double fill, double* cost) {
    const int cus = 256;
    auto cost_of = [&](int zc) {
        const int64_t units = (int64_t)tiles * ((nz + zc - 1) / zc);
        return (double)((units + cus - 1) / cus) * (zc + fill);
    };
    int best = std::min(nz, kNestedRun);
    *cost = cost_of(best);
    for (int rounds = 1; rounds <= 4; ++rounds) {
        const int runs = std::min(rounds * cus / tiles, nz);
        if (runs < 1) continue;
        const int zc = (nz + runs - 1) / runs;
        if (zc <= 160 && cost_of(zc) < *cost) {
            best = zc;
            *cost = cost_of(zc);
        }
    }
    return best;
}

template <typename T, int R>
static void staged_run(const StagedArgs& a, const T* qin, T* dq, T* qout, T* nf) {
    const BoxConst<T>& c = *(const BoxConst<T>*)a.box;
    auto grid_of = [&](int tiles, int zc) {
        const int64_t units = (int64_t)tiles * ((c.n[2] + zc - 1) / zc);
        return (unsigned)(kStagedXcds * ((units + kStagedXcds - 1) / kStagedXcds));
    };
    auto nested = [&](auto tn) {
        constexpr int TN = decltype(tn)::value;
        const int tx = (c.n[0] + TN - 1) / TN, ty = (c.n[1] + TN - 1) / TN;
        // Both steps, us a stage, runs of 64 -> this: 32^3, FP64, order 8: 100 -> 22; 64^3:
        // 222 -> 36; 96^3: 268 -> 92; 128^3: 379 -> 198; 160^3: 514 -> 377; 256^3 keeps 64.
        double cost;
        const int zn = run_planes(tx * ty, c.n[2], R, &cost);
        if (sizeof(T) == 4 && a.mode == kModeRHS)   // kPlain
            staged_nested_zring_kernel<T, R, TN, kPlain<T, kModeRHS>><<<grid_of(tx * ty, zn), TN * TN, 0, a.stream>>>(
                qin, nf, c, tx, ty, zn);
        else
            staged_nested_zring_kernel<T, R, TN, false><<<grid_of(tx * ty, zn), TN * TN, 0, a.stream>>>(qin, nf, c, tx,
                                                                                                         ty, zn);
    };
    // The nested-field step in 32x32 tiles where the register and LDS budget allows
    // (every radius in FP32, up to R = 4 in FP64): each tile then fetches its R-wide
    // x-arms, 32-byte row pieces of 128-byte lines, for four times as many own points.
    // In 16x16 tiles on grids whose 32x32 tiles, plane by plane, are no more than the CUs
    // (up to 64^3): both steps, FP64 order 8, 32^3 21.8 -> 16.4 us, 64^3 35.4 -> 32.0, but
    // 96^3 70.6 -> 72.5 and 256^3 1,150 -> 1,184; FP32 16.2 -> 13.6, 26.1 -> 23.7, 57.1 ->
    // 60.9, 776 -> 840.
    constexpr bool kWide = sizeof(T) == 4 || R <= 4;
    const int64_t wide_units = (int64_t)((c.n[0] + 31) / 32) * ((c.n[1] + 31) / 32) * c.n[2];
    if (kWide && wide_units > 256)
        nested(std::integral_constant<int, kWide ? 2 * kStagedTile : kStagedTile>{});
    else
        nested(std::integral_constant<int, kStagedTile>{});
    const int tx = (c.n[0] + kStagedTile - 1) / kStagedTile, ty = (c.n[1] + kStagedTile - 1) / kStagedTile;
    constexpr int NT = kStagedTile * kStagedTile;
    const T dt = (T)a.dt, A = (T)a.A, B = (T)a.B;
    const T* clos = (const T*)a.clos;
    if constexpr (R >= 3) {
        // Marching runs of planes (orders 6 and up) where they fill the chip; single planes on
        // small grids, which have too few tiles for it, and at orders 2 and 4, where the fused
        // kernel is faster than either.  A single-plane launch takes about 1.7 times as long
        // for a tile's plane (1.2 to 1.4 times where HBM bounds both).  Both steps, us a stage,
        // single planes -> marching: FP64 order 8: 64^3 37 -> 33, 96^3 94 -> 81, 128^3 222 ->
        // 182, 256^3 1,548 -> 1,207; order 12: 64^3 42 -> 56, 96^3 115 -> 118, 128^3 280 -> 251,
        // 256^3 1,943 -> 1,593; FP32 order 8: 64^3 25 -> 25, 128^3 127 -> 114, 256^3 1,012 -> 776.
        double cost;
        const int run = run_planes(tx * ty, c.n[2], 1.5 * R, &cost);
        if (cost <= 1.7 * tx * ty * c.n[2] / 256.0) {
            const dim3 mgrid(tx * ty * ((c.n[2] + run - 1) / run));
            switch (a.mode) {
                case kModeRHS:
                    staged_march_kernel<T, R, kModeRHS><<<mgrid, 2 * NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B, clos,
                                                                                        a.cflag, tx, ty, run);
                    break;
                case kModeStage1:
                    staged_march_kernel<T, R, kModeStage1><<<mgrid, 2 * NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B,
                                                                                           clos, a.cflag, tx, ty, run);
                    break;
                case kModeStage2:
                    staged_march_kernel<T, R, kModeStage2><<<mgrid, 2 * NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B,
                                                                                           clos, a.cflag, tx, ty, run);
                    break;
                default:
                    staged_march_kernel<T, R, kModeStage3><<<mgrid, 2 * NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B,
                                                                                           clos, a.cflag, tx, ty, run);
                    break;
            }
            return;
        }
    }
    const int zc = 1;   // one plane per workgroup: see staged_unit
    const unsigned grid = grid_of(tx * ty, zc);
    switch (a.mode) {
        case kModeRHS:
            staged_tiled_kernel<T, R, kModeRHS><<<grid, NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B, clos,
                                                                           a.cflag, tx, ty, zc);
            break;
        case kModeStage1:
            staged_tiled_kernel<T, R, kModeStage1><<<grid, NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B, clos,
                                                                              a.cflag, tx, ty, zc);
            break;
        case kModeStage2:
            staged_tiled_kernel<T, R, kModeStage2><<<grid, NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B, clos,
                                                                              a.cflag, tx, ty, zc);
            break;
        default:
            staged_tiled_kernel<T, R, kModeStage3><<<grid, NT, 0, a.stream>>>(qin, nf, dq, qout, c, dt, A, B, clos,
                                                                              a.cflag, tx, ty, zc);
            break;
    }
}

template <typename T>
static void staged_dispatch(const StagedArgs& a, const void* qin, void* dq, void* qout) {
    T* nf = (T*)a.scratch;
    const T* qi = (const T*)qin;
    T* d = (T*)dq;
    T* qo = (T*)qout;
    switch (a.r) {
        case 1: staged_run<T, 1>(a, qi, d, qo, nf); break;
        case 2: staged_run<T, 2>(a, qi, d, qo, nf); break;
        case 3: staged_run<T, 3>(a, qi, d, qo, nf); break;
        case 4: staged_run<T, 4>(a, qi, d, qo, nf); break;
        case 5: staged_run<T, 5>(a, qi, d, qo, nf); break;
        default: staged_run<T, 6>(a, qi, d, qo, nf); break;
    }
}

void staged_launch(const StagedArgs& a, const void* qin, void* dq, void* qout) {
    if (a.f64) staged_dispatch<double>(a, qin, dq, qout);
    else staged_dispatch<float>(a, qin, dq, qout);
}

}  // namespace sbli
