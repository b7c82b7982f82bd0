// Launches of the staged form of the stage kernel (kernels_staged.h) for every
// element type, radius 1..6 and mode; compiled in a translation unit of its own.
#include "kernels_staged.h"
#include "staged.h"

#include <algorithm>

namespace sbli {

// Planes per run of the nested-field step.  A workgroup (a tile and a run) fills a CU, and
// the plane loop is one chain, so few long runs leave the chip idle (96^3 in 32x32 tiles
// and runs of 64 planes: 18 workgroups) and a number of them just over a multiple of the
// CUs costs a further round; each run loads 2R planes of its own columns first, worth
// about R planes of the loop.  So: the run that makes rounds x (planes + R) least, up to
// 160 planes (runs of 32, 64 and 128 measure the same at 512^3).  Both steps, us a stage,
// runs of 64 -> this: 32^3, FP64, order 8: 100 -> 22; 64^3: 222 -> 36; 96^3: 268 -> 92;
// 128^3: 379 -> 198; 160^3: 514 -> 377; 256^3 keeps 64 (1,490; 32: 1,507; 128: 1,681).
static int nested_run(int tiles, int nz, int R) {
    const int cus = 256;
    int best = std::min(nz, kNestedRun);
    auto cost = [&](int zc) {
        const int64_t units = (int64_t)tiles * ((nz + zc - 1) / zc);
        return ((units + cus - 1) / cus) * (zc + R);
    };
    int64_t least = cost(best);
    for (int rounds = 1; rounds <= 4; ++rounds) {
        const int runs = std::min(rounds * cus / tiles, nz);
        if (runs < 1) continue;
        const int zc = (nz + runs - 1) / runs;
        if (zc <= 160 && cost(zc) < least) {
            best = zc;
            least = cost(zc);
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
    {
        // The nested-field step in 32x32 tiles where the register and LDS budget allows
        // (every radius in FP32, up to R = 4 in FP64): each tile then fetches its R-wide
        // x-arms, 32-byte row pieces of 128-byte lines, for four times as many own points.
        constexpr int TN = (sizeof(T) == 8 && R > 4) ? kStagedTile : 2 * kStagedTile;
        const int tx = (c.n[0] + TN - 1) / TN, ty = (c.n[1] + TN - 1) / TN;
        const int zn = nested_run(tx * ty, c.n[2], R);
        if (sizeof(T) == 4 && a.mode == kModeRHS)   // kPlain
            staged_nested_zring_kernel<T, R, TN, kPlain<T, kModeRHS>><<<grid_of(tx * ty, zn), TN * TN, 0, a.stream>>>(
                qin, nf, c, tx, ty, zn);
        else
            staged_nested_zring_kernel<T, R, TN, false><<<grid_of(tx * ty, zn), TN * TN, 0, a.stream>>>(qin, nf, c, tx,
                                                                                                         ty, zn);
    }
    const int tx = (c.n[0] + kStagedTile - 1) / kStagedTile, ty = (c.n[1] + kStagedTile - 1) / kStagedTile;
    constexpr int NT = kStagedTile * kStagedTile;
    const T dt = (T)a.dt, A = (T)a.A, B = (T)a.B;
    const T* clos = (const T*)a.clos;
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
