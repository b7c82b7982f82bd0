// Launch configurations of the fused stage kernel: the compiled variants, the model that
// gives a grid its default, and what the searches time.  Host arithmetic only, so that it
// can be compiled and tested without a device.
#pragma once

#include <algorithm>
#include <climits>
#include <cmath>

#include "../../include/sbli.h"

namespace sbli {

struct StageVariant {
    int tx, ty, pre, rot;
    int minw;   // wavefronts per SIMD the register allocation must allow (1 = as many VGPRs as needed)
    int db;     // barrier schedule: 0 two barriers a plane, 1 one, 2 one and the work split between
                // column and plane wavefronts (kernels_stage_fused.h)
    int zl;     // 1: the R planes below the output plane in LDS instead of registers
};

// X-macro lists of (TX, TY, PRE, RT, MINW, DB, ZL) per (type, radius).  An index is what
// sbli_set_tuning takes and callers store: entries keep their places, new ones go at the end.
#define SBLI_VARIANTS_D1(X) \
    X(16, 16, 1, 0, 1, 0, 0) X(16, 16, 1, 1, 1, 0, 0) X(32, 8, 1, 1, 1, 0, 0) X(16, 8, 1, 1, 2, 0, 0) X(16, 16, 1, 1, 1, 1, 0)
#define SBLI_VARIANTS_D2(X)                                                                                    \
    X(16, 16, 1, 0, 1, 0, 0) X(16, 16, 1, 1, 1, 0, 0) X(16, 16, 0, 1, 1, 0, 0) X(32, 8, 0, 0, 1, 0, 0) X(16, 8, 1, 1, 2, 0, 0) \
    X(16, 16, 1, 1, 1, 1, 0) X(16, 16, 1, 0, 1, 1, 0) X(16, 16, 1, 1, 1, 2, 0) X(16, 8, 1, 1, 2, 2, 0)
#define SBLI_VARIANTS_D3(X) X(8, 8, 0, 0, 1, 0, 0) X(8, 8, 1, 0, 1, 0, 0) X(16, 8, 1, 0, 1, 0, 0) X(16, 8, 1, 0, 1, 1, 0)
#define SBLI_VARIANTS_D4(X) \
    X(16, 4, 0, 0, 1, 0, 0) X(16, 4, 1, 0, 1, 0, 0) X(8, 8, 0, 0, 1, 0, 0) X(16, 4, 1, 0, 1, 0, 1) X(8, 8, 1, 0, 1, 0, 1)
#define SBLI_VARIANTS_F1(X) \
    X(16, 16, 1, 0, 1, 0, 0) X(16, 16, 1, 1, 1, 0, 0) X(32, 8, 1, 1, 1, 0, 0) X(16, 8, 1, 0, 1, 0, 0) X(16, 16, 1, 1, 1, 1, 0)
#define SBLI_VARIANTS_F2(X)                                                                                   \
    X(16, 8, 1, 0, 1, 0, 0) X(16, 8, 1, 1, 1, 0, 0) X(16, 16, 1, 1, 1, 0, 0) X(32, 8, 1, 1, 1, 0, 0) X(32, 8, 1, 1, 3, 0, 0) \
    X(16, 16, 1, 1, 3, 0, 0) X(16, 16, 1, 1, 1, 1, 0) X(32, 8, 1, 1, 1, 1, 0) X(16, 16, 1, 1, 3, 1, 0)            \
    X(32, 16, 1, 1, 1, 0, 0) X(32, 16, 1, 1, 1, 1, 0) X(16, 16, 1, 1, 1, 2, 0)
#define SBLI_VARIANTS_F3(X) \
    X(16, 16, 0, 0, 1, 0, 0) X(16, 16, 1, 0, 1, 0, 0) X(16, 8, 1, 0, 1, 0, 0) X(16, 16, 1, 1, 1, 2, 0)
#define SBLI_VARIANTS_F4(X) X(16, 8, 0, 0, 1, 0, 0) X(16, 8, 1, 0, 1, 0, 0) X(16, 4, 1, 0, 1, 0, 0)

#define SBLI_ENTRY(TX_, TY_, PRE_, RT_, MINW_, DB_, ZL_) StageVariant{TX_, TY_, PRE_, RT_, MINW_, DB_, ZL_},
struct VariantList {
    const StageVariant* v;
    int n;
};

// The fused variants of (dtype, radius), radius 1 .. 4.
inline VariantList fused_variants(int dtype, int r) {
    static const StageVariant d1[] = {SBLI_VARIANTS_D1(SBLI_ENTRY)}, d2[] = {SBLI_VARIANTS_D2(SBLI_ENTRY)},
                              d3[] = {SBLI_VARIANTS_D3(SBLI_ENTRY)}, d4[] = {SBLI_VARIANTS_D4(SBLI_ENTRY)},
                              f1[] = {SBLI_VARIANTS_F1(SBLI_ENTRY)}, f2[] = {SBLI_VARIANTS_F2(SBLI_ENTRY)},
                              f3[] = {SBLI_VARIANTS_F3(SBLI_ENTRY)}, f4[] = {SBLI_VARIANTS_F4(SBLI_ENTRY)};
#define SBLI_LIST(t) VariantList{t, (int)(sizeof(t) / sizeof(t[0]))}
    const bool d = dtype == SBLI_F64;
    switch (r) {
        case 1: return d ? SBLI_LIST(d1) : SBLI_LIST(f1);
        case 2: return d ? SBLI_LIST(d2) : SBLI_LIST(f2);
        case 3: return d ? SBLI_LIST(d3) : SBLI_LIST(f3);
        default: return d ? SBLI_LIST(d4) : SBLI_LIST(f4);
    }
#undef SBLI_LIST
}
#undef SBLI_ENTRY

// Default launch configuration.  A workgroup of the fused kernel takes zchunk + 4R serial
// steps of one plane, and the chip runs 256 workgroups at a time; its time is modelled as
// (zchunk + 4R) plane_us (1 + beside (rounds - 1)), rounds = ceil(workgroups / 256): a
// small grid takes chunks of a few planes (32^3: of one), a large one the longest that
// still fill the last round.  Each (type, radius) has one or two variants to choose from,
// a small tile for small grids and the one that is fastest on large grids; `beside` < 1
// where two workgroups fit a CU.  Within 15 % of the fastest of all variants and chunks
// from 20^3 to 256^3.  Measured us a stage, first variant with chunks of 32
// planes or the whole grid -> this choice (and the fastest of all variants and chunks),
// FP64 order 4: 32^3 71 -> 12 (12), 64^3 76 -> 24 (24), 96^3 66 -> 47 (47), 160^3 237 ->
// 179 (179), 256^3 742 -> 592 (592); FP32 order 4: 75 -> 11 (11), 78 -> 18 (18), 69 -> 34
// (34), 127 -> 98 (98), 392 -> 335 (335).
struct LaunchCand {
    int variant;        // index into the variant list of (type, radius)
    double plane_us;    // a workgroup's time for a plane with a CU to itself
    double beside;      // cost of a further round relative to the first
};

inline const LaunchCand* launch_cands(int dtype, int r, int& n) {
    static const LaunchCand d1[] = {{3, 1.2, 0.8}, {2, 1.6, 1.0}}, d2[] = {{8, 1.35, 0.75}, {7, 1.7, 1.0}},
                            d3[] = {{1, 2.0, 1.0}}, d4[] = {{4, 2.4, 1.0}}, f1[] = {{3, 0.9, 0.8}, {2, 1.2, 0.8}},
                            f2[] = {{11, 1.4, 1.0}, {10, 1.95, 1.0}}, f3[] = {{3, 1.5, 1.0}}, f4[] = {{2, 1.9, 0.35}};
    const bool d = dtype == SBLI_F64;
    n = r <= 2 ? 2 : 1;
    switch (r) {
        case 1: return d ? d1 : f1;
        case 2: return d ? d2 : f2;
        case 3: return d ? d3 : f3;
        default: return d ? d4 : f4;
    }
}

constexpr int kCus = 256;

// The chunk of at most `cap` planes that makes the modelled time of variant v over `count`
// boxes least; *cost receives it (in plane times).
inline int best_zchunk(int dtype, int r, int v, double beside, const sbli_params* p, int count, int cap, double* cost) {
    const StageVariant sv = fused_variants(dtype, r).v[v];
    int zmax = 1, best = 1;
    for (int i = 0; i < count; ++i) zmax = std::max(zmax, p[i].nz);
    *cost = HUGE_VAL;
    zmax = std::min(zmax, cap);
    for (int zc = 1; zc <= zmax; ++zc) {
        double units = 0;
        for (int i = 0; i < count; ++i)
            units += (double)((p[i].nx + sv.tx - 1) / sv.tx) * ((p[i].ny + sv.ty - 1) / sv.ty) *
                     ((p[i].nz + zc - 1) / zc);
        const double rounds = std::max(1.0, std::ceil(units / kCus));
        const double t = (zc + 4 * r) * (1.0 + beside * (rounds - 1.0));
        if (t < *cost) {
            *cost = t;
            best = zc;
        }
    }
    return best;
}

inline void choose_fused(int dtype, int r, const sbli_params* p, int count, int* variant, int* zchunk) {
    int n = 0;
    const LaunchCand* c = launch_cands(dtype, r, n);
    double least = HUGE_VAL;
    for (int k = 0; k < n; ++k) {
        double t = 0;
        const int zc = best_zchunk(dtype, r, c[k].variant, c[k].beside, p, count, INT_MAX, &t);
        if (t * c[k].plane_us < least) {
            least = t * c[k].plane_us;
            *variant = c[k].variant;
            *zchunk = zc;
        }
    }
}

// Cost of a further round for any variant: the rule's own where it has one.
inline double beside_of(int dtype, int r, int v) {
    int n = 0;
    const LaunchCand* c = launch_cands(dtype, r, n);
    for (int k = 0; k < n; ++k)
        if (c[k].variant == v) return c[k].beside;
    return 1.0;
}

// Planes per workgroup of variant v over `count` boxes under the cap zmax.  Chunks so long
// that the chip has CUs to spare are shortened to what the model prefers: two FP32 boxes of
// 32^3 at order 4 take 33.6 us a stage in chunks of 16 planes or more, 12.6 in single planes.
inline int capped_chunk(int dtype, int r, int v, const sbli_params* p, int count, int zmax) {
    const StageVariant sv = fused_variants(dtype, r).v[v];
    double units = 0;
    for (int i = 0; i < count; ++i) {
        const int zc = std::min(zmax, p[i].nz);
        units += (double)((p[i].nx + sv.tx - 1) / sv.tx) * ((p[i].ny + sv.ty - 1) / sv.ty) * ((p[i].nz + zc - 1) / zc);
    }
    if (units >= kCus) return zmax;
    double cost;
    return best_zchunk(dtype, r, v, beside_of(dtype, r, v), p, count, zmax, &cost);
}

struct Launch {
    int variant, zchunk;
};

// What a search keeps.  A later candidate replaces the best one only when it is faster by more
// than 1 %: candidates within timing noise of each other then resolve to the same (earlier)
// choice on every run.  The configuration in use comes first, before the clocks are up (64
// FP32 boxes: 2.97 ms a step for what then takes 2.67), and a launch timed after a slow variant
// reads 2 to 3 % high.  So a winner and the configuration in use are timed in turn at the end,
// twice each, and the latter is left only for one that is 1 % faster there.  Without this the
// search over those boxes left caps of 48 planes for 128, equal over the two steps it times:
// 26.1 instead of 25.5 ms for ten steps together, and 305 instead of 192 box by box, where
// long chunks leave most of the chip idle.
constexpr float kTuneMargin = 0.99f;
constexpr int kTuneTurns = 4;   // the winner first, whose own predecessor may be a slow one
struct TuneBest {
    Launch start, at;      // the configuration in use, and the best so far
    float ms = 1e30f, ms_start = 1e30f, ms_at = 1e30f;
    bool moved = false;    // at is another one than start
    explicit TuneBest(Launch s) : start(s), at(s) {}
    void offer(Launch c, float t, bool first) {
        if (t < ms * kTuneMargin) {
            at = c;
            ms = t;
            moved = !first;
        }
    }
    int turns() const { return moved ? kTuneTurns : 0; }
    Launch turn(int k) const { return k & 1 ? start : at; }
    void turned(int k, float t) {
        float& m = k & 1 ? ms_start : ms_at;
        m = std::min(m, t);
    }
    void settle() {   // without turns, or where one could not be launched, `at` stays
        if (ms_start == 1e30f || ms_at == 1e30f) return;
        moved = ms_at < ms_start * kTuneMargin;
        ms = moved ? ms_at : ms_start;
        if (!moved) at = start;
    }
};
constexpr int kMaxTried = 256;

// What sbli_autotune times of the fused form, in order: the configuration in use (unless it
// is the staged form), then each variant with chunks of the whole grid halved down to 16
// planes and with the chunk that sbli_init's rule would give it.
inline int tuning_candidates(int dtype, int r, const sbli_params* p, Launch entry, Launch* out) {
    const VariantList l = fused_variants(dtype, r);
    int n = 0;
    auto add = [&](int v, int zc) {
        for (int k = 0; k < n; ++k)
            if (out[k].variant == v && out[k].zchunk == zc) return;
        if (n < kMaxTried) out[n++] = {v, zc};
    };
    if (entry.variant < l.n) add(entry.variant, entry.zchunk);
    for (int v = 0; v < l.n; ++v) {
        int zc = p->nz;
        for (int k = 0; k < 6 && (zc >= 16 || k == 0); ++k) {
            add(v, zc);
            if (zc == 16) break;
            zc = (zc + 1) / 2;
        }
        double cost;
        add(v, best_zchunk(dtype, r, v, beside_of(dtype, r, v), p, 1, p->nz, &cost));
    }
    return n;
}

// What sbli_batch_autotune times, in order: the configuration in use (as a cap of the list
// below where one launches alike), then each variant under caps of 128 to 16 planes; one that
// launches like an earlier one is left out.
inline int batch_candidates(int dtype, int r, const sbli_params* p, int count, Launch entry, Launch* out) {
    const VariantList l = fused_variants(dtype, r);
    int nmax = 1, n = 0, chunk[kMaxTried];
    for (int i = 0; i < count; ++i) nmax = std::max(nmax, p[i].nz);
    auto planes = [&](int v, int zmax) { return std::min(capped_chunk(dtype, r, v, p, count, zmax), nmax); };
    auto add = [&](int v, int zmax) {
        const int zc = planes(v, zmax);
        for (int k = 0; k < n; ++k)
            if (out[k].variant == v && chunk[k] == zc) return;
        if (n == kMaxTried) return;
        chunk[n] = zc;
        out[n++] = {v, zmax};
    };
    constexpr int caps[] = {128, 96, 64, 48, 32, 16};
    for (int zmax : caps)
        if (n == 0 && planes(entry.variant, zmax) == planes(entry.variant, entry.zchunk)) add(entry.variant, zmax);
    add(entry.variant, entry.zchunk);
    for (int v = 0; v < l.n; ++v)
        for (int zmax : caps) add(v, zmax);
    return n;
}

}  // namespace sbli
