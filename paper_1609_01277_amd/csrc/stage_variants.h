// Compiled launch variants of the fused stage kernel and their dispatch.
//
// A variant fixes the (x, y) tile of a workgroup and how far the global loads
// run ahead (see fused_stage_body).  Every variant performs the same arithmetic
// per point in the same order, so all of them give bitwise identical states;
// they differ only in speed, which the autotuner measures.
#pragma once

#include "kernels_stage_fused.h"
#include "launch_rule.h"

namespace sbli {

// One launch: the boxes (device table), their total workgroup count, the mode
// and the RK coefficients.
struct StageArgs {
    hipStream_t stream;
    const void* inst;   // device array of BoxInst<T>
    int ninst;
    int total_wg;
    int mode;
    double dt_scale, A, B;
    int sym;            // 1 if a box of the launch has a symmetry axis
};

template <typename T, int R, int TX, int TY, int PRE, int RT, int MINW, int DB, int ZL, int MODE>
inline void launch_fused_cfg(const StageArgs& a, const T* qin, T* dq, T* qout) {
    constexpr int nt = fused_threads<R, TX, TY, DB>();
    if (a.sym)
        fused_stage_kernel<T, R, TX, TY, MODE, PRE, RT, MINW, 1, DB, ZL><<<dim3(a.total_wg), nt, 0, a.stream>>>(
            qin, dq, qout, (const BoxInst<T>*)a.inst, a.ninst, (T)a.dt_scale, (T)a.A, (T)a.B);
    else
        fused_stage_kernel<T, R, TX, TY, MODE, PRE, RT, MINW, 0, DB, ZL><<<dim3(a.total_wg), nt, 0, a.stream>>>(
            qin, dq, qout, (const BoxInst<T>*)a.inst, a.ninst, (T)a.dt_scale, (T)a.A, (T)a.B);
}

template <typename T, int R, int TX, int TY, int PRE, int RT, int MINW, int DB, int ZL>
inline bool try_variant(int& k, int want, const StageArgs& a, const T* qin, T* dq, T* qout) {
    if (k++ != want) return false;
    switch (a.mode) {
        case kModeRHS: launch_fused_cfg<T, R, TX, TY, PRE, RT, MINW, DB, ZL, kModeRHS>(a, qin, dq, qout); break;
        case kModeStage1: launch_fused_cfg<T, R, TX, TY, PRE, RT, MINW, DB, ZL, kModeStage1>(a, qin, dq, qout); break;
        case kModeStage2: launch_fused_cfg<T, R, TX, TY, PRE, RT, MINW, DB, ZL, kModeStage2>(a, qin, dq, qout); break;
        default: launch_fused_cfg<T, R, TX, TY, PRE, RT, MINW, DB, ZL, kModeStage3>(a, qin, dq, qout); break;
    }
    return true;
}

#define SBLI_TRY(TX_, TY_, PRE_, RT_, MINW_, DB_, ZL_) \
    if (try_variant<T, R, TX_, TY_, PRE_, RT_, MINW_, DB_, ZL_>(k, v, a, qin, dq, qout)) return true;

template <typename T, int R>
struct VariantSet;

// The launch function of a (type, radius) -- which instantiates its kernels --
// is defined only in the translation unit stage_{f64,f32}_r{1..4}.hip that sets
// SBLI_STAGE_TU_{TYPE,R,LIST}, so the variants compile in parallel.
#define SBLI_VARIANT_SET(TYPE, RR)                                                                        \
    template <>                                                                                           \
    struct VariantSet<TYPE, RR> {                                                                         \
        using T = TYPE;                                                                                   \
        static constexpr int R = RR;                                                                      \
        static bool launch(int v, const StageArgs& a, const T* qin, T* dq, T* qout);                  \
    };

SBLI_VARIANT_SET(double, 1)
SBLI_VARIANT_SET(double, 2)
SBLI_VARIANT_SET(double, 3)
SBLI_VARIANT_SET(double, 4)
SBLI_VARIANT_SET(float, 1)
SBLI_VARIANT_SET(float, 2)
SBLI_VARIANT_SET(float, 3)
SBLI_VARIANT_SET(float, 4)

#if defined(SBLI_STAGE_TU_TYPE) && defined(SBLI_STAGE_TU_R) && defined(SBLI_STAGE_TU_LIST)
bool VariantSet<SBLI_STAGE_TU_TYPE, SBLI_STAGE_TU_R>::launch(int v, const StageArgs& a, const T* qin, T* dq,
                                                             T* qout) {
    int k = 0;
    SBLI_STAGE_TU_LIST(SBLI_TRY)
    return false;
}
#endif

#undef SBLI_TRY
#undef SBLI_VARIANT_SET

// Runtime dispatch over (radius, variant) for one element type.
template <typename T>
struct StageDispatch {
    static int count(int r) { return fused_variants(sizeof(T) == 8 ? SBLI_F64 : SBLI_F32, r).n; }
    static StageVariant get(int r, int i) { return fused_variants(sizeof(T) == 8 ? SBLI_F64 : SBLI_F32, r).v[i]; }
    static bool launch(int r, int v, const StageArgs& a, const T* qin, T* dq, T* qout);
};

template <typename T>
inline bool StageDispatch<T>::launch(int r, int v, const StageArgs& a, const T* qin, T* dq, T* qout) {
    switch (r) {
        case 1: return VariantSet<T, 1>::launch(v, a, qin, dq, qout);
        case 2: return VariantSet<T, 2>::launch(v, a, qin, dq, qout);
        case 3: return VariantSet<T, 3>::launch(v, a, qin, dq, qout);
        default: return VariantSet<T, 4>::launch(v, a, qin, dq, qout);
    }
}

// Fills the launch-geometry part of a box entry for tile (tx, ty) and zchunk;
// returns the number of workgroups the box takes.
template <typename T>
inline int set_box_geometry(BoxInst<T>& b, int tx, int ty, int zchunk, int first_wg) {
    b.tiles_x = (b.c.n[0] + tx - 1) / tx;
    b.tiles_y = (b.c.n[1] + ty - 1) / ty;
    b.zchunk = zchunk;
    b.first_wg = first_wg;
    b.num_wg = b.tiles_x * b.tiles_y * ((b.c.n[2] + zchunk - 1) / zchunk);
    return b.num_wg;
}

}  // namespace sbli
