// kern_bra.hip -- kernel instantiations for one bra angular pair (JK_LI, JK_LJ),
// compiled once per pair with -DJK_LI=.. -DJK_LJ=.. so the classes build in
// parallel.  Kets (LK, LL) run over every canonical pair with LK >= LL and
// (LK, LL) <= (JK_LI, JK_LJ) lexicographically.
#include "jk_registry.h"

#ifndef JK_LI
#error "JK_LI / JK_LJ must be defined"
#endif

namespace jk {

template <int LI, int LJ, int LK, int LL, typename R>
static hipError_t launch_k1(const JkArgs &a, const ClsArgs *cls, const ClsGroup &g, const Batch &b, int units, size_t,
                            hipStream_t s) {
    static_assert(ArgsFirst<decltype(&jk_k1<LI, LJ, LK, LL, R, MODE_JK>)>::ok, "find_work reads the arguments' start");
    if (units <= 0) return hipSuccess;
    hipLaunchKernelGGL((jk_k1<LI, LJ, LK, LL, R, MODE_JK>), dim3((units + 3) / 4), dim3(256), 0, s, a, cls, g, b.descs, b.ndesc,
                       units);
    return hipGetLastError();
}

template <int LI, int LJ, int LK, int LL, typename R>
static hipError_t export_k1(const JkArgs &a, hipStream_t s) {
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL((jk_k1<LI, LJ, LK, LL, R, MODE_EXPORT>), dim3((a.nq + 255) / 256), dim3(256), 0, s, a,
                       (const ClsArgs *)nullptr, ClsGroup{}, (const BatchDesc *)nullptr, 0, 0);
    return hipGetLastError();
}

// Dynamic LDS above 64 KB needs a per-kernel opt-in (once per kernel).
template <typename K>
static hipError_t lds_opt_in(K kernel, size_t lds, bool &done) {
    if (lds <= 64 * 1024 || done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, ROW_LDS_MAX);
    if (e == hipSuccess) done = true;
    return e;
}

// Row tasks with one of the row kernels.
#define JK_LAUNCH_ROW(kernel)                                                                                     \
    static_assert(ArgsFirst<decltype(&kernel<LI, LJ, LK, LL, R, NT>)>::ok, "find_work reads the arguments' start"); \
    if (units <= 0) return hipSuccess;                                                                            \
    if (lds > (size_t)ROW_LDS_MAX) return hipErrorInvalidValue;                                                   \
    static bool opted_in = false;                                                                                 \
    const hipError_t e = lds_opt_in(&kernel<LI, LJ, LK, LL, R, NT>, lds, opted_in);                               \
    if (e != hipSuccess) return e;                                                                                \
    hipLaunchKernelGGL((kernel<LI, LJ, LK, LL, R, NT>), dim3(units), dim3(NT), lds, s, a, cls, g, b.descs, b.ndesc); \
    return hipGetLastError();

template <int LI, int LJ, int LK, int LL, typename R, int NT>
static hipError_t launch_row(const JkArgs &a, const ClsArgs *cls, const ClsGroup &g, const Batch &b, int units, size_t lds,
                             hipStream_t s) {
    JK_LAUNCH_ROW(jk_k1_row)
}

template <int LI, int LJ, int LK, int LL, typename R, int NT>
static hipError_t launch_row2(const JkArgs &a, const ClsArgs *cls, const ClsGroup &g, const Batch &b, int units, size_t lds,
                              hipStream_t s) {
    JK_LAUNCH_ROW(jk_k2_row)
}

template <int LI, int LJ, int LK, int LL, typename R, int NT>
static hipError_t launch_row3(const JkArgs &a, const ClsArgs *cls, const ClsGroup &g, const Batch &b, int units, size_t lds,
                              hipStream_t s) {
    JK_LAUNCH_ROW(jk_k3_row)
}

template <int LI, int LJ, int LK, int LL, typename R>
static hipError_t launch_k2(const JkArgs &a, const ClsArgs *cls, const ClsGroup &g, const Batch &b, int units, size_t,
                            hipStream_t s) {
    static_assert(ArgsFirst<decltype(&jk_k2<LI, LJ, LK, LL, R, MODE_JK>)>::ok, "find_work reads the arguments' start");
    if (units <= 0) return hipSuccess;
    hipLaunchKernelGGL((jk_k2<LI, LJ, LK, LL, R, MODE_JK>), dim3(units), dim3(k2_lanes(LI, LJ, LK, LL)), 0, s, a, cls, g, b.descs,
                       b.ndesc);
    return hipGetLastError();
}

template <int LI, int LJ, int LK, int LL, typename R>
static hipError_t export_k2(const JkArgs &a, hipStream_t s) {
    constexpr int QW = k2_qw(LI, LJ, LK, LL);
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL((jk_k2<LI, LJ, LK, LL, R, MODE_EXPORT>), dim3((a.nq + QW - 1) / QW),
                       dim3(k2_lanes(LI, LJ, LK, LL)), 0, s, a, (const ClsArgs *)nullptr, ClsGroup{},
                       (const BatchDesc *)nullptr, 0);
    return hipGetLastError();
}

// Classes with a g shell (l = 4) have no 64-lane short-bra row kernels, which
// keeps their compile time in bounds: short bras run as tiles, and batched
// builds of such molecules report JK_EUNSUPPORTED.
template <int LK, int LL>
static void reg_one() {
    constexpr int LI = JK_LI, LJ = JK_LJ;
    constexpr bool FULL = LI < 4;
    if constexpr (LK >= LL && (LK < LI || (LK == LI && LL <= LJ))) {
        ClassEntry &e = g_classes[class_id(LI, LJ, LK, LL)];
        if constexpr (has_family1(LI, LJ, LK, LL)) {
            e.tiles[0][0] = &launch_k1<LI, LJ, LK, LL, double>;
            e.tiles[0][1] = &launch_k1<LI, LJ, LK, LL, float>;
            e.row[0][0] = &launch_row<LI, LJ, LK, LL, double, 256>;
            e.row[0][1] = &launch_row<LI, LJ, LK, LL, float, 256>;
            if constexpr (FULL) {
                e.srow[0][0] = &launch_row<LI, LJ, LK, LL, double, 64>;
                e.srow[0][1] = &launch_row<LI, LJ, LK, LL, float, 64>;
            }
        }
        if constexpr (has_family2(LI, LJ, LK, LL)) {
            e.tiles[1][0] = &launch_k2<LI, LJ, LK, LL, double>;
            e.tiles[1][1] = &launch_k2<LI, LJ, LK, LL, float>;
            e.row[1][0] = &launch_row2<LI, LJ, LK, LL, double, 256>;
            e.row[1][1] = &launch_row2<LI, LJ, LK, LL, float, 256>;
            if constexpr (FULL) {
                e.srow[1][0] = &launch_row2<LI, LJ, LK, LL, double, 64>;
                e.srow[1][1] = &launch_row2<LI, LJ, LK, LL, float, 64>;
            }
            e.row_fixed[1][0] = K2RowLds<LI, LJ, LK, LL>::template fixed<double>();
            e.row_fixed[1][1] = K2RowLds<LI, LJ, LK, LL>::template fixed<float>();
        }
        if constexpr (has_family3(LI, LJ, LK, LL)) {
            e.row[2][0] = &launch_row3<LI, LJ, LK, LL, double, 256>;
            e.row[2][1] = &launch_row3<LI, LJ, LK, LL, float, 256>;
            if constexpr (FULL) {
                e.srow[2][0] = &launch_row3<LI, LJ, LK, LL, double, 64>;
                e.srow[2][1] = &launch_row3<LI, LJ, LK, LL, float, 64>;
            }
            e.row_fixed[2][0] = K3Cfg<LI, LJ, LK, LL>::template wave_bytes<double>();
            e.row_fixed[2][1] = K3Cfg<LI, LJ, LK, LL>::template wave_bytes<float>();
        }
        if constexpr (default_family(LI, LJ, LK, LL) == 1) {
            e.ex64 = &export_k1<LI, LJ, LK, LL, double>;
            e.ex32 = &export_k1<LI, LJ, LK, LL, float>;
        } else {
            e.ex64 = &export_k2<LI, LJ, LK, LL, double>;
            e.ex32 = &export_k2<LI, LJ, LK, LL, float>;
        }
    }
}

static int reg_all() {
    reg_one<0, 0>();
    reg_one<1, 0>(); reg_one<1, 1>();
    reg_one<2, 0>(); reg_one<2, 1>(); reg_one<2, 2>();
    reg_one<3, 0>(); reg_one<3, 1>(); reg_one<3, 2>(); reg_one<3, 3>();
    reg_one<4, 0>(); reg_one<4, 1>(); reg_one<4, 2>(); reg_one<4, 3>(); reg_one<4, 4>();
    return 0;
}

static const int registered = reg_all();

}  // namespace jk
