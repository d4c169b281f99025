// Variants and launcher of the narrow single-read pass (kernel and reasoning: narrow.h).
#include "common.h"
#include "narrow.h"

namespace lb {

namespace {

typedef void (*NarrowLaunch)(const Dims&, int, const Buffers&, const APassArgs&, const double*, hipStream_t, hipEvent_t, hipEvent_t);

struct NarrowVariant {
    int dtype, lanes, kc, sets;
    // [0] with non-temporal loads of the matrix, [1] with ordinary ones (matrix_cached)
    NarrowLaunch launch[2][3];
    NarrowLaunch own[2][2];   // the direction passes that make Algorithm 2's choice themselves, quadratic and logistic (null: none)
};

template <typename T, int L, int KC, int S, int LOGI, bool OWN, bool CACHED>
void launch_t(const Dims& dm, int blocks, const Buffers& bf, const APassArgs& a, const double* psi, hipStream_t st,
              hipEvent_t ev0, hipEvent_t ev1) {
    hipExtLaunchKernelGGL((narrow::k_narrow<T, L, KC, S, LOGI, OWN, CACHED>), dim3(blocks), dim3(kBlock), 0, st, ev0, ev1, 0,
                          (const T*)a.A, dm.ld, dm.rows, dm.cols, a, bf.scal, bf.row, bf.t, psi, bf.wpart, bf.losspart);
}
// With few lanes to a row (up to 192 fp32 or 96 fp64 columns) vectors are short for most m (small_step_ok) and nothing is
// gained by the choice being made here; beyond, it saves the direction kernel's arrival and up to 10 pairs the Gram
// kernel's too.  Whole iterations, us, choice read / made here: lasso fp64 122 x 1024 33.2 / 30.6, 2441 x 1024 35.0 / 32.2,
// 48828 x 1024 89.9 / 86.8; least squares fp32 4882 x 1024 35.7 / 32.4, m = 30 657 x 380 41.2 / 39.3.
template <typename T, int L, int KC, int S, int LOGI, bool CACHED>
constexpr NarrowLaunch own_t() {
    if constexpr (L >= 32) return launch_t<T, L, KC, S, LOGI, true, CACHED>;
    else return nullptr;
}

#define LB_NARROW_ALL(T, L, KC, S, C) {launch_t<T, L, KC, S, 0, false, C>, launch_t<T, L, KC, S, 1, false, C>, launch_t<T, L, KC, S, 2, false, C>}
#define LB_NARROW(dt, T, L, KC, S) {dt, L, KC, S, {LB_NARROW_ALL(T, L, KC, S, false), LB_NARROW_ALL(T, L, KC, S, true)},               \
                                    {{own_t<T, L, KC, S, 0, false>(), own_t<T, L, KC, S, 2, false>()},                                  \
                                     {own_t<T, L, KC, S, 0, true>(), own_t<T, L, KC, S, 2, true>()}}}
// the quadratic kinds only (the logistic row operations do not fit the registers beside the rows)
#define LB_NARROW_QUAD(dt, T, L, KC, S) {dt, L, KC, S, {{launch_t<T, L, KC, S, 0, false, false>, nullptr, nullptr},                      \
                                                        {launch_t<T, L, KC, S, 0, false, true>, nullptr, nullptr}},                     \
                                         {{own_t<T, L, KC, S, 0, false>(), nullptr}, {own_t<T, L, KC, S, 0, true>(), nullptr}}}
// By capacity L * KC in 16-byte chunks; the first whose capacity covers a row is used.  The line to the ring kernel is
// where it measured faster (0.4 GB matrices, us per pass, this kernel / ring): fp32 least squares 100 columns 69 / 271,
// 512 69 / 70, 1024 66 / 70, 1536 66 / 72, 1800 76 / 75; fp32 logistic 100 81 / 390, 512 72 / 89, 1000 66 / 94,
// 1536 77 / 83, 2000 78 / 77; fp64 least squares 100 64 / 270, 512 62 / 70, 1024 64 / 67; fp64 logistic 100 68 / 426,
// 512 67 / 97, 768 63 / 75, 900 80 / 76 (spills).
// Whole iterations at 1, 2, 5, 20, 80 and 400 MB, 100 to 1536 columns, m = 10, 20 and 30, all kinds: between 0.27 and 1.00 of
// the ring kernel's time (nearest to it the lasso of 1-2 MB at 1600 to 2048 variables).
#define LB_NARROW_TABLE(dt, T)                                                                                       \
    LB_NARROW(dt, T, 8, 1, 8), LB_NARROW(dt, T, 8, 2, 8), LB_NARROW(dt, T, 8, 3, 8), LB_NARROW(dt, T, 16, 2, 8),     \
    LB_NARROW(dt, T, 16, 3, 8), LB_NARROW(dt, T, 32, 2, 8), LB_NARROW(dt, T, 32, 3, 8), LB_NARROW(dt, T, 64, 2, 8),  \
    LB_NARROW(dt, T, 64, 3, 8), LB_NARROW_QUAD(dt, T, 64, 4, 8), LB_NARROW(dt, T, 64, 4, 4), LB_NARROW(dt, T, 64, 5, 4),  \
    LB_NARROW(dt, T, 64, 6, 4)
const NarrowVariant kNarrow[] = {
    LB_NARROW_TABLE(LBFGSB_F32, float),
    LB_NARROW_TABLE(LBFGSB_F64, double), LB_NARROW_QUAD(LBFGSB_F64, double, 64, 8, 4),
};
constexpr int kNumNarrow = sizeof(kNarrow) / sizeof(kNarrow[0]);

}  // namespace

bool narrow_shape_ok(const Dims& dm, int* variant, int* blocks) {
    *variant = -1;
    *blocks = 0;
    const int vec = dm.dtype == LBFGSB_F32 ? 4 : 2;
    if (dm.kind == LBFGSB_OBJ_QP || is_transport(dm.kind) || dm.cols < vec) return false;
    // byte offsets inside a set of rows are 32-bit, and so are the numbers of rows, those of a tile behind the last included
    if (dm.ld > (int64_t)1 << 24 || dm.rows > 0x7fffff00) return false;
    const int64_t chunks = (dm.cols + vec - 1) / vec;
    for (int i = 0; i < kNumNarrow; ++i) {
        const NarrowVariant& v = kNarrow[i];
        if (v.dtype != dm.dtype || v.lanes * v.kc < chunks || dm.rows < 64 / v.lanes) continue;
        if (dm.kind == LBFGSB_OBJ_LOGISTIC_L2 && !v.launch[0][2]) continue;
        const int64_t rt = v.sets * (64 / v.lanes), tiles = (dm.rows + rt - 1) / rt;
        const int64_t b = (tiles + kWaves - 1) / kWaves;
        *variant = i;
        *blocks = (int)(b > kNarrowBlocksMax ? kNarrowBlocksMax : b);
        return true;
    }
    return false;
}

bool narrow_makes_choice(const Geometry& ge) {
    return kNarrow[ge.narrow_variant].own[0][0] && ge.dir_blocks <= kPassDirBlocksMax;
}

void launch_narrow(const Dims& dm, const Geometry& ge, const Buffers& bf, const APassArgs& a, const double* psi,
                   hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const NarrowVariant& v = kNarrow[ge.narrow_variant];
    const int logi = a.mode == kRowLogiSpec ? 2 : (a.mode == kRowLogiEval ? 1 : 0);
    const int cached = matrix_cached(dm);
    (a.select_p && a.dir_blocks > 0 ? v.own[cached][logi / 2] : v.launch[cached][logi])(dm, ge.fused_blocks, bf, a, psi, st, ev0, ev1);
}

}  // namespace lb
