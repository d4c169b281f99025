// Fused single-read A pass: variant table and launchers (short rows: narrow.hip; large symmetric matrices: symmetric.hip).
// The kernel itself (and the reasoning behind its layout) is in fused_ring.h.
//
// A variant fixes the workgroup size NT, the 16-byte chunks per thread and row KC = KCU*U, the rows
// per barrier R and the ring depth NB (in slots of KCU chunks).  The table below is the outcome of
// timing on MI355X: the entries are those that keep the ring plus the fp64 accumulators of w inside
// the 256 registers a thread has at two waves per SIMD WITHOUT spilling -- a spill inside the row
// loop waits for every outstanding load and so empties the ring, which costs more than a shallower
// ring does.  Measured on matrices of 0.8-8 GB: 75-82 % of the 8 TB/s HBM peak, against 6.0-6.8 TB/s
// for a plain streaming read of the same buffers.
#include "common.h"
#include "fused_ring.h"

namespace lb {

namespace {

typedef void (*LaunchFn)(const Dims&, int64_t, int, size_t, const Buffers&, const APassArgs&, hipStream_t, hipEvent_t, hipEvent_t);

struct Variant {
    int dtype;          // LBFGSB_F64 / LBFGSB_F32
    int logistic;       // 1: the kernel instantiated for the logistic row operations, 0: for the quadratic ones
    int trans;          // 1: with the transposed accumulation, 0: row products only (quadratic form, symmetric matrix)
    int nt, kc, r;      // threads, 16-byte chunks per thread and row, rows per stage
    int wgs_per_cu;     // workgroups per compute unit the launch is sized for
    // [.][0] rows on 16-byte boundaries and whole chunks, [.][1] rows that start on any element, any number of columns (null:
    // none); [0][.] with non-temporal loads of the matrix, [1][.] with ordinary ones (matrix_cached)
    const void* kernel[2][2]; // for hipFuncSetAttribute
    LaunchFn launch[2][2];
    size_t (*lds)(int64_t cols);
    // logistic only: the instantiation for the direction pass (same geometry, deeper ring: its row operation is
    // one exponential and one division, which leaves the registers for it)
    const void* kernel_dir[2][2];
    LaunchFn launch_dir[2][2];
};

template <typename T, int NT, int KCU, int U, int R, int NB, int WPE, int LOGI, int KR, bool TRANS, bool ANY, bool CACHED>
void launch_variant(const Dims& dm, int64_t rows_per_wg, int blocks, size_t lds, const Buffers& bf, const APassArgs& a,
                    hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    hipExtLaunchKernelGGL((ring::k_fused_ring<T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, ANY, CACHED>), dim3(blocks), dim3(NT), lds, st, ev0, ev1,
                          0, (const T*)a.A, dm.ld, dm.rows, dm.cols, rows_per_wg, a, bf.scal, bf.row, bf.t, bf.wpart,
                          bf.losspart);
}

#define LB_KERNEL(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, ANY, CACHED)                                                   \
    (const void*)ring::k_fused_ring<T, NT, KCU, U, R, NB, WPE, LOGI, KR, (TRANS) != 0, ANY, CACHED>
#define LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, ANY, CACHED)                                                   \
    launch_variant<T, NT, KCU, U, R, NB, WPE, LOGI, KR, (TRANS) != 0, ANY, CACHED>
#define LB_KERNELS(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS)                                                               \
    {{LB_KERNEL(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, false, false), LB_KERNEL(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, true, false)},  \
     {LB_KERNEL(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, false, true), LB_KERNEL(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, true, true)}},   \
    {{LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, false, false), LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, true, false)},  \
     {LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, false, true), LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS, true, true)}}
#define LB_VARIANT_FULL(dt, LOGI, T, NT, KCU, U, R, NB, WPE, WGS, KR, TRANS)                                                \
    {dt, LOGI, TRANS, NT, (KCU) * (U), R, WGS, LB_KERNELS(T, NT, KCU, U, R, NB, WPE, LOGI, KR, TRANS),                       \
     ring::lds_bytes<T, NT, (KCU) * (U), KR, R>, {}, {}}
#define LB_VARIANT_LOGI(dt, T, NT, KCU, U, R, NB, NBDIR, WPE, WGS)                                                           \
    {dt, 1, 1, NT, (KCU) * (U), R, WGS, LB_KERNELS(T, NT, KCU, U, R, NB, WPE, 1, 0, 1),                                      \
     ring::lds_bytes<T, NT, (KCU) * (U), 0, R>, LB_KERNELS(T, NT, KCU, U, R, NBDIR, WPE, 2, 0, 1)}
#define LB_VARIANT_KR(dt, LOGI, T, NT, KCU, U, R, NB, WPE, WGS, KR) LB_VARIANT_FULL(dt, LOGI, T, NT, KCU, U, R, NB, WPE, WGS, KR, 1)
#define LB_VARIANT(dt, LOGI, T, NT, KCU, U, R, NB, WPE, WGS) LB_VARIANT_FULL(dt, LOGI, T, NT, KCU, U, R, NB, WPE, WGS, 0, 1)
// (a quadratic form is not read with ordinary loads: matrix_cached)
#define LB_VARIANT_ROWS(dt, T, NT, KCU, U, R, NB, WPE, WGS)                                                                  \
    {dt, 0, 0, NT, (KCU) * (U), R, WGS,                                                                                      \
     {{LB_KERNEL(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, false, false), LB_KERNEL(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, true, false)}, {}},  \
     {{LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, false, false), LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, true, false)}, {}},  \
     ring::lds_bytes<T, NT, (KCU) * (U), 0, R>, {}, {}}
#define LB_VARIANT_ROWS_ALIGNED(dt, T, NT, KCU, U, R, NB, WPE, WGS)                                                          \
    {dt, 0, 0, NT, (KCU) * (U), R, WGS,                                                                                      \
     {{LB_KERNEL(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, false, false), nullptr}, {}},                                           \
     {{LB_LAUNCH(T, NT, KCU, U, R, NB, WPE, 0, 0, 0, false, false), nullptr}, {}},                                           \
     ring::lds_bytes<T, NT, (KCU) * (U), 0, R>, {}, {}}

// Ordered by capacity within a (matrix type, objective family) group: the first variant of the group
// whose NT*KC*VEC columns cover a row and whose LDS need (v for every column) fits is used.  (Narrower rows --
// narrow_shape_ok: up to 1536 fp32, 1024 or 768 fp64 columns -- have a kernel of their own, narrow.h; they come here
// only with a leading dimension past 2^24.)
// What a pass over a tile that is not full pays: the chunks past the row's end are loads of its last chunk (the cache serves
// them) and multiplications by zero, and they hold ring slots that could be rows in flight.  Between two widths that lie
// apart by 1.6 or more there is therefore a variant where one leaves the ring as deep or deeper and measured faster, two under
// twenty chunks in 64 bits and ten in 32 for the quadratic kinds (the second gives 3 to 4 %, 8 % in 32 bits); four chunks under
// five, six or seven under ten in 64 bits and sixteen under twenty measured the same or slower and are not there (the fp32
// logistic ones under five chunks, 2 to 8 % faster, are).  Whole iterations, us, before / now: fp32 50001 x 3001 149 / 137, 50000 x 2500 145 / 121, 30000 x 2100 104 / 83, 50000 x 5500 249 /
// 220, 25000 x 11001 264 / 225, 20000 x 13000 239 / 219; fp64 20000 x 2500 108 / 100 (2900: the same), 20000 x 11000 377 /
// 344, 20000 x 13000 415 / 398, 20000 x 14200 442 / 428; logistic fp32 100000 x 2500 297 / 230, 100001 x 3001 307 / 275,
// 80000 x 3400 241 / 231, 40000 x 6000 252 / 200, 40000 x 7000 256 / 236, 20000 x 12000 229 / 205, fp64 100000 x 1500 262 /
// 234, 60000 x 2500 283 / 239, 20000 x 11000 384 / 345.
// The logistic evaluation kernels spend ~100 registers on exp/log1p, so their rings are shallower; the direction
// pass of the logistic objective has its own instantiation with the deepest ring that does not spill.
const Variant kVariants[] = {
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 2, 1, 4, 8, 2, 1),    // cols <=  2048
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 3, 1, 2, 4, 2, 1),    // cols <=  3072
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 5, 1, 2, 4, 2, 1),    // cols <=  5120
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 10, 1, 1, 2, 2, 1),   // cols <= 10240
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 12, 1, 1, 1, 2, 1),   // cols <= 12288
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 14, 1, 1, 1, 2, 1),   // cols <= 14336
    LB_VARIANT(LBFGSB_F64, 0, double, 512, 20, 1, 1, 1, 2, 1),   // cols <= 20480 (LDS: <= 20428)
    LB_VARIANT_KR(LBFGSB_F64, 0, double, 512, 22, 1, 1, 1, 2, 1, 3),   // cols <= 22528, v of the last 3 chunks in registers
    LB_VARIANT_KR(LBFGSB_F64, 0, double, 512, 24, 1, 1, 1, 2, 1, 5),   // cols <= 24576, v of the last 5 chunks in registers
    LB_VARIANT(LBFGSB_F32, 0, float, 256, 2, 1, 4, 12, 2, 2),    // cols <=  2048 (the geometry of the logistic direction pass)
    LB_VARIANT(LBFGSB_F32, 0, float, 256, 3, 1, 4, 4, 2, 2),     // cols <=  3072
    LB_VARIANT(LBFGSB_F32, 0, float, 256, 5, 1, 1, 2, 2, 2),     // cols <=  5120
    LB_VARIANT(LBFGSB_F32, 0, float, 512, 3, 1, 2, 4, 2, 1),     // cols <=  6144
    LB_VARIANT(LBFGSB_F32, 0, float, 512, 5, 1, 2, 4, 2, 1),     // cols <= 10240
    LB_VARIANT(LBFGSB_F32, 0, float, 512, 6, 1, 1, 2, 2, 1),     // cols <= 12288
    LB_VARIANT(LBFGSB_F32, 0, float, 512, 7, 1, 1, 2, 2, 1),     // cols <= 14336
    LB_VARIANT(LBFGSB_F32, 0, float, 512, 10, 1, 1, 2, 2, 1),    // cols <= 20480 (LDS: <= 20428)
    //              (…, R, ring depth of the evaluation kernel, of the direction kernel, …)
    LB_VARIANT_LOGI(LBFGSB_F64, double, 256, 2, 1, 4, 8, 12, 2, 2),    // cols <=  1024
    LB_VARIANT_LOGI(LBFGSB_F64, double, 256, 3, 1, 2, 4, 6, 2, 2),     // cols <=  1536
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 2, 1, 4, 4, 8, 2, 1),     // cols <=  2048
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 3, 1, 2, 4, 6, 2, 1),     // cols <=  3072
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 5, 1, 1, 2, 4, 2, 1),     // cols <=  5120
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 10, 1, 1, 1, 2, 2, 1),    // cols <= 10240
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 12, 1, 1, 1, 2, 2, 1),    // cols <= 12288
    LB_VARIANT_LOGI(LBFGSB_F64, double, 512, 20, 1, 1, 1, 1, 2, 1),    // cols <= 20480 (LDS: <= 20428)
    LB_VARIANT_LOGI(LBFGSB_F32, float, 256, 2, 1, 4, 8, 12, 2, 2),     // cols <=  2048
    LB_VARIANT_LOGI(LBFGSB_F32, float, 256, 3, 1, 2, 2, 4, 2, 2),      // cols <=  3072
    LB_VARIANT_LOGI(LBFGSB_F32, float, 256, 4, 1, 2, 2, 4, 2, 2),      // cols <=  4096
    LB_VARIANT_LOGI(LBFGSB_F32, float, 256, 5, 1, 1, 2, 4, 2, 2),      // cols <=  5120
    LB_VARIANT_LOGI(LBFGSB_F32, float, 512, 3, 1, 2, 4, 6, 2, 1),      // cols <=  6144
    LB_VARIANT_LOGI(LBFGSB_F32, float, 512, 4, 1, 2, 2, 4, 2, 1),      // cols <=  8192
    LB_VARIANT_LOGI(LBFGSB_F32, float, 512, 5, 1, 1, 2, 4, 2, 1),      // cols <= 10240
    LB_VARIANT_LOGI(LBFGSB_F32, float, 512, 6, 1, 1, 2, 2, 2, 1),      // cols <= 12288
    LB_VARIANT_LOGI(LBFGSB_F32, float, 512, 10, 1, 1, 1, 2, 2, 1),     // cols <= 20480 (LDS: <= 20428)
    // row products only: no accumulators of w, so the ring is deeper (4096 to 15872 columns: symmetric.hip).  A form of
    // a few thousand variables is in the caches: rows in flight count, not bytes.  Pass, us, in the tile for 5120 columns / in
    // its own (mean over a solve, launches that find it finished among them): fp64 n = 1200 12.4 / 7.8, 2000 13.7 / 9.9, 2400
    // 19.9 / 13.8, 3000 21.7 / 16.3, 4000 25.5 / 22.2; fp32 1200 12.2 / 9.9, 2000 12.5 / 10.2, 3000 14.9 / 12.3, 4000 17.6 /
    // 14.9.  The two-pass
    // organisation reads A once for these too (no transposed pass), and on rows that start on any element its kernel of four
    // rows per wave is the faster one while the caches serve much of the matrix.  Whole iterations, us, ring / k_gemv: fp64
    // n = 301 25.0 / 22.4, 1025 41.5 / 38.0, 2201 50.0 / 45.0, 3001 53.0 / 48.8, 4095 59.1 / 54.7, 15873 347 / 377, 20001
    // 535 / 630; fp32 301 25.0 / 22.1, 1025 40.8 / 37.0, 2001 42.6 / 40.6, 2501 43.8 / 42.8, 2801 44.7 / 45.6, 4095 48.8 / 50.3.
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F64, double, 256, 2, 1, 4, 8, 4, 4),  // cols <=  1024
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F64, double, 256, 4, 1, 2, 4, 4, 2),  // cols <=  2048
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F64, double, 512, 3, 1, 2, 6, 2, 1),  // cols <=  3072
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F64, double, 512, 4, 1, 1, 4, 2, 1),  // cols <=  4096
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F64, double, 512, 5, 1, 2, 8, 2, 1),  // cols <=  5120
    LB_VARIANT_ROWS(LBFGSB_F64, double, 512, 20, 1, 1, 2, 2, 1), // cols <= 20480 (LDS: <= 20428)
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F32, float, 256, 1, 1, 4, 8, 4, 4),   // cols <=  1024
    LB_VARIANT_ROWS_ALIGNED(LBFGSB_F32, float, 256, 2, 1, 4, 8, 4, 4),   // cols <=  2048
    LB_VARIANT_ROWS(LBFGSB_F32, float, 256, 3, 1, 2, 6, 2, 2),   // cols <=  3072, on any element from kRowsAnyMin on
    LB_VARIANT_ROWS(LBFGSB_F32, float, 256, 4, 1, 1, 4, 2, 2),   // cols <=  4096
    LB_VARIANT_ROWS(LBFGSB_F32, float, 256, 5, 1, 2, 8, 2, 2),   // cols <=  5120, on any element from kRowsAnyMin on
    LB_VARIANT_ROWS(LBFGSB_F32, float, 512, 10, 1, 1, 4, 2, 1),  // cols <= 20480 (LDS: <= 20428)
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr int64_t kRowsAnyMin = 2600;
constexpr size_t kLdsPerWorkgroup = 160 * 1024;   // gfx950

int compute_units() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess &&
            prop.multiProcessorCount > 0)
            cus = prop.multiProcessorCount;
        else
            cus = 256;   // MI355X; also the answer on a machine without a GPU (sizes only)
        (void)hipGetLastError();
    }
    return cus;
}

int64_t rows_per_wg_for(const Dims& dm, const Variant& v) {
    const int64_t slots = (int64_t)compute_units() * v.wgs_per_cu;
    int64_t rpw = (dm.rows + slots - 1) / slots;
    rpw = (rpw + v.r - 1) / v.r * v.r;
    return rpw < v.r ? v.r : rpw;
}

}  // namespace

bool fused_shape_ok(const Dims& dm, bool aligned, int* variant, int* blocks) {
    *variant = -1;
    *blocks = 0;
    const int vec = dm.dtype == LBFGSB_F32 ? 4 : 2;
    if (dm.cols < vec) return false;   // narrower than one 16-byte load (rows may start on any element)
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant& v = kVariants[i];
        if (v.dtype != dm.dtype || v.logistic != (dm.kind == LBFGSB_OBJ_LOGISTIC_L2) ||
            v.trans != (dm.kind != LBFGSB_OBJ_QP))
            continue;
        if ((int64_t)v.nt * v.kc * vec < dm.cols) continue;
        if (v.lds(dm.cols) > kLdsPerWorkgroup - 256) continue;   // (a few bytes of static LDS come on top)
        if (!aligned && (!v.launch[0][1] || (!v.trans && dm.cols < kRowsAnyMin))) return false;
        const int64_t rpw = rows_per_wg_for(dm, v);
        *variant = i;
        *blocks = (int)((dm.rows + rpw - 1) / rpw);
        return true;
    }
    return false;
}

// The kernels use more dynamic LDS than the default limit of a launch.  The limit is a property of the
// kernel, not of a solver, and several solvers of different widths may share a variant: it is raised to the
// most the variant can ever ask for (its widest row, capped by what a workgroup can have).
hipError_t fused_prepare(const Dims& dm, const Geometry& ge) {
    if (ge.narrow_variant >= 0 || ge.sym_strips > 0) return hipSuccess;   // (static LDS only)
    const Variant& v = kVariants[ge.fused_variant];
    const int vec = v.dtype == LBFGSB_F32 ? 4 : 2;
    size_t most = v.lds((int64_t)v.nt * v.kc * vec);
    const size_t cap = kLdsPerWorkgroup - 256;   // the kernels also hold a few bytes of static LDS
    if (most > cap) most = cap;
    if (v.lds(dm.cols) > most) most = v.lds(dm.cols);
    const int any = ge.vec == 1, cached = matrix_cached(dm);
    hipError_t e = hipFuncSetAttribute(v.kernel[cached][any], hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    if (e == hipSuccess && v.kernel_dir[cached][any])   // (may also hold two numbers per row of a workgroup: whatever fits)
        e = hipFuncSetAttribute(v.kernel_dir[cached][any], hipFuncAttributeMaxDynamicSharedMemorySize, (int)cap);
    return e;
}

// LDS the logistic direction pass needs on top when it also sums the loss differences of the first trial step:
// two numbers per row of a workgroup
static size_t ls_first_lds(const Dims& dm, const Variant& v) { return (size_t)rows_per_wg_for(dm, v) * 16; }

bool fused_ls_first_ok(const Dims& dm, const Geometry& ge) {
    if (ge.narrow_variant >= 0) return true;
    const Variant& v = kVariants[ge.fused_variant];
    return v.launch_dir[0][0] && v.lds(dm.cols) + ls_first_lds(dm, v) <= kLdsPerWorkgroup - 256;
}

void launch_fused(const Dims& dm, const Geometry& ge, const Buffers& bf, const APassArgs& a, hipStream_t st,
                  hipEvent_t ev0, hipEvent_t ev1) {
    if (ge.sym_strips > 0) {
        launch_sym(dm, ge, bf, a, st, ev0, ev1);
        return;
    }
    if (ge.narrow_variant >= 0) {
        launch_narrow(dm, ge, bf, a, nullptr, st, ev0, ev1);
        return;
    }
    const Variant& v = kVariants[ge.fused_variant];
    const int any = ge.vec == 1, cached = matrix_cached(dm);
    auto launch = (a.mode == kRowLogiSpec && v.launch_dir[cached][any]) ? v.launch_dir[cached][any] : v.launch[cached][any];
    const size_t extra = a.mode == kRowLogiSpec && a.ls_first ? ls_first_lds(dm, v) : 0;
    launch(dm, rows_per_wg_for(dm, v), ge.fused_blocks, v.lds(dm.cols) + extra, bf, a, st, ev0, ev1);
}

}  // namespace lb
