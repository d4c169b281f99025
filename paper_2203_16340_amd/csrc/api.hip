// C-ABI layer of liblbfgsb: argument checks, workspace layout, the fixed kernel sequence of one
// iteration of Algorithm 1, the loops of lbfgsb_solve and of the augmented Lagrangian that follow the device and the primitive-level hooks.
// No solver arithmetic happens on the host.
#include <sched.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "common.h"

using namespace lb;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                           \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess) return fail(LBFGSB_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kMaxTimed = 4096;

// Host memory that kernels write while the host looks at it: coherent by request, not by the runtime's default (which the
// environment can change).
constexpr unsigned kPinned = hipHostMallocCoherent;

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

// Workspace of lbfgsb_solve_static, for callers that cannot allocate.  In host code this name is only a stand-in
// for the symbol: the device address comes from hipGetSymbolAddress, once per device (static_slot()), and that
// address is what every kernel argument, fill and copy uses.
// (No `used` attribute: it keeps the symbol local in the code object, and the runtime, which finds a device variable
// by name among the code object's global symbols, then aborts in hipGetSymbolAddress.  The host code's use of the
// variable is what makes the compiler export it.)
static __device__ __align__(256) unsigned char scratch[LBFGSB_STATIC_SCRATCH_BYTES];

struct lbfgsb_solver {
    Dims dm;
    Opts op;
    lbfgsb_options options;
    lbfgsb_objective obj;
    Geometry ge;
    Buffers bf;
    hipStream_t stream;
    Scal* h_scal;            // host copy (pinned, allocated by lbfgsb_create)
    bool owns_h_scal;
    int* h_flag;             // pinned, behind the host copy: kernels report a start point that is no good (null: not pinned)
    unsigned long long* h_progress;   // pinned, behind it: the last step whose outcome is known, and the status then
    int use_fused;
    int use_resident;        // small least squares: whole iterations in one resident workgroup
    // logistic objective on the fused pass: steps still to be enqueued with the full launch sequence (after a
    // rejected first trial step), and short-sequence steps enqueued since the host last looked at the scalar block
    int logi_full_left;
    int short_steps_unseen;
    bool short_ok;           // the short sequence is available (the pass has the LDS for its per-row numbers)
    bool commit_needed;      // resident solver: a kernel of the multi-kernel path may have left an update pending
    // lbfgsb_solve: steps enqueued since it began, redone ones included (Opts::seq), and the next one to report
    unsigned steps_enqueued = 0, note_at = 0;
    // the last launch that touched x, g or the pairs has left the next Gram kernel's records (launch_update_gram_gauss, _form)
    bool gram_ready = false;
    // a graph may hold steps of this solver: its replays move the state unseen, so whether there are records is asked on the device
    // from then on (Scal::gram_left), by a launch that returns at once where there are
    bool recorded = false;
    int steps_since_refresh;
    long long steps_since_set_x;
    bool x_set;
    // timing
    bool timing;
    std::vector<hipEvent_t> ev0, ev1;
    int timed;
    bool steps_only;         // nothing but lbfgsb_step since the records were discarded: a solver still running has timed no launch in vain
};

namespace {

// objective is a quadratic along every direction: closed-form line search, gradient carried by recurrence
bool is_quadratic(int kind) { return kind != LBFGSB_OBJ_LOGISTIC_L2 && kind != LBFGSB_OBJ_OT_ENTROPY; }

int check_objective(int64_t n, int m, const lbfgsb_objective* o) {
    if (!o) return fail(LBFGSB_E_INVALID_ARG, "objective is NULL");
    if (n <= 0) return fail(LBFGSB_E_INVALID_ARG, "n must be positive (got %lld)", (long long)n);
    if (m <= 0 || m > LBFGSB_MAX_M) return fail(LBFGSB_E_INVALID_ARG, "m must be in 1..%d (got %d)", LBFGSB_MAX_M, m);
    if (o->kind < LBFGSB_OBJ_LSQ || o->kind > LBFGSB_OBJ_OT_ENTROPY)
        return fail(LBFGSB_E_INVALID_ARG, "unknown objective kind %d", o->kind);
    if (o->kind == LBFGSB_OBJ_QP && o->rows != o->cols)
        return fail(LBFGSB_E_INVALID_ARG, "the quadratic form needs a square matrix (got %lld x %lld)", (long long)o->rows,
                    (long long)o->cols);
    if (o->n_extra < 0 || o->n_extra > kMaxExtra) return fail(LBFGSB_E_INVALID_ARG, "n_extra must be in 0..%d", kMaxExtra);
    if (o->n_extra > 0 && (o->kind == LBFGSB_OBJ_LOGISTIC_L2 || is_transport(o->kind)))
        return fail(LBFGSB_E_INVALID_ARG, "extra rows go with the least-squares and quadratic-form kinds");
    if (is_transport(o->kind) && !(o->lambda > 0.0))
        return fail(LBFGSB_E_INVALID_ARG, "the transport kinds need lambda > 0");
    if (o->dtype != LBFGSB_F64 && o->dtype != LBFGSB_F32) return fail(LBFGSB_E_INVALID_ARG, "unknown dtype %d", o->dtype);
    if (o->rows <= 0 || o->cols <= 0) return fail(LBFGSB_E_INVALID_ARG, "rows and cols must be positive");
    if (o->rows > (1ll << 31) - 1 || o->cols > (1ll << 31) - 1) return fail(LBFGSB_E_INVALID_ARG, "rows/cols exceed 2^31-1");
    if (o->ld < o->cols) return fail(LBFGSB_E_INVALID_ARG, "ld (%lld) < cols (%lld)", (long long)o->ld, (long long)o->cols);
    if (is_transport(o->kind) && o->rows > ((1ll << 40) / o->cols))
        return fail(LBFGSB_E_INVALID_ARG, "rows*cols exceeds 2^40 variables");
    const int64_t expect = is_transport(o->kind) ? o->rows * o->cols
                         : o->kind == LBFGSB_OBJ_LSQ_L1SPLIT ? 2 * o->cols : o->cols;
    if (n != expect) return fail(LBFGSB_E_INVALID_ARG, "n = %lld does not match the objective (%lld variables)", (long long)n, (long long)expect);
    return LBFGSB_OK;
}

int check_options(const lbfgsb_options* o) {
    if (!(o->eps >= 0.0) || !(o->armijo_c1 > 0.0 && o->armijo_c1 < 1.0) || !(o->backtrack > 0.0 && o->backtrack < 1.0) ||
        o->max_backtracks < 0 || !(o->tol >= 0.0) || o->max_iter < 0 || o->refresh_every < 0 || o->poll_every < 1 ||
        o->a_pass < LBFGSB_APASS_AUTO || o->a_pass > LBFGSB_APASS_RESIDENT)
        return fail(LBFGSB_E_INVALID_ARG, "bad option value");
    return LBFGSB_OK;
}

// Which rows may be read once only.  lbfgsb_solve_static, whose workspace is fixed, does with less where the partial columns
// of the kernels for rows on any element would not fit: the two-pass kernels, which it ran for such rows before there were
// any, leave fewer; and the Gram kernel on long vectors gets half the workgroups, whose records take no more than those of the
// kernel that odd lengths had before.  (Rows on 16-byte boundaries are left the ring kernel, which needs no less: at the widths of the other
// two the partial columns of the transposed pass, for which the workspace has room as well, are at least as many.)
enum SingleRead { kReadAligned = 0,   // rows on 16-byte boundaries, by the ring kernel
                  kReadAny = 1 };     // any rows; also the kernels for short rows and for symmetric matrices
Geometry make_geometry(const Dims& dm, const void* A, SingleRead reads = kReadAny) {
    Geometry ge{};
    const int per16 = dm.dtype == LBFGSB_F32 ? 4 : 2;
    const bool aligned = ((uintptr_t)A % 16 == 0) && (dm.cols % per16 == 0) && (dm.ld % per16 == 0);
    ge.vec = aligned ? per16 : 1;
    int64_t gb = (dm.rows + kWaves * 4 - 1) / (kWaves * 4);
    ge.gemv_blocks = (int)(gb > 2048 ? 2048 : gb);
    const int64_t cols_per_tile = (int64_t)kBlock * ge.vec;
    ge.gemvt_col_tiles = (int)((dm.cols + cols_per_tile - 1) / cols_per_tile);
    int64_t rb = 2048 / ge.gemvt_col_tiles;
    const int64_t rb_max = (dm.rows + 31) / 32;
    if (rb > rb_max) rb = rb_max;
    if (rb > 512) rb = 512;
    if (rb < 1) rb = 1;
    ge.gemvt_rows_per_block = (dm.rows + rb - 1) / rb;
    ge.gemvt_row_blocks = (int)((dm.rows + ge.gemvt_rows_per_block - 1) / ge.gemvt_rows_per_block);
    const bool any = reads == kReadAny;
    int strips = 0, grid = 0, nv, nb;
    const bool sym = any && sym_shape_ok(dm, &strips, &grid);
    ge.fused_ok = !is_transport(dm.kind) && (aligned || any) &&
                  (fused_shape_ok(dm, aligned, &ge.fused_variant, &ge.fused_blocks) || sym) ? 1 : 0;
    ge.narrow_variant = -1;
    if (ge.fused_ok && any && narrow_shape_ok(dm, &nv, &nb)) { ge.narrow_variant = nv; ge.fused_blocks = nb; }
    if (sym) { ge.sym_strips = strips; ge.fused_blocks = grid; }
    ge.gram_blocks = gram_blocks_for(dm.n, dm.m, !any);
    int64_t db = (dm.n + kBlock - 1) / kBlock;
    ge.dir_blocks = (int)(db > kDirBlocksMax ? kDirBlocksMax : db);
    int64_t ub = (dm.cols + 15) / 16;   // 16 columns per workgroup in the column-sum kernels
    ge.upd_blocks = ge.fin_blocks = (int)(ub > 2048 ? 2048 : ub);
    int64_t lb_ = (dm.rows + kBlock - 1) / kBlock;
    // (The line search ends in a single-address arrival: few workgroups, until the transcendental functions of the rows
    // outweigh it.  10^6 rows, first trial step in a sweep of its own: 35 us with 128 workgroups, 22 with 512.)
    const int64_t ls_cap = dm.rows > (1 << 18) ? 512 : 128;
    ge.ls_blocks = (int)(lb_ > ls_cap ? ls_cap : lb_);
    ge.lrows_blocks = (int)(lb_ > 512 ? 512 : lb_);   // the margins' update has no such ending: 512 measured faster than 128
    {
        // workgroups for the columns plus workgroups for the margins (four rows per thread), at most 512 in all
        int64_t rb4 = (dm.rows + 4 * kBlock - 1) / (4 * kBlock);
        int64_t tot = rb4 + ge.upd_blocks;
        ge.updl_blocks = (int)(tot > 512 ? 512 : tot);
    }
    if (is_transport(dm.kind)) {
        int rpw = 1;
        while (rpw < kOtRpwMax && (dm.rows + rpw - 1) / rpw > 512) rpw *= 2;
        ge.ot_rpw = rpw;
        ge.ot_row_blocks = (int)((dm.rows + rpw - 1) / rpw);
        int64_t cb = (dm.cols + kCX - 1) / kCX;
        ge.ot_col_blocks = (int)(cb > 2048 ? 2048 : cb);
        ge.ot_el_blocks = ot_entry_blocks(dm);
        int64_t eb = (dm.n + ot_threads(dm) - 1) / ot_threads(dm);
        ge.ls_blocks = (int)(eb > 512 ? 512 : eb);
    }
    return ge;
}

struct Layout {
    size_t scal, scal_next, x, g, l, u, d, p1, p2, mask, S, Y, row, t, psi, wpart, losspart, grampart, redpart, lspart, wextra, xres, hist, total;
};

Layout make_layout(const Dims& dm, const Geometry& ge) {
    Layout L{};
    size_t off = 0;
    // (wextra / xres are appended at the end so that the offsets of everything else do not depend on n_extra)
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    const size_t nb = (size_t)dm.n * 8, rb = (size_t)row_entries(dm.kind, dm.rows, dm.cols) * 8;
    L.scal = take(sizeof(Scal));
    L.scal_next = take(sizeof(Scal));
    L.x = take(nb); L.g = take(nb); L.l = take(nb); L.u = take(nb); L.d = take(nb); L.p1 = take(nb); L.p2 = take(nb);
    L.mask = take((size_t)dm.n);
    L.S = take(nb * dm.m); L.Y = take(nb * dm.m);
    L.row = take(rb); L.t = take(rb); L.psi = take(rb);
    int wparts = ge.gemvt_row_blocks;
    if (ge.fused_ok && ge.sym_strips == 0 && ge.fused_blocks > wparts) wparts = ge.fused_blocks;
    if (is_transport(dm.kind)) wparts = ge.ot_row_blocks;
    size_t wdoubles = (size_t)wparts * dm.cols;
    if (ge.sym_strips > 0 && sym_workspace(dm, ge) > wdoubles) wdoubles = sym_workspace(dm, ge);
    L.wpart = take(wdoubles * 8);
    int lparts = ge.gemv_blocks;
    if (ge.fused_ok && ge.fused_blocks > lparts) lparts = ge.fused_blocks;
    if (ge.sym_strips > 0 && sym_loss_parts(dm) > lparts) lparts = sym_loss_parts(dm);
    if (ge.ls_blocks > lparts) lparts = ge.ls_blocks;
    if (ge.lrows_blocks > lparts) lparts = ge.lrows_blocks;
    if (is_transport(dm.kind) && ge.ot_row_blocks + ge.ot_col_blocks > lparts) lparts = ge.ot_row_blocks + ge.ot_col_blocks;
    L.losspart = take((size_t)lparts * 8);
    L.grampart = take(gram_partial_bytes(ge.gram_blocks, dm.m));
    size_t red = (size_t)ge.dir_blocks * (8 + 2 * kFoldMax);
    if ((size_t)ge.upd_blocks * 2 > red) red = (size_t)ge.upd_blocks * 2;
    if ((size_t)ge.updl_blocks * 2 > red) red = (size_t)ge.updl_blocks * 2;
    if (is_transport(dm.kind) && (size_t)ge.ot_el_blocks > red) red = (size_t)ge.ot_el_blocks;
    L.redpart = take(red * 8);
    L.lspart = take((size_t)ge.ls_blocks * 64 * 8);   // up to 64 step lengths per sweep (entropy line search)
    L.wextra = take(dm.n_extra > 0 ? (size_t)dm.n * 8 : 8);
    L.xres = take((size_t)(dm.n_extra + 1) * 8);
    L.hist = take((size_t)LBFGSB_HISTORY_CAPACITY * sizeof(lbfgsb_iter_record));
    L.total = off;
    return L;
}

Dims make_dims(int64_t n, int m, const lbfgsb_objective* o) {
    Dims dm{};
    dm.n = n; dm.rows = o->rows; dm.cols = o->cols; dm.ld = o->ld; dm.m = m; dm.kind = o->kind; dm.dtype = o->dtype;
    dm.lambda = o->lambda; dm.mu = o->mu;
    dm.n_extra = (int)o->n_extra;
    return dm;
}

void enqueue_step(lbfgsb_solver* s);

// Logistic objective on the single-read pass: the columns X^T psi of an accepted step that was not the first trial step
// (returns at once when it was).
void enqueue_redo_columns(lbfgsb_solver* s) {
    if (s->ge.narrow_variant >= 0) {
        APassArgs a{};
        a.A = s->obj.A;
        a.mode = kRowPsiGiven;
        a.check_status = 2;
        launch_narrow(s->dm, s->ge, s->bf, a, s->bf.psi, s->stream);
    } else {
        launch_gemvt_from(s->dm, s->ge, s->bf, s->obj.A, s->bf.psi, 2, s->stream, nullptr, nullptr);
    }
}

// A problem that backtracks once tends to do so again: this many steps behind a rejected first trial step take the full
// launch sequence.  Counted from the step that was rejected, so that which steps take which sequence does not depend on how many
// had been enqueued when the host found out (an accepted first trial step is the same in both, f included).
constexpr int kLogiFullSteps = 8;
// Steps enqueued again between two looks at the device: those behind a further rejection have to be enqueued a third time.
constexpr int kRedoBatch = 16;

// Reads the scalar block after applying any update the last step left pending.  If the short logistic launch sequence
// has parked the solver (first trial step rejected: kStatusBail), the iteration is finished here with the launches
// that sequence leaves out, the steps that found the solver parked are enqueued again, and the block is read anew.
hipError_t read_scal(lbfgsb_solver* s) {
    int owed = 0;   // steps that found the solver parked and have not been enqueued again
    for (;;) {
        // (the resident solver applies its updates itself; only its evaluations by the multi-kernel path leave one pending)
        hipError_t e = hipSuccess;
        if (s->owns_h_scal) {
            launch_commit(s->dm, s->bf, s->stream, s->h_scal);   // (writes the pinned host copy itself)
        } else {
            if (!s->use_resident || s->commit_needed) launch_commit(s->dm, s->bf, s->stream);
            e = hipMemcpyAsync(s->h_scal, s->bf.scal, sizeof(Scal), hipMemcpyDeviceToHost, s->stream);
            if (e != hipSuccess) return e;
        }
        s->commit_needed = false;
        e = hipStreamSynchronize(s->stream);
        if (e != hipSuccess) return e;
        s->short_steps_unseen = 0;
        if (s->h_scal->status == kStatusBail) {
            owed += s->h_scal->bail_skipped;
            launch_clear_bail(s->bf, s->stream);
            // the rest of the interrupted iteration: more step lengths, new margins and row weights, the transposed
            // pass for the accepted step, the update
            launch_ls_logistic(s->dm, s->op, s->ge, s->bf, s->obj.b, 1, 2, 0, s->stream);
            launch_rows_logistic(s->dm, s->ge, s->bf, s->obj.b, 0, s->stream);
            enqueue_redo_columns(s);
            launch_update_logistic(s->dm, s->op, s->ge, s->bf, 0, 0, s->stream);
            s->logi_full_left = kLogiFullSteps;
        } else if (owed == 0 || s->h_scal->status != LBFGSB_RUNNING) {
            return hipSuccess;
        }
        const int now = owed < kRedoBatch ? owed : kRedoBatch;
        owed -= now;
        for (int k = 0; k < now; ++k) enqueue_step(s);
    }
}

// Uploads a fresh scalar block (host template in h_scal) and waits for it.
hipError_t write_scal(lbfgsb_solver* s) {
    hipError_t e = hipMemcpyAsync(s->bf.scal, s->h_scal, sizeof(Scal), hipMemcpyHostToDevice, s->stream);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(s->stream);
}

void fill_info(const Scal& sc, lbfgsb_info* info) {
    info->status = sc.status; info->iters = sc.iters; info->fevals = sc.fevals; info->f = sc.f;
    info->pg2 = sc.pg2; info->pginf = sc.pginf; info->n_fixed = sc.n_fixed; info->branch = sc.branch;
    info->backtracks = sc.backtracks; info->pairs_used = sc.pairs_used; info->memory_resets = sc.memory_resets;
    info->alpha = sc.alpha; info->alpha_ub = sc.alpha_ub; info->gp = sc.gp;
}

// Events for the next launch of a kernel that reads A (null when timing is off or the store is full).
struct TimedSlot {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    explicit TimedSlot(lbfgsb_solver* s, bool wanted = true) {
        if (wanted && s->timing && s->timed < kMaxTimed) {
            e0 = s->ev0[s->timed];
            e1 = s->ev1[s->timed];
            s->timed++;
        }
    }
};

APassArgs base_args(const lbfgsb_solver* s) {
    APassArgs a{};
    a.A = s->obj.A; a.b = s->obj.b;
    a.w = (s->dm.kind == LBFGSB_OBJ_LSQ || s->dm.kind == LBFGSB_OBJ_LSQ_L1SPLIT) ? s->obj.row_weight : nullptr;
    a.vs = s->dm.kind == LBFGSB_OBJ_QP ? s->obj.sign : nullptr;
    a.p1 = s->bf.p1; a.p2 = s->bf.p2;
    a.split = s->dm.kind == LBFGSB_OBJ_LSQ_L1SPLIT;
    return a;
}

OtArgs ot_args(const lbfgsb_solver* s) {
    return OtArgs{s->obj.A, s->obj.b, s->obj.row_weight};
}

// f, g (and the residual / margins) from scratch at the current x.  fresh: the scalar block holds no pending update.  reopen: the
// solver has stopped there and is to go on, unless *over (or null) is set (not the transport kinds).  host_flag: whether the gradient is
// finite is reported there.
void enqueue_eval(lbfgsb_solver* s, int check_status, bool fresh = false, bool reopen = false, int* host_flag = nullptr,
                  const int* over = nullptr) {
    s->gram_ready = false;
    if (!fresh) launch_commit(s->dm, s->bf, s->stream);   // a pending f must not overwrite the one computed here
    if (is_transport(s->dm.kind)) {
        const OtArgs oa = ot_args(s);
        launch_ot_sums(s->dm, s->ge, s->bf, oa, 1, check_status, s->stream);
        launch_ot_eval_finish(s->dm, s->ge, s->bf, oa, s->stream);
        if (host_flag) launch_check_finite(s->dm, s->bf.g, host_flag, s->stream);
        return;
    }
    APassArgs a = base_args(s);
    a.va = s->bf.x;
    a.vb = a.split ? s->bf.x + s->dm.cols : nullptr;
    a.select_p = 0;
    const bool qp = s->dm.kind == LBFGSB_OBJ_QP;
    a.mode = qp ? kRowQpEval : (is_quadratic(s->dm.kind) ? kRowLsqEval : kRowLogiEval);
    a.check_status = check_status;
    if (qp) {
        // symmetric matrix: the gradient needs the row products only
        TimedSlot ts(s);
        if (s->use_fused) launch_fused(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
        else launch_gemv(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
    } else if (s->use_fused) {
        TimedSlot ts(s);
        launch_fused(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
    } else {
        { TimedSlot ts(s); launch_gemv(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1); }
        { TimedSlot ts(s); launch_gemvt_from(s->dm, s->ge, s->bf, s->obj.A, s->bf.psi, check_status, s->stream, ts.e0, ts.e1); }
    }
    if (s->dm.n_extra > 0)
        launch_extra_rows(s->dm, s->bf, s->obj.extra_rows, s->obj.extra_target, s->obj.extra_weight,
                          host_flag ? 2 : 1, s->stream);
    launch_eval_finish(s->dm, s->ge, s->bf, s->obj.b, s->obj.sign, s->stream, reopen, host_flag, over);
}

bool is_recording(const lbfgsb_solver* s) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s->stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusActive;
}

// One iteration of Algorithm 1 as a fixed sequence of launches; nothing here waits for the device.
void enqueue_step(lbfgsb_solver* s) {
    s->op.seq = ++s->steps_enqueued;
    s->op.note = s->op.seq == s->note_at;
    if (s->use_resident) {
        // (the periodic recomputation and the pending-update bookkeeping happen inside the kernel)
        launch_resident(s->dm, s->op, s->bf, s->obj.A, s->obj.b, 1, s->options.refresh_every, s->stream);
        return;
    }
    const bool quad = is_quadratic(s->dm.kind);
    const bool may_leave_gram = update_gram_ok(s->dm);
    if (may_leave_gram && !s->recorded) s->recorded = is_recording(s);
    if (quad && s->options.refresh_every > 0 && s->steps_since_refresh >= s->options.refresh_every) {
        enqueue_eval(s, 1);
        s->steps_since_refresh = 0;
    }
    if (is_transport(s->dm.kind)) {
        // no matrix product: the iteration streams the pair memory twice (Gram matrix, direction) and the
        // iterate-sized vectors a few times.  The Gram kernel is the longest and the one that is timed.
        // (timed only once the pair memory is full, so that every timed launch moves the same bytes)
        // (the Gram kernel ends without its closing step, which the direction kernel does, and that kernel without its own: the
        // row-sum kernel, the first to need Algorithm 2's choice, makes it from the per-workgroup sums)
        const int open_gram = gram_can_skip_close(s->dm) ? 1 : 0;
        if (!s->gram_ready || s->timing || s->recorded) {   // (timed: the sums that the update has left, once more, the same bit for bit)
            TimedSlot ts(s, s->steps_since_set_x >= s->dm.m);
            launch_gram(s->dm, s->op, s->ge, s->bf, 0, 1, s->stream, ts.e0, ts.e1,
                        !open_gram ? kGramClose : (s->timing ? kGramOpen : kGramOpenUnlessLeft));
        }
        launch_dir(s->dm, s->op, s->ge, s->bf, 0, 0, s->stream, nullptr, nullptr, 1, open_gram);
        const OtArgs oa = ot_args(s);
        launch_ot_sums(s->dm, s->ge, s->bf, oa, 0, 1, s->stream, s->ge.dir_blocks, s->op.eps, open_gram ? s->bf.scal_next : nullptr);
        s->gram_ready = may_leave_gram;
        if (s->gram_ready)
            launch_update_gram_gauss(s->dm, s->op, s->ge, s->bf, s->bf.psi, s->ge.ot_row_blocks + s->ge.ot_col_blocks, s->stream);
        else if (quad) launch_ot_update_gauss(s->dm, s->op, s->ge, s->bf, oa, s->stream);
        else launch_ot_step_entropy(s->dm, s->op, s->ge, s->bf, oa, s->stream);
        s->steps_since_refresh++;
        s->steps_since_set_x++;
        return;
    }
    // one or two extra rows ride along with the direction kernel; more get the kernel of their own
    const bool fold = quad && dir_folds_extra_rows(s->dm);
    const double* fold_rows = fold ? s->obj.extra_rows : nullptr;
    // The single-read pass can make Algorithm 2's choice itself from the direction kernel's partial sums, which then
    // needs no closing step (not with extra rows that have a kernel of their own, which reads the choice from the
    // scalar block; rows folded into the direction kernel get their coefficients in the update kernel)
    const bool small = small_step_ok(s->dm);
    const bool pass_chooses = s->ge.narrow_variant >= 0 ? narrow_makes_choice(s->ge)
                                                        : (s->ge.sym_strips == 0 || s->ge.dir_blocks <= kPassDirBlocksMax);
    const bool defer = s->use_fused && pass_chooses && !small && (s->dm.n_extra == 0 || fold);
    // ... and then the Gram kernel needs no closing step either, where its grid is small enough for the direction
    // kernel's workgroups to add its partial sums themselves: they finish its work on private copies of the scalar
    // block, and the pass moves workgroup 0's copy into place (Buffers::scal_next)
    const bool open_gram = defer && gram_can_skip_close(s->dm);
    // ... and the quadratic form's update leaves the next step's records itself, no Gram kernel at all
    const bool update_gram = open_gram && may_leave_gram;
    const bool ready = update_gram && s->gram_ready && !s->recorded;
    s->gram_ready = false;
    if (small) {
        launch_small_step(s->dm, s->op, s->bf, fold_rows, s->obj.extra_weight, s->stream);
    } else {
        if (!ready) launch_gram(s->dm, s->op, s->ge, s->bf, 0, 1, s->stream, nullptr, nullptr, open_gram ? kGramOpenUnlessLeft : kGramClose);
        launch_dir(s->dm, s->op, s->ge, s->bf, 0, 0, s->stream, fold_rows, s->obj.extra_weight, defer ? 1 : 0,
                   open_gram ? 1 : 0);
    }
    APassArgs a = base_args(s);
    a.select_p = 1;
    a.check_status = 1;
    if (defer) {
        a.dir_part = s->bf.redpart; a.dir_blocks = s->ge.dir_blocks; a.eps = s->op.eps;
        if (open_gram) a.scal_next = s->bf.scal_next;
    }
    const int fold_blocks = defer && fold ? s->ge.dir_blocks : 0;   // the update kernel forms the folded rows' coefficients
    if (quad && s->dm.n_extra > 0 && !fold)
        launch_extra_rows(s->dm, s->bf, s->obj.extra_rows, s->obj.extra_target, s->obj.extra_weight, 0, s->stream);
    if (s->dm.kind == LBFGSB_OBJ_QP) {
        a.mode = kRowQpDir;
        {
            TimedSlot ts(s);
            if (s->use_fused) launch_fused(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
            else launch_gemv(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
        }
        if (update_gram) launch_update_gram_form(s->dm, s->op, s->ge, s->bf, s->obj.sign, s->stream, fold_rows, s->obj.extra_weight, fold_blocks);
        else launch_update_quadratic(s->dm, s->op, s->ge, s->bf, s->obj.sign, s->stream, fold_rows, s->obj.extra_weight, fold_blocks);
        s->gram_ready = update_gram;
    } else if (quad) {
        a.mode = kRowDir;
        if (s->use_fused) {
            TimedSlot ts(s);
            launch_fused(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1);
        } else {
            { TimedSlot ts(s); launch_gemv(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1); }
            { TimedSlot ts(s); launch_gemvt_from(s->dm, s->ge, s->bf, s->obj.A, s->bf.psi, 1, s->stream, ts.e0, ts.e1); }
        }
        launch_update_quadratic(s->dm, s->op, s->ge, s->bf, nullptr, s->stream, fold_rows, s->obj.extra_weight, fold_blocks);
    } else if (s->use_fused) {
        // One read of X yields t = X p AND X^T psi for the first trial step min(1, alpha_ub).  The line
        // search over the margins then decides; only if it does not accept that first step does a second
        // (transposed) pass over X run, otherwise that launch returns at once.  The transposed pass is not
        // among the timed launches: it reads A only in the iterations that backtrack.
        a.mode = kRowLogiSpec;
        // (Steps recorded into a graph are not seen by the bookkeeping that redoes parked ones.  Rows on 16-byte
        // boundaries have always been recorded with the short sequence, see lbfgsb_get_x; other rows are recorded with
        // the sequence that finishes every iteration on the device.)
        const bool recording = s->ge.vec == 1 && is_recording(s);
        const bool full = s->logi_full_left > 0 || !s->short_ok || recording;
        a.ls_first = s->short_ok ? 1 : 0;
        const int first_parts = s->short_ok ? s->ge.fused_blocks : 0;
        { TimedSlot ts(s); launch_fused(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1); }
        if (full) {
            if (s->logi_full_left > 0) s->logi_full_left--;
            launch_ls_logistic(s->dm, s->op, s->ge, s->bf, s->obj.b, 1, s->short_ok ? 2 : 3, first_parts, s->stream);
            launch_rows_logistic(s->dm, s->ge, s->bf, s->obj.b, s->short_ok ? 1 : 0, s->stream);
            enqueue_redo_columns(s);
            launch_update_logistic(s->dm, s->op, s->ge, s->bf, first_parts, 0, s->stream);
        } else {
            // Short sequence: the pass itself sums the loss differences of the first trial step over each workgroup's
            // rows, and the update kernel takes the Armijo decision from those partials; the update of an accepted
            // first step also moves the margins.  The search kernels, the recomputation of the row weights and the
            // second transposed pass -- launches that almost never do work -- are left out; should the first step be
            // rejected, the solver parks itself and read_scal() supplies them.
            launch_update_logistic(s->dm, s->op, s->ge, s->bf, first_parts, 1, s->stream);
            s->short_steps_unseen++;
        }
    } else {
        a.mode = kRowLogiDir;
        { TimedSlot ts(s); launch_gemv(s->dm, s->ge, s->bf, a, s->stream, ts.e0, ts.e1); }
        launch_ls_logistic(s->dm, s->op, s->ge, s->bf, s->obj.b, 0, 3, 0, s->stream);
        launch_rows_logistic(s->dm, s->ge, s->bf, s->obj.b, 0, s->stream);
        { TimedSlot ts(s); launch_gemvt_from(s->dm, s->ge, s->bf, s->obj.A, s->bf.psi, 1, s->stream, ts.e0, ts.e1); }
        launch_update_logistic(s->dm, s->op, s->ge, s->bf, 0, 0, s->stream);
    }
    s->steps_since_refresh++;
}

void fresh_scal(lbfgsb_solver* s) {
    std::memset(s->h_scal, 0, sizeof(Scal));
    s->h_scal->status = LBFGSB_RUNNING;
    s->h_scal->alpha_ub = 1.0;
    s->h_scal->hist = s->bf.hist;
}

// The first bound that is no good, for the message (the device has found that there is one).
int report_bounds(lbfgsb_solver* s, const double* l, const double* u) {
    const int64_t n = s->dm.n;
    std::vector<double> hl((size_t)n), hu((size_t)n);
    HIP_TRY(hipMemcpyAsync(hl.data(), l, (size_t)n * 8, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipMemcpyAsync(hu.data(), u, (size_t)n * 8, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    for (int64_t i = 0; i < n; ++i)
        if (!(hl[(size_t)i] <= hu[(size_t)i]))
            return fail(LBFGSB_E_BOUNDS, "bounds cross or are NaN at index %lld (l = %g, u = %g)", (long long)i, hl[(size_t)i],
                        hu[(size_t)i]);
    for (int64_t i = 0; i < n; ++i)
        if (!(hl[(size_t)i] > 0.0))
            return fail(LBFGSB_E_BOUNDS, "the entropy regulariser needs l > 0 (l[%lld] = %g)", (long long)i, hl[(size_t)i]);
    return fail(LBFGSB_E_BOUNDS, "a bound was no good when it was checked");
}

// The first x0_i outside its bounds, for the message (the device has found that there is one).
int report_infeasible(lbfgsb_solver* s, const double* x0) {
    const int64_t n = s->dm.n;
    std::vector<double> hx((size_t)n), hl((size_t)n), hu((size_t)n);
    HIP_TRY(hipMemcpyAsync(hx.data(), x0, (size_t)n * 8, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipMemcpyAsync(hl.data(), s->bf.l, (size_t)n * 8, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipMemcpyAsync(hu.data(), s->bf.u, (size_t)n * 8, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    for (int64_t i = 0; i < n; ++i) {
        const double v = hx[(size_t)i];
        if (!(v >= hl[(size_t)i]) || !(v <= hu[(size_t)i]))
            return fail(LBFGSB_E_INFEASIBLE_X0, "x0[%lld] = %g is outside [%g, %g]", (long long)i, v, hl[(size_t)i],
                        hu[(size_t)i]);
    }
    return fail(LBFGSB_E_INFEASIBLE_X0, "x0 was outside its bounds when it was checked");
}

// trusted: x0 is the solver's own iterate, or has been checked by the caller: only f is checked for finiteness
int set_x_impl(lbfgsb_solver* s, const double* x0, bool trusted) {
    volatile int* flag = s->h_flag;
    if (s->timed > 0) s->steps_only = false;
    const bool one = !trusted && s->owns_h_scal && s->dm.n <= kStartOneMax && !s->timing;
    if (!trusted) {
        // nothing of the solver's state changes before this has been found to be all right
        flag[0] = flag[1] = 0;
        if (one) {
            launch_check_start(s->dm, s->op, s->bf, x0, s->h_flag, s->stream);
        } else {
            launch_check_box(s->dm, s->op, s->bf, x0, s->h_flag, s->stream);
            HIP_TRY(hipStreamSynchronize(s->stream));
            HIP_TRY(hipGetLastError());
            if (flag[0]) return report_infeasible(s, x0);
        }
    }
    if (!one) launch_start(s->dm, s->bf, x0, s->stream);
    const bool gram_ready = s->gram_ready, commit_needed = s->commit_needed;
    const int short_steps_unseen = s->short_steps_unseen;
    enqueue_eval(s, one ? 1 : 0, true, false, trusted ? nullptr : s->h_flag);
    s->short_steps_unseen = 0;
    HIP_TRY(read_scal(s));
    HIP_TRY(hipGetLastError());
    if (one && flag[0]) {
        s->gram_ready = gram_ready;
        s->commit_needed = commit_needed;
        s->short_steps_unseen = short_steps_unseen;
        launch_admit(s->bf, s->stream);
        return report_infeasible(s, x0);
    }
    s->steps_since_refresh = 0;
    s->steps_since_set_x = 0;
    s->logi_full_left = 0;
    if (!std::isfinite(s->h_scal->f) || (!trusted && flag[1])) {
        s->x_set = false;
        return fail(LBFGSB_E_NONFINITE, "f or grad f is not finite at x0");
    }
    s->x_set = true;
    return LBFGSB_OK;
}


// Argument checks shared by the entry points that set a solver up; *o receives the options (defaults when opt is NULL).
int check_create_args(int64_t n, int m, const double* l, const double* u, const lbfgsb_objective* obj,
                      const lbfgsb_options* opt, const void* workspace, lbfgsb_options* o) {
    int rc = check_objective(n, m, obj);
    if (rc) return rc;
    const bool ot = is_transport(obj->kind);
    if (!l || !u || !obj->A || !workspace) return fail(LBFGSB_E_INVALID_ARG, "NULL device pointer");
    if (ot ? (obj->row_weight && !obj->b) : !obj->b) return fail(LBFGSB_E_INVALID_ARG, "NULL device pointer (b)");
    if (obj->n_extra > 0 && (!obj->extra_rows || !obj->extra_target))
        return fail(LBFGSB_E_INVALID_ARG, "NULL extra_rows / extra_target");
    if (opt) *o = *opt; else lbfgsb_default_options(o);
    rc = check_options(o);
    if (rc) return rc;
    if ((uintptr_t)workspace % 256) return fail(LBFGSB_E_INVALID_ARG, "workspace must be 256-byte aligned");
    const int esz = obj->dtype == LBFGSB_F32 ? 4 : 8;
    if ((uintptr_t)obj->A % esz || (uintptr_t)obj->b % 8 || (uintptr_t)obj->row_weight % 8 || (uintptr_t)l % 8 ||
        (uintptr_t)u % 8)
        return fail(LBFGSB_E_INVALID_ARG, "misaligned device pointer");
    return LBFGSB_OK;
}

// Fills the host object for a checked problem: launch geometry, kernel preparation, and the device arrays carved
// out of `workspace`.  Allocates nothing and touches no device memory; *total receives the bytes of workspace in use.
int setup_solver(lbfgsb_solver* s, int64_t n, int m, const lbfgsb_objective* obj, const lbfgsb_options& o,
                 void* workspace, size_t workspace_bytes, hipStream_t stream, size_t* total, SingleRead reads = kReadAny) {
    s->dm = make_dims(n, m, obj);
    s->options = o;
    s->op = Opts{o.eps, o.armijo_c1, o.backtrack, o.tol, o.max_backtracks, o.tol_relative, o.max_iter, 0, 0.0, 0.0, nullptr, 0u, 0};
    s->obj = *obj;
    s->ge = make_geometry(s->dm, obj->A, reads);
    s->stream = stream;
    s->h_scal = nullptr;
    s->owns_h_scal = false;
    s->h_flag = nullptr;
    s->h_progress = nullptr;
    s->steps_since_refresh = 0;
    s->steps_since_set_x = 0;
    s->logi_full_left = 0;
    s->short_steps_unseen = 0;
    s->commit_needed = true;
    s->x_set = s->gram_ready = false;
    s->timing = false;
    s->timed = 0;
    s->steps_only = true;
    const Layout L = make_layout(s->dm, s->ge);
    *total = L.total;
    if (workspace_bytes < L.total)
        return fail(LBFGSB_E_INVALID_ARG, "workspace too small: %zu < %zu bytes", workspace_bytes, L.total);
    // (asked for by name the fused pass takes rows on 16-byte boundaries only, as documented; AUTO uses it for any)
    if (o.a_pass == LBFGSB_APASS_FUSED && (!s->ge.fused_ok || s->ge.vec == 1))
        return fail(LBFGSB_E_UNSUPPORTED, "the fused A pass does not support this shape");
    {
        const hipError_t ge_ = gram_prepare(s->dm, 0);
        if (ge_ != hipSuccess) return fail(LBFGSB_E_HIP, "preparing the Gram kernel: %s", hipGetErrorString(ge_));
    }
    const bool resident_ok = resident_shape_ok(s->dm, obj->row_weight != nullptr);
    if (o.a_pass == LBFGSB_APASS_RESIDENT && !resident_ok)
        return fail(LBFGSB_E_UNSUPPORTED, "the resident solver does not take this problem (kind, shape or size)");
    s->use_resident = resident_ok && (o.a_pass == LBFGSB_APASS_AUTO || o.a_pass == LBFGSB_APASS_RESIDENT);
    if (s->use_resident) {
        const hipError_t re = resident_prepare(s->dm);
        if (re != hipSuccess) return fail(LBFGSB_E_HIP, "preparing the resident solver: %s", hipGetErrorString(re));
    }
    if (small_step_ok(s->dm)) {
        const hipError_t se = small_step_prepare(s->dm);
        if (se != hipSuccess) return fail(LBFGSB_E_HIP, "preparing the short-vector kernel: %s", hipGetErrorString(se));
    }
    s->use_fused = s->ge.fused_ok && o.a_pass != LBFGSB_APASS_TWO_PASS;
    if (!s->use_fused) s->ge.sym_strips = 0;
    if (s->use_fused) {
        const hipError_t fe = fused_prepare(s->dm, s->ge);
        if (fe != hipSuccess) return fail(LBFGSB_E_HIP, "preparing the fused A pass: %s", hipGetErrorString(fe));
    }
    s->short_ok = s->use_fused && s->dm.kind == LBFGSB_OBJ_LOGISTIC_L2 && fused_ls_first_ok(s->dm, s->ge);
    s->ge.w_parts = s->use_fused ? s->ge.fused_blocks : s->ge.gemvt_row_blocks;
    s->ge.redo_parts = s->use_fused && s->ge.narrow_variant >= 0 ? s->ge.fused_blocks : s->ge.gemvt_row_blocks;
    s->ge.loss_parts = s->ge.sym_strips > 0 ? sym_loss_parts(s->dm) : (s->use_fused ? s->ge.fused_blocks : s->ge.gemv_blocks);

    char* w = (char*)workspace;
    Buffers& b = s->bf;
    b.scal = (Scal*)(w + L.scal);
    b.scal_next = (Scal*)(w + L.scal_next);
    b.x = (double*)(w + L.x); b.g = (double*)(w + L.g); b.l = (double*)(w + L.l); b.u = (double*)(w + L.u);
    b.d = (double*)(w + L.d); b.p1 = (double*)(w + L.p1); b.p2 = (double*)(w + L.p2);
    b.mask = (uint8_t*)(w + L.mask);
    b.S = (double*)(w + L.S); b.Y = (double*)(w + L.Y);
    b.row = (double*)(w + L.row); b.t = (double*)(w + L.t); b.psi = (double*)(w + L.psi);
    b.wpart = (double*)(w + L.wpart); b.losspart = (double*)(w + L.losspart);
    b.grampart = (double*)(w + L.grampart); b.redpart = (double*)(w + L.redpart); b.lspart = (double*)(w + L.lspart);
    b.wextra = (double*)(w + L.wextra); b.xres = (double*)(w + L.xres);
    b.hist = (lbfgsb_iter_record*)(w + L.hist);
    return LBFGSB_OK;
}

// The workspace starts from all-zero memory (fill kernel: no memset node ever enters a captured graph); the bounds
// are copied in.  Waits for both.
int init_workspace(lbfgsb_solver* s, const double* l, const double* u, void* workspace, size_t total) {
    launch_fill_zero(workspace, total, s->stream);
    hipError_t e = hipMemcpyAsync(s->bf.l, l, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(s->bf.u, u, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return fail(LBFGSB_E_HIP, "initialising the workspace: %s", hipGetErrorString(e));
    return LBFGSB_OK;
}

// Free set and stopping test at x, whose gradient has just been evaluated from scratch.
void enqueue_retest(lbfgsb_solver* s) {
    Opts quiet = s->op;                // (not one of the steps the host is following)
    quiet.progress = nullptr;
    launch_gram(s->dm, quiet, s->ge, s->bf, 0, 1, s->stream);
}

// The stopping quantity was computed from a gradient carried by recurrence: residual and gradient are recomputed from x
// and the test is made again before convergence is declared (the status is then in the host copy).
bool one_workgroup_retests(const lbfgsb_solver* s) { return s->dm.n <= kRetestMax && !is_transport(s->dm.kind); }
hipError_t confirm_convergence(lbfgsb_solver* s) {
    if (one_workgroup_retests(s)) {
        enqueue_eval(s, 0, true, true);
        s->steps_since_refresh = 0;
        launch_retest(s->dm, s->op, s->bf, s->stream, s->owns_h_scal ? s->h_scal : nullptr);
        return s->owns_h_scal ? hipStreamSynchronize(s->stream) : read_scal(s);
    }
    launch_reopen(s->dm, s->bf, s->stream);
    enqueue_eval(s, 0, true);          // (nothing is pending)
    s->steps_since_refresh = 0;
    enqueue_retest(s);
    return read_scal(s);
}

constexpr int kPollMax = 64;   // steps between two looks at the device status, at most

// Where the host copy is pinned, the kernel that takes an iteration's stopping decision reports it there, and the
// host follows without stopping the device: when the outcome of a reporting step is known -- before that step's pass
// over A has begun -- it enqueues the steps up to the next one that reports and none behind it: what is left of the reporting
// step keeps the device busy meanwhile.  The first eight steps report, then every fourth, in long runs every eighth (a report
// costs 2 us; a run that ends reports at once).  A run that is over in k steps has enqueued none (k <= 8) to 7 in vain, at 4.2 us a
// launch, 13-18 us a step (none when the iteration limit ends it: no step is enqueued behind the first that can find the limit
// reached before that one has reported).  Whole calls, us, first four reporting and one or two steps ahead / this: NNLS 3001 x 301
// 358 / 341, 9000 x 900 589 / 557, 20000 x 5000 2806 / 2786, over a simplex 8000 x 2000 6964 / 6660, 4000 x 1000 4615 / 4070; two
// steps ahead behind the eighth: as before; 16 or 32 steps that report: no better.  Waiting for the
// device every eight steps instead left it idle for ~25 us each time, and 0 to 7 steps in vain.
struct Follower {
    lbfgsb_solver* s;
    unsigned origin = 0;       // steps enqueued when the run began: the reporting ones are counted from there
    unsigned known = 0;        // reports of steps up to this one are not this run's, or have been acted upon
    unsigned reporting = 1;    // the step whose outcome is waited for next
    unsigned limit = 1;        // steps after which the iteration limit can have been reached
    long long steps = 0, cap;
    explicit Follower(lbfgsb_solver* solver) : s(solver), cap(2ll * solver->options.max_iter + 64) {   // (accepted iterations + memory-reset retries)
        *(volatile unsigned long long*)s->h_progress = 0;
        s->steps_enqueued = 0;
        s->op.progress = s->h_progress;
    }
    ~Follower() { s->op.progress = nullptr; s->note_at = 0; }

    // a run begins: iters iterations of max_iter are behind
    void begin(long long iters) {
        const long long left = s->options.max_iter - iters + 1;
        limit = left < 1 ? 1u : (left > 0x7fffffff ? 0x7fffffffu : (unsigned)left);
        origin = s->steps_enqueued;
        steps = 0;
        resume();
    }
    // on with it from here
    void resume() {
        known = s->steps_enqueued;
        s->note_at = reporting = known + 1;
    }
    unsigned next_report(unsigned step) const {
        const unsigned k = step - origin, n = k + (k < 8 ? 1 : (k < 32 ? 4 : 8));
        return origin + (k < limit && n > limit ? limit : n);
    }
    // Enqueues steps until a report says that the run is over: *st is the status then, RUNNING when `cap` steps have not
    // sufficed, -1 when the stream has run dry or failed (the scalar block says what there is to know).
    int until_over(int* st) {
        volatile unsigned long long* seen = s->h_progress;
        for (;;) {
            while (s->steps_enqueued - origin < reporting - origin && steps < cap) {
                enqueue_step(s);
                ++steps;
                if (s->steps_enqueued == s->note_at) s->note_at = next_report(s->note_at);
            }
            HIP_TRY(hipGetLastError());
            for (unsigned spins = 1;; ++spins) {
                const unsigned long long p = *seen;
                const unsigned step = (unsigned)(p >> 32);
                *st = (int)(unsigned)p;
                if (step > known && (step >= reporting || *st != LBFGSB_RUNNING)) break;
                // (now and then: has the stream run dry, or failed?)
                __builtin_ia32_pause();
                if (spins % 64 == 0) sched_yield();   // (to other threads that want this core)
                if (spins % 1024 == 0) {
                    if (hipStreamQuery(s->stream) != hipErrorNotReady) { *st = -1; return LBFGSB_OK; }
                    (void)hipGetLastError();   // (a stream that is busy is no error)
                }
            }
            if (*st != LBFGSB_RUNNING || steps >= cap) return LBFGSB_OK;
            reporting = next_report(reporting);
        }
    }
};

// The stopping logic of lbfgsb_solve, for a solver whose arguments have been checked.
int solve_impl(lbfgsb_solver* s, lbfgsb_info* info) {
    s->steps_only = false;
    const bool quad = is_quadratic(s->dm.kind);
    const long long cap = 2ll * s->options.max_iter + 64;   // accepted iterations + memory-reset retries
    if (s->use_resident) {
        // one launch runs until the device-side status changes (it re-evaluates the gradient from x before it
        // reports convergence) or the cap is reached
        const int steps_cap = (int)(cap > 0x3fffffff ? 0x3fffffff : cap);
        if (s->owns_h_scal) {
            // (pinned host copy: the kernel writes the scalar block there itself, with every pending update applied)
            launch_resident(s->dm, s->op, s->bf, s->obj.A, s->obj.b, steps_cap, s->options.refresh_every, s->stream, s->h_scal);
            s->commit_needed = false;
            HIP_TRY(hipStreamSynchronize(s->stream));
        } else {
            launch_resident(s->dm, s->op, s->bf, s->obj.A, s->obj.b, steps_cap, s->options.refresh_every, s->stream);
            HIP_TRY(read_scal(s));
        }
        HIP_TRY(hipGetLastError());
        if (info) fill_info(*s->h_scal, info);
        return LBFGSB_OK;
    }
    if (s->h_progress) {
        Follower run(s);
        run.begin(s->h_scal->iters);   // (from what the host has last seen)
        for (;;) {
            int st = LBFGSB_RUNNING;
            const int rc = run.until_over(&st);
            if (rc) return rc;
            // (The first step is known to have gone on, so at least one iteration is behind: see the condition below.  The
            // number in the report does not say so: a step behind the one that ended the run reports the end as well, and
            // which of the two is seen depends on the host's pace.)
            if (st == LBFGSB_CONVERGED && quad && s->steps_since_refresh > 0 && run.reporting - run.origin >= 2) {
                HIP_TRY(confirm_convergence(s));
                st = s->h_scal->status;
            } else {
                HIP_TRY(read_scal(s));
                st = s->h_scal->status;
                if (st == LBFGSB_CONVERGED && quad && s->steps_since_refresh > 0 && s->h_scal->iters > 0) {
                    HIP_TRY(confirm_convergence(s));
                    st = s->h_scal->status;
                }
            }
            if (st != LBFGSB_RUNNING || run.steps >= run.cap) break;
            run.resume();   // (a parked step has been finished, or convergence was not confirmed: the device is idle)
        }
        HIP_TRY(hipGetLastError());
        if (info) fill_info(*s->h_scal, info);
        return LBFGSB_OK;
    }
    long long steps = 0;
    // A poll leaves the device idle for about 30 us (commit, copy of the scalar block, the host's wake-up and the next
    // launches), a step enqueued after the solver has stopped costs about 6.  Long runs are therefore polled less
    // often: the interval doubles whenever eight intervals' worth of steps have gone by, up to 64.
    int batch = s->options.poll_every;
    for (;;) {
        for (int k = 0; k < batch; ++k) enqueue_step(s);
        steps += batch;
        if (batch < kPollMax && steps >= 8ll * batch) batch = 2 * batch > kPollMax ? kPollMax : 2 * batch;
        HIP_TRY(read_scal(s));
        int st = s->h_scal->status;
        if (st == LBFGSB_CONVERGED && quad && s->steps_since_refresh > 0 && s->h_scal->iters > 0) {
            HIP_TRY(confirm_convergence(s));
            st = s->h_scal->status;
        }
        if (st != LBFGSB_RUNNING) break;
        if (steps >= cap) break;
    }
    HIP_TRY(hipGetLastError());
    if (info) fill_info(*s->h_scal, info);
    return LBFGSB_OK;
}


// ---- lbfgsb_solve_static: per-device state, nothing of it allocated at run time ----------------------------

constexpr int kMaxDevices = 64;
constexpr int kHostChunk = 2048;   // doubles per host-side validation chunk (stack arrays)

struct StaticSlot {
    void* ptr = nullptr;       // device address of this device's copy of `scratch`
    lbfgsb_solver solver;      // host object, reused by every call on the device
    Scal h_scal;               // host copy of the scalar block (pageable: allocating pinned memory is an allocation)
};
StaticSlot g_static[kMaxDevices];

// The calling thread's current device's slot, with the address of that device's scratch array resolved.
int static_slot(StaticSlot** out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(LBFGSB_E_INVALID_ARG, "device index %d is not supported", dev);
    StaticSlot* sl = &g_static[dev];
    if (!sl->ptr) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (uintptr_t)p % 256) return fail(LBFGSB_E_HIP, "the scratch array has no usable device address");
        sl->ptr = p;
    }
    *out = sl;
    return LBFGSB_OK;
}

// Bounds and start point checked on the host in chunks that live on the stack: l <= u, l <= x0 <= u, no NaN,
// l > 0 for the entropy kind; also finds out whether all variables share one pair of bounds.
int check_box_chunked(lbfgsb_solver* s, const double* l, const double* u, const double* x0) {
    double hl[kHostChunk], hu[kHostChunk], hx[kHostChunk];
    const int64_t n = s->dm.n;
    bool same = true;
    double lo0 = 0.0, hi0 = 0.0;
    for (int64_t i0 = 0; i0 < n; i0 += kHostChunk) {
        const int64_t cnt = n - i0 < kHostChunk ? n - i0 : kHostChunk;
        HIP_TRY(hipMemcpyAsync(hl, l + i0, (size_t)cnt * 8, hipMemcpyDeviceToHost, s->stream));
        HIP_TRY(hipMemcpyAsync(hu, u + i0, (size_t)cnt * 8, hipMemcpyDeviceToHost, s->stream));
        HIP_TRY(hipMemcpyAsync(hx, x0 + i0, (size_t)cnt * 8, hipMemcpyDeviceToHost, s->stream));
        HIP_TRY(hipStreamSynchronize(s->stream));
        if (i0 == 0) { lo0 = hl[0]; hi0 = hu[0]; }
        for (int64_t k = 0; k < cnt; ++k) {
            if (!(hl[k] <= hu[k]))
                return fail(LBFGSB_E_BOUNDS, "bounds cross or are NaN at index %lld (l = %g, u = %g)", (long long)(i0 + k),
                            hl[k], hu[k]);
            if (s->dm.kind == LBFGSB_OBJ_OT_ENTROPY && !(hl[k] > 0.0))
                return fail(LBFGSB_E_BOUNDS, "the entropy regulariser needs l > 0 (l[%lld] = %g)", (long long)(i0 + k), hl[k]);
            if (!(hx[k] >= hl[k]) || !(hx[k] <= hu[k]))
                return fail(LBFGSB_E_INFEASIBLE_X0, "x0[%lld] = %g is outside [%g, %g]", (long long)(i0 + k), hx[k], hl[k],
                            hu[k]);
            same = same && hl[k] == lo0 && hu[k] == hi0;
        }
    }
    s->op.uniform_bounds = same ? 1 : 0;
    s->op.lo = lo0;
    s->op.hi = hi0;
    return LBFGSB_OK;
}

int check_finite_chunked(lbfgsb_solver* s, const double* v) {
    double hv[kHostChunk];
    for (int64_t i0 = 0; i0 < s->dm.n; i0 += kHostChunk) {
        const int64_t cnt = s->dm.n - i0 < kHostChunk ? s->dm.n - i0 : kHostChunk;
        HIP_TRY(hipMemcpyAsync(hv, v + i0, (size_t)cnt * 8, hipMemcpyDeviceToHost, s->stream));
        HIP_TRY(hipStreamSynchronize(s->stream));
        for (int64_t k = 0; k < cnt; ++k)
            if (!std::isfinite(hv[k])) return fail(LBFGSB_E_NONFINITE, "f or grad f is not finite at x0");
    }
    return LBFGSB_OK;
}

}  // namespace

extern "C" {

const char* lbfgsb_last_error(void) { return g_err.c_str(); }

void lbfgsb_default_options(lbfgsb_options* o) {
    if (!o) return;
    o->eps = 1e-10; o->armijo_c1 = 1e-4; o->backtrack = 0.5; o->max_backtracks = 60; o->tol = 1e-8;
    o->tol_relative = 0; o->max_iter = 1000; o->refresh_every = 32; o->poll_every = 8; o->a_pass = LBFGSB_APASS_AUTO;
}

size_t lbfgsb_workspace_bytes(int64_t n, int m, const lbfgsb_objective* obj, const lbfgsb_options* opt) {
    (void)opt;
    if (check_objective(n, m, obj) != LBFGSB_OK) return 0;
    const Dims dm = make_dims(n, m, obj);
    const Geometry ge = make_geometry(dm, obj->A);
    return make_layout(dm, ge).total;
}

int lbfgsb_create(lbfgsb_solver** out, int64_t n, int m, const double* l, const double* u, const lbfgsb_objective* obj,
                  const lbfgsb_options* opt, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!out) return fail(LBFGSB_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    lbfgsb_options o;
    int rc = check_create_args(n, m, l, u, obj, opt, workspace, &o);
    if (rc) return rc;
    lbfgsb_solver* s = new (std::nothrow) lbfgsb_solver();
    if (!s) return fail(LBFGSB_E_INVALID_ARG, "out of host memory");
    size_t total = 0;
    rc = setup_solver(s, n, m, obj, o, workspace, workspace_bytes, (hipStream_t)hip_stream, &total);
    if (rc) { delete s; return rc; }

    auto bail = [&](int code) { lbfgsb_destroy(s); return code; };
    {
        const size_t flag_at = (sizeof(Scal) + 63) / 64 * 64;
        hipError_t e = hipHostMalloc((void**)&s->h_scal, flag_at + 64, kPinned);
        if (e != hipSuccess) { s->h_scal = nullptr; return bail(fail(LBFGSB_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e))); }
        s->owns_h_scal = true;
        s->h_flag = (int*)((char*)s->h_scal + flag_at);
        s->h_progress = (unsigned long long*)((char*)s->h_scal + flag_at + 32);
    }
    {
        // the device looks at the bounds; only to name an offending one does the host fetch them
        static_assert(sizeof(BoundsReport) <= sizeof(Scal), "reported where the scalar block's copy will be");
        BoundsReport* br = (BoundsReport*)s->h_scal;
        std::memset(br, 0, sizeof *br);
        launch_check_bounds(s->dm, l, u, br, s->stream);
        hipError_t e = hipStreamSynchronize(s->stream);
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) return bail(fail(LBFGSB_E_HIP, "reading the bounds: %s", hipGetErrorString(e)));
        if (br->flag[0] || (obj->kind == LBFGSB_OBJ_OT_ENTROPY && br->flag[2])) return bail(report_bounds(s, l, u));
        s->op.uniform_bounds = br->flag[1] ? 0 : 1;
        s->op.lo = br->lo;
        s->op.hi = br->hi;
    }
    rc = init_workspace(s, l, u, workspace, total);
    if (rc) return bail(rc);
    *out = s;
    return LBFGSB_OK;
}

void lbfgsb_destroy(lbfgsb_solver* s) {
    if (!s) return;
    for (hipEvent_t ev : s->ev0) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : s->ev1) (void)hipEventDestroy(ev);
    if (s->h_scal && s->owns_h_scal) (void)hipHostFree(s->h_scal);
    delete s;
}

int lbfgsb_set_x(lbfgsb_solver* s, const double* x0) {
    if (!s || !x0) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    return set_x_impl(s, x0, false);
}

int lbfgsb_step(lbfgsb_solver* s, lbfgsb_info* info) {
    if (!s) return fail(LBFGSB_E_INVALID_ARG, "solver is NULL");
    if (!s->x_set) return fail(LBFGSB_E_INVALID_ARG, "lbfgsb_set_x has not been called");
    enqueue_step(s);
    if (info) {
        HIP_TRY(read_scal(s));
        HIP_TRY(hipGetLastError());
        fill_info(*s->h_scal, info);
    }
    return LBFGSB_OK;
}

int lbfgsb_solve(lbfgsb_solver* s, lbfgsb_info* info) {
    if (!s) return fail(LBFGSB_E_INVALID_ARG, "solver is NULL");
    if (!s->x_set) return fail(LBFGSB_E_INVALID_ARG, "lbfgsb_set_x has not been called");
    return solve_impl(s, info);
}

int lbfgsb_solve_static(int64_t n, int m, const double* l, const double* u, const lbfgsb_objective* obj,
                        const lbfgsb_options* opt, double* x, lbfgsb_info* info, void* hip_stream) {
    if (!x) return fail(LBFGSB_E_INVALID_ARG, "x is NULL");
    if ((uintptr_t)x % 8) return fail(LBFGSB_E_INVALID_ARG, "misaligned device pointer");
    StaticSlot* sl = nullptr;
    int rc = static_slot(&sl);
    if (rc) return rc;
    lbfgsb_options o;
    rc = check_create_args(n, m, l, u, obj, opt, sl->ptr, &o);
    if (rc) return rc;
    size_t need = lbfgsb_workspace_bytes(n, m, obj, &o);
    SingleRead reads = kReadAny;
    if (need > (size_t)LBFGSB_STATIC_SCRATCH_BYTES) {
        const Dims dm = make_dims(n, m, obj);
        const size_t without = make_layout(dm, make_geometry(dm, obj->A, kReadAligned)).total;
        if (without < need) { need = without; reads = kReadAligned; }
    }
    if (need == 0 || need > (size_t)LBFGSB_STATIC_SCRATCH_BYTES)
        return fail(LBFGSB_E_INVALID_ARG,
                    "this problem needs %zu bytes of workspace, lbfgsb_solve_static holds %zu: use lbfgsb_create with a "
                    "workspace of your own", need, (size_t)LBFGSB_STATIC_SCRATCH_BYTES);
    lbfgsb_solver* s = &sl->solver;
    if (s->timing || !s->ev0.empty()) return fail(LBFGSB_E_INVALID_ARG, "the static solver object is in an unexpected state");
    size_t total = 0;
    rc = setup_solver(s, n, m, obj, o, sl->ptr, (size_t)LBFGSB_STATIC_SCRATCH_BYTES, (hipStream_t)hip_stream, &total, reads);
    if (rc) return rc;
    s->h_scal = &sl->h_scal;
    rc = check_box_chunked(s, l, u, x);
    if (rc) return rc;
    // the array keeps the previous call's contents: everything this problem uses starts from zero again
    rc = init_workspace(s, l, u, sl->ptr, total);
    if (rc) return rc;
    rc = set_x_impl(s, x, true);
    if (rc) return rc;
    rc = check_finite_chunked(s, s->bf.g);
    if (rc) { s->x_set = false; return rc; }
    rc = solve_impl(s, info);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(x, s->bf.x, (size_t)n * 8, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    s->x_set = false;
    return LBFGSB_OK;
}

int lbfgsb_get_history(lbfgsb_solver* s, lbfgsb_iter_record* records, int capacity, int* count) {
    if (!s || !records || !count || capacity < 0) return fail(LBFGSB_E_INVALID_ARG, "NULL argument or negative capacity");
    *count = 0;
    HIP_TRY(read_scal(s));
    const long long written = s->h_scal->hist_count;
    long long have = written < LBFGSB_HISTORY_CAPACITY ? written : LBFGSB_HISTORY_CAPACITY;
    if (have > capacity) have = capacity;
    // the `have` most recent records, oldest first: ring positions (written - have) .. (written - 1)
    for (long long k = 0; k < have; ++k) {
        const long long pos = (written - have + k) % LBFGSB_HISTORY_CAPACITY;
        HIP_TRY(hipMemcpyAsync(records + k, s->bf.hist + pos, sizeof(lbfgsb_iter_record), hipMemcpyDeviceToHost, s->stream));
    }
    HIP_TRY(hipStreamSynchronize(s->stream));
    *count = (int)have;
    return LBFGSB_OK;
}

int lbfgsb_get_info(lbfgsb_solver* s, lbfgsb_info* info) {
    if (!s || !info) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    HIP_TRY(read_scal(s));
    fill_info(*s->h_scal, info);
    return LBFGSB_OK;
}

int lbfgsb_get_x(lbfgsb_solver* s, double* x_out) {
    if (!s || !x_out) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    if (s->short_steps_unseen > 0) HIP_TRY(read_scal(s));   // a parked solver is brought up to date first (this waits)
    HIP_TRY(hipMemcpyAsync(x_out, s->bf.x, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    return LBFGSB_OK;
}

int lbfgsb_get_g(lbfgsb_solver* s, double* g_out) {
    if (!s || !g_out) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    if (s->short_steps_unseen > 0) HIP_TRY(read_scal(s));
    HIP_TRY(hipMemcpyAsync(g_out, s->bf.g, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    return LBFGSB_OK;
}

int lbfgsb_enable_apass_timing(lbfgsb_solver* s, int enable) {
    if (!s) return fail(LBFGSB_E_INVALID_ARG, "solver is NULL");
    if (enable && s->ev0.empty()) {
        s->ev0.resize(kMaxTimed);
        s->ev1.resize(kMaxTimed);
        for (int i = 0; i < kMaxTimed; ++i) {
            HIP_TRY(hipEventCreate(&s->ev0[i]));
            HIP_TRY(hipEventCreate(&s->ev1[i]));
        }
    }
    s->timing = enable != 0;
    if (enable == 2) { s->timed = 0; s->steps_only = true; }
    return LBFGSB_OK;
}

int lbfgsb_apass_timing(lbfgsb_solver* s, int64_t* count, double* total_ms, double* bytes_per_pass) {
    if (!s || !count || !total_ms || !bytes_per_pass) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    // launches enqueued after the solver had stopped return at once without touching A: they are recognised
    // by their duration (below half of a typical long launch: the 90th percentile, so that a single launch
    // stretched by a profiler or a clock ramp does not set the scale) and left out.  Two stretched launches of ten, or passes
    // of unlike length, can set it all the same, so a solver that is known to have had none (steps alone, and still running; the logistic
    // objective's parked steps are in vain as well) is not judged that way: 2000 x 500 by two passes lost some of its 20 in 4 runs of 10.
    int status = LBFGSB_MAX_ITER;
    if (s->steps_only && s->x_set && s->dm.kind != LBFGSB_OBJ_LOGISTIC_L2)
        HIP_TRY(hipMemcpyAsync(&status, &s->bf.scal->status, sizeof(int), hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    std::vector<float> dur((size_t)s->timed);
    for (int i = 0; i < s->timed; ++i) HIP_TRY(hipEventElapsedTime(&dur[(size_t)i], s->ev0[i], s->ev1[i]));
    float longest = 0.f;
    if (!dur.empty()) {
        std::vector<float> sorted(dur);
        std::sort(sorted.begin(), sorted.end());
        longest = status == LBFGSB_RUNNING ? 0.f : sorted[(size_t)((sorted.size() - 1) * 9 / 10)];
    }
    double tot = 0.0;
    int64_t n = 0;
    for (int i = 0; i < s->timed; ++i)
        if (dur[(size_t)i] >= 0.5f * longest) { tot += dur[(size_t)i]; ++n; }
    *count = n;
    *total_ms = tot;
    *bytes_per_pass = (double)s->dm.rows * (double)s->dm.cols * (s->dm.dtype == LBFGSB_F32 ? 4.0 : 8.0);
    if (s->ge.sym_strips > 0) {
        // the upper triangle in strips of columns, with the blocks on the diagonal whole
        *bytes_per_pass = 0.0;
        for (int J = 0; J < s->ge.sym_strips; ++J) {
            const double rows = std::min<double>((double)(J + 1) * kSymStrip, (double)s->dm.cols);
            *bytes_per_pass += rows * (rows - (double)J * kSymStrip) * (s->dm.dtype == LBFGSB_F32 ? 4.0 : 8.0);
        }
    }
    // transport kinds: the timed kernel is the Gram kernel, timed in iterations m, m+1, ... after lbfgsb_set_x, when
    // all m pairs are stored.  It reads x, g, the newest y (and l, u unless every variable has the same bounds) in
    // full and writes the one-byte free mask; the 2m pair vectors are read at the free variables only (count taken
    // from the last status the host has seen)
    if (is_transport(s->dm.kind)) {
        const double n_free = (double)(s->dm.n - s->h_scal->n_fixed);
        *bytes_per_pass = (double)s->dm.n * (s->op.uniform_bounds ? 25.0 : 41.0) + n_free * 2.0 * s->dm.m * 8.0;
    }
    return LBFGSB_OK;
}


const char* lbfgsb_apass_name(const lbfgsb_solver* s) {
    if (s && s->use_resident) return "resident";
    return s && s->use_fused ? "fused" : "two_pass";
}

// ---- primitive-level hooks ------------------------------------------------------------------------------

int lbfgsb_dbg_fg(lbfgsb_solver* s, const double* x, double* f_host, double* g, double* rowvec) {
    if (!s || !x || !f_host || !g) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    s->x_set = s->gram_ready = false;
    HIP_TRY(hipMemcpyAsync(s->bf.x, x, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    fresh_scal(s);
    HIP_TRY(write_scal(s));
    enqueue_eval(s, 0);
    HIP_TRY(hipMemcpyAsync(g, s->bf.g, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    if (rowvec)
        HIP_TRY(hipMemcpyAsync(rowvec, s->bf.row, (size_t)row_entries(s->dm.kind, s->dm.rows, s->dm.cols) * 8,
                               hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(read_scal(s));
    HIP_TRY(hipGetLastError());
    *f_host = s->h_scal->f;
    return LBFGSB_OK;
}

int lbfgsb_dbg_free_mask(lbfgsb_solver* s, const double* x, const double* g, uint8_t* mask) {
    if (!s || !x || !g || !mask) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    s->x_set = s->gram_ready = false;
    HIP_TRY(hipMemcpyAsync(s->bf.x, x, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipMemcpyAsync(s->bf.g, g, (size_t)s->dm.n * 8, hipMemcpyDeviceToDevice, s->stream));
    fresh_scal(s);
    HIP_TRY(write_scal(s));
    launch_gram(s->dm, s->op, s->ge, s->bf, 0, 0, s->stream);
    HIP_TRY(hipMemcpyAsync(mask, s->bf.mask, (size_t)s->dm.n, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    HIP_TRY(hipGetLastError());
    return LBFGSB_OK;
}

int lbfgsb_dbg_two_loop(lbfgsb_solver* s, const double* S, const double* Y, const double* ynorm2, int npairs,
                        const double* g, const uint8_t* mask, double* d, int* pairs_used) {
    if (!s || !g || !mask || !d) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    if (npairs < 0 || npairs > s->dm.m) return fail(LBFGSB_E_INVALID_ARG, "npairs must be in 0..m");
    if (npairs > 0 && (!S || !Y || !ynorm2)) return fail(LBFGSB_E_INVALID_ARG, "NULL pair arrays");
    s->x_set = s->gram_ready = false;
    const size_t nb = (size_t)s->dm.n * 8;
    fresh_scal(s);
    if (npairs > 0) {
        HIP_TRY(hipMemcpyAsync(s->bf.S, S, nb * npairs, hipMemcpyDeviceToDevice, s->stream));
        HIP_TRY(hipMemcpyAsync(s->bf.Y, Y, nb * npairs, hipMemcpyDeviceToDevice, s->stream));
        HIP_TRY(hipMemcpyAsync(s->h_scal->ynorm2, ynorm2, (size_t)npairs * 8, hipMemcpyDeviceToHost, s->stream));
        HIP_TRY(hipStreamSynchronize(s->stream));
    }
    s->h_scal->count = npairs;
    s->h_scal->head = npairs % s->dm.m;
    HIP_TRY(write_scal(s));
    HIP_TRY(hipMemcpyAsync(s->bf.g, g, nb, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipMemcpyAsync(s->bf.mask, mask, (size_t)s->dm.n, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(gram_prepare(s->dm, 1));
    launch_gram(s->dm, s->op, s->ge, s->bf, 1, 0, s->stream);
    launch_dir(s->dm, s->op, s->ge, s->bf, 0, 1, s->stream);
    HIP_TRY(hipMemcpyAsync(d, s->bf.d, nb, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(read_scal(s));
    HIP_TRY(hipGetLastError());
    if (pairs_used) *pairs_used = s->h_scal->pairs_used;
    return LBFGSB_OK;
}

int lbfgsb_dbg_project_direction(lbfgsb_solver* s, const double* x, const double* g, const double* d, double* p,
                                 int* branch, double* alpha_ub) {
    if (!s || !x || !g || !d || !p) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    s->x_set = s->gram_ready = false;
    const size_t nb = (size_t)s->dm.n * 8;
    HIP_TRY(hipMemcpyAsync(s->bf.x, x, nb, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipMemcpyAsync(s->bf.g, g, nb, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipMemcpyAsync(s->bf.d, d, nb, hipMemcpyDeviceToDevice, s->stream));
    fresh_scal(s);
    HIP_TRY(write_scal(s));
    launch_dir(s->dm, s->op, s->ge, s->bf, 1, 1, s->stream);
    HIP_TRY(read_scal(s));
    HIP_TRY(hipGetLastError());
    const int br = s->h_scal->branch;
    HIP_TRY(hipMemcpyAsync(p, br == 1 ? s->bf.p1 : s->bf.p2, nb, hipMemcpyDeviceToDevice, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    if (branch) *branch = br;
    if (alpha_ub) *alpha_ub = s->h_scal->alpha_ub;
    return LBFGSB_OK;
}


// ---- augmented Lagrangian algorithm (Algorithm 4 of the appendix, Eq. (augLag)) ------------------------------
//
// Linear equality constraints h(x) = C x - d = 0 on the least-squares objective.  The rows of C are
// appended to A, and   rho/2 ||C x - d + lambda/rho||^2   is then a block of least-squares rows with weight
// rho and target d - lambda/rho: every outer iteration rewrites those targets and weights and runs the box
// solver on  L(., lambda, rho) = 0.5 sum_r w_r (a_r . x - beta_r)^2,  so the single-read pass, the closed-form
// line search and everything else of the path serve the constrained problem unchanged.

}  // extern "C"

// The algorithm's own state, on the device (a copy goes to the host when a run is over).
struct AlState {
    double rho, violation;     // violation: at the last outer iterate, to begin with at x0
    double L, f, pg2;
    long long inner_iters;
    int outer, status;
    int inner_status;          // how the inner solve that is being wound up ended
    int turned;                // the last k_al_turn has set up another inner solve
    int done, nonfinite;
};

struct lbfgsb_auglag {
    lbfgsb_solver* inner;
    lbfgsb_auglag_options ao;
    int64_t n_eq, n;
    // the constraint rows' targets d (caller's), and the targets / weights the algorithm rewrites (workspace):
    // entries of the stacked matrix's row vectors, or the inner objective's extra rows
    const double* d_c;
    double *beta_c, *omega_c;
    const double* res_c;     // where the inner solver leaves a_r . x - beta_r of the constraint rows after an evaluation
    double* lambda;          // multipliers
    AlState* state;
    AlState* h_state;        // pinned
    hipStream_t stream;
    enum { kStacked, kRows, kMarginals } variant;
    // the constraint rows (c_ld entries from one to the next, of type c_dtype; not the marginals, which have none), and n_eq
    // doubles of scratch (the change of weight * residual per constraint row)
    const void* c_rows = nullptr;
    int64_t c_ld = 0;
    int c_dtype = LBFGSB_F64;
    double* coef = nullptr;
};

namespace {

__global__ void k_al_init(int64_t rows, const double* __restrict__ bd, double* __restrict__ beta,
                          double* __restrict__ omega) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < rows; r += (int64_t)gridDim.x * blockDim.x) {
        beta[r] = bd[r];
        omega[r] = 1.0;
    }
}

// targets d - lambda/rho and weights rho of the constraint rows for the next inner solve
__global__ void k_al_prepare(int64_t n_eq, double rho, const double* __restrict__ d, const double* __restrict__ lambda,
                             double* __restrict__ beta, double* __restrict__ omega) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n_eq; r += (int64_t)gridDim.x * blockDim.x) {
        beta[r] = d[r] - lambda[r] / rho;
        omega[r] = rho;
    }
}

// ||h||_inf over a workgroup of NT threads, from each thread's share; every thread gets it.  lds: NT/64 doubles.
template <int NT>
__device__ __forceinline__ double block_max(double v, double* lds) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    v = lds[0];
    for (int w = 1; w < NT / 64; ++w) v = fmax(v, lds[w]);
    return v;
}

// Algorithm 4 begins: lambda^0 = 0, and residuals evaluated at x^0 with the targets d.
constexpr int kTurnThreads = 1024;
__global__ __launch_bounds__(kTurnThreads) void k_al_begin(int64_t n_eq, double rho0, const double* __restrict__ res, AlState* __restrict__ state) {
    __shared__ double lds[kTurnThreads / 64];
    double viol = 0.0;
    for (int64_t r = threadIdx.x; r < n_eq; r += kTurnThreads) viol = fmax(viol, fabs(res[r]));
    viol = block_max<kTurnThreads>(viol, lds);
    if (threadIdx.x == 0) {
        *state = AlState{};
        state->rho = rho0;
        state->violation = viol;
        state->status = LBFGSB_MAX_ITER;
    }
}

// An inner solve has ended: any pending update is applied, and the solver is open for an evaluation at its last iterate.
// (Once the run is over nothing changes any more, should the host have seen the last steps' report before it saw that.  Where the
// turn makes the test itself, k_eval_finish does this kernel's work and looks at `done` too.)
__global__ void k_al_reopen(Scal* scal, int m, AlState* state) {
    if (threadIdx.x != 0 || state->done) return;
    apply_pending(scal, m);
    state->inner_status = scal->status;
    scal->status = LBFGSB_RUNNING;
}

// Between two inner solves (one workgroup): multipliers, penalty parameter, the algorithm's own stopping test, and the next
// subproblem.  The host enqueues it behind the evaluation at the inner solve's last iterate and goes on with the next inner solve's
// steps without waiting for it: it used to fetch two scalars per outer iteration, ~60 us in which the device was idle.
//
// res: residuals a_r . x - beta_r of the constraint rows at x.  h_r = res_r - lambda_r/rho; lambda += rho h; rho doubles when
// ||h||_inf has not been halved; over when it is at most ctol and the inner solve has converged.
// Else only the targets beta and the weights omega change, so f and g at the unchanged x follow from the residuals without another
// evaluation: with c_r . x = res_r + beta_r,  res_r' = c_r . x - beta_r',  f' = f + 0.5 sum (omega' res'^2 - omega res^2),
// g' = g + C^T (omega' res' - omega res) -- the latter here where the rows are few and short (SHIFT; the sum constraint of a
// simplex is one), else by a kernel of its own from coef.  The scalar block starts afresh.
// retest: the inner solve's convergence has been tested anew on the evaluated gradient; it goes on if that was not confirmed.
struct AlTurn {
    int64_t n_eq, cols, ld;
    double ctol;
    int max_outer, retest, fevals;
    int refuse;                // a subproblem whose f is not finite ends the run with an error
    int own_test;              // retest by this workgroup, from here on (k_retest)
    int64_t n;
    Opts op;
    const double *x, *l, *u;
    const double* d;
    double *lambda, *beta, *omega, *res, *coef, *total;   // total (or null): where 0.5 sum omega res^2 is kept
    const void* Crows;
    double* g;
    Scal* scal;
    lbfgsb_iter_record* hist;
    AlState* state;
    AlState* host;
};
// Beyond 16 entries per thread one workgroup has too few loads in flight, beyond 64 rows the coefficients do not lie in LDS.
constexpr int kShiftRowsMax = 64;
constexpr int64_t kShiftMax = 16 * kTurnThreads;
template <typename T, bool SHIFT>
__global__ __launch_bounds__(kTurnThreads) void k_al_turn(AlTurn a) {
    __shared__ double lds[2 * kTurnThreads / 64];
    __shared__ double retest_s[3 * kTurnThreads / 64];
    __shared__ double coef_s[SHIFT ? kShiftRowsMax : 1];
    __shared__ double rho_s;
    __shared__ int go_s;
    const int tid = threadIdx.x;
    const double rho = a.state->rho, viol_prev = a.state->violation;
    if (a.state->done) return;
    const int status = a.own_test ? retest_point<kTurnThreads>(a.n, a.op, a.x, a.g, a.l, a.u, a.scal, retest_s)
                               : (a.retest ? a.scal->status : a.state->inner_status);
    if (a.retest && status == LBFGSB_RUNNING) {
        if (tid == 0) a.state->turned = 0;
        return;
    }
    double viol = 0.0, s[1] = {0.0};
    for (int64_t r = tid; r < a.n_eq; r += kTurnThreads) {
        const double v = a.res[r], lam = a.lambda[r], h = v - lam / rho;
        viol = fmax(viol, fabs(h));
        s[0] = fma(v, v, s[0]);
        a.lambda[r] = lam + rho * h;
    }
    viol = block_max<kTurnThreads>(viol, lds);
    block_sum<1, kTurnThreads / 64>(s, lds);
    if (tid == 0) {
        AlState st = *a.state;
        const double f = a.scal->f, rho_next = viol > 0.5 * viol_prev ? 2.0 * rho : rho;
        st.outer += 1;
        st.inner_iters += a.scal->iters;
        st.pg2 = a.scal->pg2;
        st.violation = viol;
        st.L = f;
        st.f = f - 0.5 * rho * s[0];
        const bool over = viol <= a.ctol && status == LBFGSB_CONVERGED;
        if (over) st.status = LBFGSB_CONVERGED;
        else st.rho = rho_next;
        st.done = over || st.outer >= a.max_outer;
        st.turned = !st.done;
        *a.state = st;
        if (st.done) {
            a.scal->status = status;
            *a.host = st;
        }
        rho_s = st.rho;
        go_s = !st.done;
    }
    __syncthreads();
    if (!go_s) return;
    const double rho_new = rho_s;
    double t[2] = {0.0, 0.0};
    for (int64_t r = tid; r < a.n_eq; r += kTurnThreads) {
        const double res_old = a.res[r], w_old = a.omega[r];
        const double cx = res_old + a.beta[r];
        const double b_new = a.d[r] - a.lambda[r] / rho_new;
        const double res_new = cx - b_new;
        const double c = rho_new * res_new - w_old * res_old;
        if (SHIFT) coef_s[r] = c;
        else a.coef[r] = c;
        t[0] += 0.5 * (rho_new * res_new * res_new - w_old * res_old * res_old);
        t[1] += 0.5 * rho_new * res_new * res_new;
        a.beta[r] = b_new;
        a.omega[r] = rho_new;
        a.res[r] = res_new;
    }
    block_sum<2, kTurnThreads / 64>(t, lds);
    const double f_new = a.scal->f + t[0];
    if (SHIFT) {
        for (int64_t j = tid; j < a.cols; j += kTurnThreads) {
            double acc = 0.0;
            for (int r = 0; r < (int)a.n_eq; ++r) acc = fma(coef_s[r], (double)((const T*)a.Crows)[r * a.ld + j], acc);
            a.g[j] += acc;
        }
    }
    __syncthreads();   // (every thread has read f)
    for (int k = tid; k < (int)(sizeof(Scal) / 4); k += kTurnThreads) reinterpret_cast<int*>(a.scal)[k] = 0;
    __syncthreads();
    if (tid == 0) {
        a.scal->status = LBFGSB_RUNNING;
        a.scal->alpha_ub = 1.0;
        a.scal->hist = a.hist;
        a.scal->f = f_new;
        a.scal->fevals = a.fevals;
        if (a.total) *a.total = t[1];
        if (a.refuse && !isfinite(f_new)) {
            // (refused, as a start point whose f is not finite is; stacked rows: left to the line search, which fails there)
            a.state->done = a.state->nonfinite = 1;
            a.state->turned = 0;
            a.scal->status = LBFGSB_LINESEARCH_FAILED;
            *a.host = *a.state;
        }
    }
}

// g += C^T coef behind a turn
template <typename T>
__global__ __launch_bounds__(kBlock) void k_al_shift_g(int64_t n_eq, int64_t cols, int64_t ld, const T* __restrict__ Crows,
                                                       const double* __restrict__ coef, double* __restrict__ g,
                                                       const AlState* __restrict__ state) {
    if (!state->turned) return;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < cols; j += (int64_t)gridDim.x * kBlock) {
        double acc = 0.0;
        for (int64_t r = 0; r < n_eq; ++r) acc = fma(coef[r], (double)Crows[r * ld + j], acc);
        g[j] += acc;
    }
}
// ... where the rows are the marginals of a rows x cols matrix: one row at a time, four columns' loads in flight
__global__ __launch_bounds__(kBlock) void k_al_shift_marginals(int64_t rows, int64_t cols, const double* __restrict__ coef,
                                                               double* __restrict__ g, const AlState* __restrict__ state) {
    if (!state->turned) return;
    const int64_t tiles = (cols + 4 * kBlock - 1) / (4 * kBlock);
    for (int64_t b = blockIdx.x; b < rows * tiles; b += gridDim.x) {
        const int64_t i = b / tiles, j0 = (b - i * tiles) * 4 * kBlock + threadIdx.x;
        const double ci = coef[i];
        double gv[4], cv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t j = j0 + k * kBlock < cols ? j0 + k * kBlock : cols - 1;
            gv[k] = g[i * cols + j];
            cv[k] = coef[rows + j];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j0 + k * kBlock < cols) g[i * cols + j0 + k * kBlock] = gv[k] + (ci + cv[k]);
    }
}
__global__ void k_al_report(const AlState* state, AlState* host) {
    if (threadIdx.x == 0) *host = *state;
}

size_t al_extra_bytes(int64_t rows, int64_t n_eq) {
    return align_up((size_t)rows * 8) * 2 + 2 * align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8) + align_up(sizeof(AlState));
}

int check_al(int64_t n, const lbfgsb_objective* o, int64_t n_eq) {
    if (!o) return fail(LBFGSB_E_INVALID_ARG, "objective is NULL");
    if (o->kind != LBFGSB_OBJ_LSQ) return fail(LBFGSB_E_INVALID_ARG, "lbfgsb_auglag_create takes the least-squares objective with the constraint rows stacked under A");
    if (n_eq < 0 || n_eq >= o->rows) return fail(LBFGSB_E_INVALID_ARG, "n_eq must be in 0..rows-1 (rows counts the constraint rows)");
    if (o->row_weight) return fail(LBFGSB_E_INVALID_ARG, "row_weight must be NULL: the weights are the algorithm's");
    if (o->n_extra) return fail(LBFGSB_E_INVALID_ARG, "n_extra must be 0");
    (void)n;
    return LBFGSB_OK;
}

int check_al_rows(const lbfgsb_objective* o, int64_t n_eq, const double* C, const double* d) {
    if (!o) return fail(LBFGSB_E_INVALID_ARG, "objective is NULL");
    if (o->kind == LBFGSB_OBJ_LOGISTIC_L2) return fail(LBFGSB_E_INVALID_ARG, "the augmented Lagrangian entry points take the quadratic objective kinds");
    if (n_eq < 0 || n_eq > kMaxExtra) return fail(LBFGSB_E_INVALID_ARG, "n_eq must be in 0..%d for constraint rows passed separately", kMaxExtra);
    if (o->n_extra) return fail(LBFGSB_E_INVALID_ARG, "n_extra must be 0: the extra rows are the algorithm's");
    if (n_eq > 0 && (!C || !d)) return fail(LBFGSB_E_INVALID_ARG, "NULL constraint rows / targets");
    return LBFGSB_OK;
}

size_t al_rows_extra_bytes(int64_t n_eq) {
    return 4 * align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8) + align_up(sizeof(AlState));
}

// The inner solver has ended, or `confirm`: has found the end by a gradient carried by recurrence.  Everything up to the next inner
// solve's first step is enqueued here, nothing is waited for.
void enqueue_turn(lbfgsb_auglag* al, bool confirm) {
    lbfgsb_solver* s = al->inner;
    // (a convergence to be confirmed: the evaluation reopens the solver and the turn makes the test itself)
    const bool own_test = confirm && s->steps_since_refresh > 0 && one_workgroup_retests(s);
    if (!own_test) hipLaunchKernelGGL(k_al_reopen, dim3(1), dim3(64), 0, al->stream, s->bf.scal, s->dm.m, al->state);
    if (s->steps_since_refresh > 0) {
        enqueue_eval(s, 0, true, own_test, nullptr, &al->state->done);
        if (confirm && !own_test) enqueue_retest(s);
    }
    s->steps_since_refresh = 0;
    s->steps_since_set_x = 0;
    const bool stacked = al->variant == lbfgsb_auglag::kStacked, marginals = al->variant == lbfgsb_auglag::kMarginals;
    AlTurn a{};
    s->gram_ready = false;             // (the gradient is shifted, the pairs are dropped)
    a.n_eq = al->n_eq; a.cols = stacked ? s->dm.cols : s->dm.n; a.ld = al->c_ld;
    a.ctol = al->ao.ctol; a.max_outer = al->ao.max_outer; a.retest = confirm ? 1 : 0;
    a.fevals = stacked ? 0 : 1;        // (of a stacked subproblem's start this never counted)
    a.refuse = stacked ? 0 : 1;
    a.own_test = own_test ? 1 : 0; a.n = s->dm.n; a.op = s->op; a.x = s->bf.x; a.l = s->bf.l; a.u = s->bf.u;
    a.d = al->d_c; a.lambda = al->lambda; a.beta = al->beta_c; a.omega = al->omega_c; a.res = (double*)al->res_c; a.coef = al->coef;
    a.total = s->dm.n_extra > 0 ? s->bf.xres + s->dm.n_extra : nullptr;
    a.Crows = al->c_rows; a.g = s->bf.g; a.scal = s->bf.scal; a.hist = s->bf.hist; a.state = al->state; a.host = al->h_state;
    const bool f32 = al->c_dtype == LBFGSB_F32;
    if (!marginals && al->n_eq <= kShiftRowsMax && al->n_eq * a.cols <= kShiftMax) {
        hipLaunchKernelGGL((f32 ? k_al_turn<float, true> : k_al_turn<double, true>), dim3(1), dim3(kTurnThreads), 0, al->stream, a);
        return;
    }
    hipLaunchKernelGGL((k_al_turn<double, false>), dim3(1), dim3(kTurnThreads), 0, al->stream, a);
    if (marginals) {
        const int64_t blocks = s->dm.rows * ((s->dm.cols + 4 * kBlock - 1) / (4 * kBlock));
        hipLaunchKernelGGL(k_al_shift_marginals, dim3((unsigned)(blocks > 2048 ? 2048 : blocks)), dim3(kBlock), 0, al->stream, s->dm.rows,
                           s->dm.cols, (const double*)al->coef, s->bf.g, (const AlState*)al->state);
        return;
    }
    int64_t blocks = (a.cols + kBlock - 1) / kBlock;
    if (blocks > 1024) blocks = 1024;
    if (f32)
        hipLaunchKernelGGL(k_al_shift_g<float>, dim3((unsigned)blocks), dim3(kBlock), 0, al->stream, al->n_eq, a.cols, a.ld,
                           (const float*)al->c_rows, (const double*)al->coef, s->bf.g, (const AlState*)al->state);
    else
        hipLaunchKernelGGL(k_al_shift_g<double>, dim3((unsigned)blocks), dim3(kBlock), 0, al->stream, al->n_eq, a.cols, a.ld,
                           (const double*)al->c_rows, (const double*)al->coef, s->bf.g, (const AlState*)al->state);
}

}  // namespace

extern "C" {

void lbfgsb_auglag_default_options(lbfgsb_auglag_options* o) {
    if (!o) return;
    o->rho0 = 1.0; o->ctol = 1e-8; o->max_outer = 100;
}

size_t lbfgsb_auglag_workspace_bytes(int64_t n, int m, const lbfgsb_objective* obj, int64_t n_eq,
                                     const lbfgsb_options* opt) {
    if (check_al(n, obj, n_eq) != LBFGSB_OK) return 0;
    const size_t inner = lbfgsb_workspace_bytes(n, m, obj, opt);
    return inner ? inner + al_extra_bytes(obj->rows, n_eq) : 0;
}

int lbfgsb_auglag_create(lbfgsb_auglag** out, int64_t n, int m, const double* l, const double* u,
                         const lbfgsb_objective* obj, int64_t n_eq, const lbfgsb_options* opt,
                         const lbfgsb_auglag_options* aopt, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!out) return fail(LBFGSB_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    int rc = check_al(n, obj, n_eq);
    if (rc) return rc;
    lbfgsb_auglag_options ao;
    if (aopt) ao = *aopt; else lbfgsb_auglag_default_options(&ao);
    if (!(ao.rho0 > 0.0) || !(ao.ctol >= 0.0) || ao.max_outer < 1) return fail(LBFGSB_E_INVALID_ARG, "bad option value");
    if (!workspace || !obj->b) return fail(LBFGSB_E_INVALID_ARG, "NULL device pointer");
    const size_t inner_bytes = lbfgsb_workspace_bytes(n, m, obj, opt);
    if (inner_bytes == 0) return LBFGSB_E_INVALID_ARG;
    const size_t extra = al_extra_bytes(obj->rows, n_eq);
    if (workspace_bytes < inner_bytes + extra)
        return fail(LBFGSB_E_INVALID_ARG, "workspace too small: %zu < %zu bytes", workspace_bytes, inner_bytes + extra);
    if ((uintptr_t)workspace % 256) return fail(LBFGSB_E_INVALID_ARG, "workspace must be 256-byte aligned");

    lbfgsb_auglag* al = new (std::nothrow) lbfgsb_auglag();
    if (!al) return fail(LBFGSB_E_INVALID_ARG, "out of host memory");
    const int64_t rows_data = obj->rows - n_eq;
    al->ao = ao; al->n_eq = n_eq; al->n = n; al->d_c = obj->b + rows_data;
    al->stream = (hipStream_t)hip_stream; al->inner = nullptr; al->h_state = nullptr;
    char* w = (char*)workspace + align_up(inner_bytes);
    double* beta = (double*)w; w += align_up((size_t)obj->rows * 8);
    double* omega = (double*)w; w += align_up((size_t)obj->rows * 8);
    al->beta_c = beta + rows_data; al->omega_c = omega + rows_data;
    al->lambda = (double*)w; w += align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8);
    al->coef = (double*)w; w += align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8);
    al->state = (AlState*)w;
    al->variant = lbfgsb_auglag::kStacked;
    al->c_ld = obj->ld; al->c_dtype = obj->dtype;
    al->c_rows = (const char*)obj->A + (size_t)rows_data * (size_t)obj->ld * (obj->dtype == LBFGSB_F64 ? 8 : 4);
    lbfgsb_objective inner_obj = *obj;
    inner_obj.b = beta;
    inner_obj.row_weight = omega;
    rc = lbfgsb_create(&al->inner, n, m, l, u, &inner_obj, opt, workspace, inner_bytes, hip_stream);
    if (rc) { delete al; return rc; }
    al->res_c = al->inner->bf.row + rows_data;
    hipError_t e = hipHostMalloc((void**)&al->h_state, sizeof(AlState), kPinned);
    if (e != hipSuccess) { al->h_state = nullptr; lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e)); }
    int blocks = (int)((obj->rows + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_al_init, dim3(blocks), dim3(256), 0, al->stream, obj->rows, obj->b, beta, omega);
    launch_fill_zero(al->lambda, align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8), al->stream);
    e = hipStreamSynchronize(al->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "initialising: %s", hipGetErrorString(e)); }
    *out = al;
    return LBFGSB_OK;
}

size_t lbfgsb_auglag_rows_workspace_bytes(int64_t n, int m, const lbfgsb_objective* obj, int64_t n_eq,
                                          const lbfgsb_options* opt) {
    if (check_al_rows(obj, n_eq, (const double*)8, (const double*)8) != LBFGSB_OK) return 0;
    lbfgsb_objective o = *obj;
    o.n_extra = n_eq;
    const size_t inner = lbfgsb_workspace_bytes(n, m, &o, opt);
    return inner ? align_up(inner) + al_rows_extra_bytes(n_eq) : 0;
}

int lbfgsb_auglag_create_rows(lbfgsb_auglag** out, int64_t n, int m, const double* l, const double* u,
                              const lbfgsb_objective* obj, int64_t n_eq, const double* C, const double* d,
                              const lbfgsb_options* opt, const lbfgsb_auglag_options* aopt, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
    if (!out) return fail(LBFGSB_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    int rc = check_al_rows(obj, n_eq, C, d);
    if (rc) return rc;
    lbfgsb_auglag_options ao;
    if (aopt) ao = *aopt; else lbfgsb_auglag_default_options(&ao);
    if (!(ao.rho0 > 0.0) || !(ao.ctol >= 0.0) || ao.max_outer < 1) return fail(LBFGSB_E_INVALID_ARG, "bad option value");
    if (!workspace) return fail(LBFGSB_E_INVALID_ARG, "NULL device pointer");
    lbfgsb_objective inner_obj = *obj;
    inner_obj.n_extra = n_eq;
    inner_obj.extra_rows = C;
    inner_obj.extra_target = (const double*)8;   // placeholders for the size computation; set below
    const size_t inner_bytes = lbfgsb_workspace_bytes(n, m, &inner_obj, opt);
    if (inner_bytes == 0) return LBFGSB_E_INVALID_ARG;
    const size_t extra = al_rows_extra_bytes(n_eq);
    if (workspace_bytes < align_up(inner_bytes) + extra)
        return fail(LBFGSB_E_INVALID_ARG, "workspace too small: %zu < %zu bytes", workspace_bytes, align_up(inner_bytes) + extra);
    if ((uintptr_t)workspace % 256) return fail(LBFGSB_E_INVALID_ARG, "workspace must be 256-byte aligned");

    lbfgsb_auglag* al = new (std::nothrow) lbfgsb_auglag();
    if (!al) return fail(LBFGSB_E_INVALID_ARG, "out of host memory");
    const size_t slot = align_up((size_t)(n_eq > 0 ? n_eq : 1) * 8);
    al->ao = ao; al->n_eq = n_eq; al->n = n; al->d_c = d;
    al->stream = (hipStream_t)hip_stream; al->inner = nullptr; al->h_state = nullptr;
    char* w = (char*)workspace + align_up(inner_bytes);
    al->beta_c = (double*)w; w += slot;
    al->omega_c = (double*)w; w += slot;
    al->lambda = (double*)w; w += slot;
    al->coef = (double*)w; w += slot;
    al->state = (AlState*)w;
    al->variant = lbfgsb_auglag::kRows;
    al->c_rows = C; al->c_ld = n; al->c_dtype = LBFGSB_F64;
    inner_obj.extra_target = al->beta_c;
    inner_obj.extra_weight = al->omega_c;
    rc = lbfgsb_create(&al->inner, n, m, l, u, &inner_obj, opt, workspace, inner_bytes, hip_stream);
    if (rc) { delete al; return rc; }
    al->res_c = al->inner->bf.xres;
    hipError_t e = hipHostMalloc((void**)&al->h_state, sizeof(AlState), kPinned);
    if (e != hipSuccess) { al->h_state = nullptr; lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e)); }
    launch_fill_zero(al->beta_c, 4 * slot, al->stream);
    e = hipStreamSynchronize(al->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "initialising: %s", hipGetErrorString(e)); }
    *out = al;
    return LBFGSB_OK;
}

size_t lbfgsb_auglag_marginals_workspace_bytes(int m, const lbfgsb_objective* obj, const lbfgsb_options* opt) {
    if (!obj || !is_transport(obj->kind)) { fail(LBFGSB_E_INVALID_ARG, "the marginal constraints go with the transport kinds"); return 0; }
    lbfgsb_objective o = *obj;
    o.n_extra = 0;
    const size_t inner = lbfgsb_workspace_bytes(o.rows * o.cols, m, &o, opt);
    return inner ? align_up(inner) + al_rows_extra_bytes(o.rows + o.cols) : 0;
}

int lbfgsb_auglag_create_marginals(lbfgsb_auglag** out, int m, const double* l, const double* u,
                                   const lbfgsb_objective* obj, const double* marginals, const lbfgsb_options* opt,
                                   const lbfgsb_auglag_options* aopt, void* workspace, size_t workspace_bytes,
                                   void* hip_stream) {
    if (!out) return fail(LBFGSB_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!obj || !is_transport(obj->kind)) return fail(LBFGSB_E_INVALID_ARG, "the marginal constraints go with the transport kinds");
    if (!marginals || !workspace) return fail(LBFGSB_E_INVALID_ARG, "NULL device pointer");
    lbfgsb_auglag_options ao;
    if (aopt) ao = *aopt; else lbfgsb_auglag_default_options(&ao);
    if (!(ao.rho0 > 0.0) || !(ao.ctol >= 0.0) || ao.max_outer < 1) return fail(LBFGSB_E_INVALID_ARG, "bad option value");
    lbfgsb_objective inner_obj = *obj;
    inner_obj.n_extra = 0;
    inner_obj.b = nullptr;
    inner_obj.row_weight = nullptr;
    const int64_t n = obj->rows * obj->cols, n_eq = obj->rows + obj->cols;
    const size_t inner_bytes = lbfgsb_workspace_bytes(n, m, &inner_obj, opt);
    if (inner_bytes == 0) return LBFGSB_E_INVALID_ARG;
    const size_t extra = al_rows_extra_bytes(n_eq);
    if (workspace_bytes < align_up(inner_bytes) + extra)
        return fail(LBFGSB_E_INVALID_ARG, "workspace too small: %zu < %zu bytes", workspace_bytes, align_up(inner_bytes) + extra);
    if ((uintptr_t)workspace % 256) return fail(LBFGSB_E_INVALID_ARG, "workspace must be 256-byte aligned");

    lbfgsb_auglag* al = new (std::nothrow) lbfgsb_auglag();
    if (!al) return fail(LBFGSB_E_INVALID_ARG, "out of host memory");
    const size_t slot = align_up((size_t)n_eq * 8);
    al->ao = ao; al->n_eq = n_eq; al->n = n; al->d_c = marginals;
    al->stream = (hipStream_t)hip_stream; al->inner = nullptr; al->h_state = nullptr;
    char* w = (char*)workspace + align_up(inner_bytes);
    al->beta_c = (double*)w; w += slot;
    al->omega_c = (double*)w; w += slot;
    al->lambda = (double*)w; w += slot;
    al->coef = (double*)w; w += slot;
    al->state = (AlState*)w;
    al->variant = lbfgsb_auglag::kMarginals;
    inner_obj.b = al->beta_c;
    inner_obj.row_weight = al->omega_c;
    int rc = lbfgsb_create(&al->inner, n, m, l, u, &inner_obj, opt, workspace, inner_bytes, hip_stream);
    if (rc) { delete al; return rc; }
    al->res_c = al->inner->bf.row;
    hipError_t e = hipHostMalloc((void**)&al->h_state, sizeof(AlState), kPinned);
    if (e != hipSuccess) { al->h_state = nullptr; lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e)); }
    launch_fill_zero(al->beta_c, 4 * slot, al->stream);
    e = hipStreamSynchronize(al->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { lbfgsb_auglag_destroy(al); return fail(LBFGSB_E_HIP, "initialising: %s", hipGetErrorString(e)); }
    *out = al;
    return LBFGSB_OK;
}

void lbfgsb_auglag_destroy(lbfgsb_auglag* al) {
    if (!al) return;
    lbfgsb_destroy(al->inner);
    if (al->h_state) (void)hipHostFree(al->h_state);
    delete al;
}

int lbfgsb_auglag_solve(lbfgsb_auglag* al, const double* x0, lbfgsb_auglag_info* info) {
    if (!al || !x0) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    lbfgsb_solver* s = al->inner;
    const int pb = (int)((al->n_eq + 255) / 256) > 0 ? (int)((al->n_eq + 255) / 256) : 1;
    // lambda^0 = 0, rho = rho0; the violation at x^0 is what the first iteration is compared with
    launch_fill_zero(al->lambda, align_up((size_t)(al->n_eq > 0 ? al->n_eq : 1) * 8), al->stream);
    hipLaunchKernelGGL(k_al_prepare, dim3(pb), dim3(256), 0, al->stream, al->n_eq, al->ao.rho0, al->d_c, al->lambda,
                       al->beta_c, al->omega_c);
    int rc = lbfgsb_set_x(s, x0);
    if (rc) return rc;
    hipLaunchKernelGGL(k_al_begin, dim3(1), dim3(kTurnThreads), 0, al->stream, al->n_eq, al->ao.rho0, al->res_c, al->state);
    volatile AlState* end = al->h_state;
    end->done = 0;
    s->steps_only = false;
    const bool quad = is_quadratic(s->dm.kind);
    Follower run(s);
    run.begin(0);
    for (int turns = 0;;) {
        int st = LBFGSB_RUNNING;
        if (s->use_resident) {
            rc = solve_impl(s, nullptr);
            st = s->h_scal->status;
        } else {
            rc = run.until_over(&st);
        }
        if (rc) return rc;
        if (end->done) break;          // (by the turn in front of the steps that report the end)
        if (st == -1) {
            HIP_TRY(read_scal(s));
            st = s->h_scal->status;
            if (st == LBFGSB_RUNNING && run.steps < run.cap) { run.resume(); continue; }
        }
        if (st == LBFGSB_LINESEARCH_FAILED) {
            hipLaunchKernelGGL(k_al_report, dim3(1), dim3(64), 0, al->stream, (const AlState*)al->state, al->h_state);
            HIP_TRY(read_scal(s));
            al->h_state->outer += 1;
            al->h_state->inner_iters += s->h_scal->iters;
            al->h_state->pg2 = s->h_scal->pg2;
            al->h_state->status = LBFGSB_LINESEARCH_FAILED;
            break;
        }
        enqueue_turn(al, st == LBFGSB_CONVERGED && quad && s->steps_since_refresh > 0);
        HIP_TRY(hipGetLastError());
        if (++turns >= al->ao.max_outer || s->use_resident) {
            // (the last one, unless convergence was not confirmed: no step is enqueued behind it in vain)
            HIP_TRY(hipStreamSynchronize(s->stream));
            if (end->done) break;
        }
        run.begin(0);
    }
    HIP_TRY(read_scal(s));             // (waits for the steps behind the end, whatever it was)
    HIP_TRY(hipGetLastError());
    if (end->nonfinite) {
        s->x_set = false;
        return fail(LBFGSB_E_NONFINITE, "the augmented Lagrangian is not finite at the iterate");
    }
    if (info) {
        const AlState& e = *al->h_state;
        *info = lbfgsb_auglag_info{};
        info->status = e.status; info->outer = e.outer; info->inner_iters = e.inner_iters;
        info->violation = e.violation; info->rho = e.rho; info->f = e.f; info->L = e.L; info->pg2 = e.pg2;
    }
    return LBFGSB_OK;
}

int lbfgsb_auglag_get_x(lbfgsb_auglag* al, double* x_out) {
    if (!al) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    return lbfgsb_get_x(al->inner, x_out);
}

int lbfgsb_auglag_get_lambda(lbfgsb_auglag* al, double* lambda_out) {
    if (!al || !lambda_out) return fail(LBFGSB_E_INVALID_ARG, "NULL argument");
    if (al->n_eq > 0)
        HIP_TRY(hipMemcpyAsync(lambda_out, al->lambda, (size_t)al->n_eq * 8, hipMemcpyDeviceToDevice, al->stream));
    return LBFGSB_OK;
}

lbfgsb_solver* lbfgsb_auglag_inner(lbfgsb_auglag* al) { return al ? al->inner : nullptr; }

}  // extern "C"

namespace {
__global__ __launch_bounds__(kBlock) void k_dbg_elementary(int which, int64_t n, const double* __restrict__ x, double* __restrict__ y) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        y[i] = which == 0 ? log_d(x[i]) : (which == 1 ? log1p_d(x[i]) : quotient_d(which == 2 ? 1.0 : x[i], 1.0 + x[i]));
}
}  // namespace

extern "C" {

int lbfgsb_dbg_elementary(int which, int64_t n, const double* x, double* y) {
    if (which < 0 || which > 3 || n <= 0 || !x || !y) return fail(LBFGSB_E_INVALID_ARG, "which must be 0 to 3, n > 0, x and y not NULL");
    const int64_t blocks = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_dbg_elementary, dim3((unsigned)(blocks > 4096 ? 4096 : blocks)), dim3(kBlock), 0, nullptr, which, n, x, y);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(nullptr));
    return LBFGSB_OK;
}

}  // extern "C"
