// Regularised optimal-transport objective of the paper's section "Joint Probability Distribution":
//     f(P) = <M,P> + lambda sum_ij phi(P_ij) + 0.5 sum_k omega_k ((K P)_k - beta_k)^2,
// P a rows x cols matrix stored row by row (the solver's variable vector), phi(p) = p^2/2 (Gaussian
// regulariser) or p log p (entropy), K P = [P 1; P^T 1] the rows + cols marginals.  The last term is how the
// augmented Lagrangian of Eq. (augLag) enters for the constraints P 1 = u, P^T 1 = v: omega = rho and
// beta = [u; v] - multipliers/rho, rewritten by Algorithm 4 between inner solves.
//
// There is no matrix-vector product here: every kernel streams n = rows*cols-entry vectors once.
//   k_ot_sums + k_ot_cols   K z for z = x (evaluation) or the selected direction p, the loss partials
//   k_ot_eval_finish        gradient M + lambda phi'(P) + K^T (omega . residual), objective value
//   k_ot_update_gauss       closed-form Armijo search (the objective is quadratic along p) and the update
//   k_ot_ls_* / k_ot_update_entropy   the same for the entropy, whose line search
//                           needs one pass over (x, p) per batch of trial steps
#include <cstddef>
#include <type_traits>

#include "common.h"

namespace lb {

namespace {

__device__ __forceinline__ double m_at(const void* M, int dtype, int64_t idx) {
    return dtype == LBFGSB_F32 ? (double)((const float*)M)[idx] : ((const double*)M)[idx];
}

// lambda * phi(p) and lambda * phi'(p)
__device__ __forceinline__ double reg_value(int kind, double lambda, double p) {
    if (kind == LBFGSB_OBJ_OT_GAUSS) return 0.5 * lambda * p * p;
    return p > 0.0 ? lambda * p * log_d(p) : 0.0;
}
__device__ __forceinline__ double reg_slope(int kind, double lambda, double p) {
    if (kind == LBFGSB_OBJ_OT_GAUSS) return lambda * p;
    return lambda * (log_d(p) + 1.0);
}

// Entropy: f(x + a p) - f(x) = a <g,p> + a^2/2 sum omega (K p)^2 + lambda sum_ij D(x_ij + a p_ij ; x_ij) with the
// Bregman divergence of p log p,  D(xt; x) = xt log(xt/x) - (xt - x) = x h(r),  r = (xt - x)/x,
// h(r) = (1 + r) log(1 + r) - r  (series for small r, where the closed form cancels).
__device__ __forceinline__ double entropy_h(double r) {
    if (r <= -1.0) return 1.0;                       // xt = 0: 0 log 0 = 0
    if (fabs(r) < 1e-2) {
        const double r2 = r * r;
        return r2 * (0.5 + r * (-1.0 / 6.0 + r * (1.0 / 12.0 + r * (-1.0 / 20.0 + r * (1.0 / 30.0 + r * (-1.0 / 42.0))))));
    }
    return (1.0 + r) * log1p_d(r) - r;
}

// Does the row-sum kernel form the first step length's sum?  It saves a launch and a trip of p from memory, where its workgroups
// fill the chip or have little to do, and are not so many that adding their sums costs more.  Whole runs, us, a launch of its own /
// in the row sums: 32 x 2000 1421 / 1401, 128 x 1000 1439 / 1404, 128 x 4000 1703 / 1687, 250 x 1000 1405 / 1350, 300 x 300 1389 / 1368,
// 1000 x 1000 2348 / 2288; but 64 x 8000 1857 / 1929, 20 000 x 40 (1250 workgroups) 3567 / 3596.
bool ot_sums_first_length(const Dims& dm, const Geometry& ge) {
    return dm.kind == LBFGSB_OBJ_OT_ENTROPY && ge.ot_row_blocks <= 512 && (ge.ot_row_blocks >= 192 || ge.ot_rpw * dm.cols <= 4096);
}

// K z, first half: the sums of the RPW rows this workgroup owns, and its partial column sums.  first (or null): the entropy's
// line search, sum_e x_e h(a_0 z_e / x_e) over these rows.  wt (or null): omega . (K z) as well.
template <int RPW>
__global__ __launch_bounds__(kBlock) void k_ot_sums(Dims dm, OtArgs a, int eval, int check_status,
                                                    const double* __restrict__ x, const double* __restrict__ p1,
                                                    const double* __restrict__ p2, Scal* __restrict__ scal,
                                                    double* __restrict__ out, double* __restrict__ wpart,
                                                    double* __restrict__ losspart, const double* __restrict__ dir_part,
                                                    int dir_blocks, double eps, Scal* __restrict__ scal_next, double* __restrict__ first, double* __restrict__ wt) {
    __shared__ double red[kWaves * (RPW + 1 > 7 ? RPW + 1 : 7)];
    const int tid = threadIdx.x;
    const int status = check_status ? (scal_next ? scal_next : scal)->status : LBFGSB_RUNNING;
    const double* z = x;
    double a0 = 1.0;
    if (!eval && dir_blocks > 0) {
        // Algorithm 2's choice from the direction kernel's per-workgroup sums (requested together with the status
        // word); workgroup 0 records it for the kernels that follow, and moves the copy of the scalar block that the
        // direction kernel has left in scal_next into place, the choice written into it on the way
        const bool move = scal_next && blockIdx.x == 0 && scal_next->fresh;
        const DirChoice ch = dir_choice_block(dir_part, dir_blocks, eps, red);
        if (move) {
            for (int k = tid; k < (int)(sizeof(Scal) / 4); k += kBlock) {
                int v = reinterpret_cast<const int*>(scal_next)[k];
                if (status == LBFGSB_RUNNING) v = scal_word_with_choice(k, v, ch);
                if (k == (int)(offsetof(Scal, fresh) / 4)) v = 0;
                reinterpret_cast<int*>(scal)[k] = v;
            }
            __syncthreads();                                   // (every thread has read `fresh`)
            if (tid == 0) scal_next->fresh = 0;
        }
        if (status != LBFGSB_RUNNING) return;
        if (blockIdx.x == 0 && tid == 0 && !move) {
            scal->branch = ch.branch; scal->gp = ch.gp; scal->alpha_ub = ch.alpha_ub; scal->pp = ch.pp; scal->xp = ch.xp;
        }
        z = ch.branch == 1 ? p1 : p2;
        a0 = fmin(1.0, ch.alpha_ub);
    } else {
        if (status != LBFGSB_RUNNING) return;
        if (!eval) { z = scal->branch == 1 ? p1 : p2; a0 = fmin(1.0, scal->alpha_ub); }
    }
    const int64_t r0 = (int64_t)blockIdx.x * RPW;
    const int nr = dm.rows - r0 < RPW ? (int)(dm.rows - r0) : RPW;
    double acc[RPW + 1];   // row sums, then the objective terms of these entries
#pragma unroll
    for (int r = 0; r <= RPW; ++r) acc[r] = 0.0;
    // several column tiles per round, all their loads issued before the first is used: the loop over the tiles is
    // otherwise a chain of dependent trips to memory, and this kernel is nothing else
    constexpr int JT = RPW <= 4 ? 4 : 2;
    for (int64_t j0 = 0; j0 < dm.cols; j0 += JT * kBlock) {
        double zv[JT][RPW];
#pragma unroll
        for (int t = 0; t < JT; ++t) {
            const int64_t j = j0 + t * kBlock + tid;
#pragma unroll
            for (int r = 0; r < RPW; ++r) zv[t][r] = (j < dm.cols && r < nr) ? z[(r0 + r) * dm.cols + j] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < JT; ++t) {
            const int64_t j = j0 + t * kBlock + tid;
            const bool in = j < dm.cols;
            double cs = 0.0;
#pragma unroll
            for (int r = 0; r < RPW; ++r) { cs += zv[t][r]; acc[r] += zv[t][r]; }
            if (eval) {
#pragma unroll
                for (int r = 0; r < RPW; ++r) {
                    if (in && r < nr) {
                        acc[RPW] = fma(m_at(a.M, dm.dtype, (r0 + r) * dm.ld + j), zv[t][r], acc[RPW]);
                        acc[RPW] += reg_value(dm.kind, dm.lambda, zv[t][r]);
                    }
                }
            }
            if (in) wpart[(int64_t)blockIdx.x * dm.cols + j] = cs;
        }
    }
    block_sum<RPW + 1, kWaves>(acc, red);
    if (tid == 0) {
        double loss = eval ? acc[RPW] : 0.0;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            if (r < nr) {
                // beta is only there together with omega (no marginal terms: the plain sums are left in `out`)
                const double res = (eval && a.omega) ? acc[r] - a.beta[r0 + r] : acc[r];
                out[r0 + r] = res;
                if (wt) wt[r0 + r] = a.omega ? a.omega[r0 + r] * res : 0.0;
                if (a.omega) loss += (eval ? 0.5 : 1.0) * a.omega[r0 + r] * res * res;
            }
        }
        losspart[blockIdx.x] = loss;
    }
    if (first) {
        // (the rows' entries once more, from the cache: the sums above want all of a column's rows in flight, the logarithms a few)
        const int64_t e_end = (r0 + nr) * dm.cols;
        double s[1] = {0.0};
        for (int64_t e0 = r0 * dm.cols + tid; e0 < e_end; e0 += 4 * kBlock) {
            double xv[4], pv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t e = e0 + k * kBlock < e_end ? e0 + k * kBlock : e0;
                xv[k] = x[e];
                pv[k] = z[e];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double h = entropy_h(a0 * (pv[k] / xv[k]));
                s[0] = e0 + k * kBlock < e_end ? fma(xv[k], h, s[0]) : s[0];
            }
        }
        block_sum<1, kWaves>(s, red);
        if (tid == 0) first[blockIdx.x] = s[0];
    }
}

// K z, second half: the column sums from the workgroups' partials.
__global__ __launch_bounds__(kBlock) void k_ot_cols(Dims dm, OtArgs a, int eval, int check_status, int parts,
                                                    const double* __restrict__ wpart, const Scal* __restrict__ scal,
                                                    double* __restrict__ out, double* __restrict__ losspart, double* __restrict__ wt) {
    __shared__ double lds[kBlock];
    __shared__ double red[kWaves];
    if (check_status && scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    double loss[1] = {0.0};
    for (int64_t c0 = (int64_t)blockIdx.x * kCX; c0 < dm.cols; c0 += (int64_t)gridDim.x * kCX) {
        const int64_t c = c0 + tid % kCX;
        const double s = column_sum(wpart, parts, dm.cols, c, lds);
        if (tid < kCX && c < dm.cols) {
            const double res = (eval && a.omega) ? s - a.beta[dm.rows + c] : s;
            out[dm.rows + c] = res;
            if (wt) wt[dm.rows + c] = a.omega ? a.omega[dm.rows + c] * res : 0.0;
            if (a.omega) loss[0] += (eval ? 0.5 : 1.0) * a.omega[dm.rows + c] * res * res;
        }
    }
    block_sum<1, kWaves>(loss, red);
    if (tid == 0) losspart[blockIdx.x] = loss[0];
}

// The gradient's and the entropy update's kernel: a workgroup takes R consecutive rows, a thread a column of them at a time, so
// that the column's coefficient -- three loads -- is formed once for R entries and the loads of all R are issued before the first
// is used.  R is the least that leaves 512 workgroups (the update ends in an arrival), four at most: registers.  What bounds
// them is memory and, for the entropy, the logarithm.  Entropy, 2 10^6 entries: update 35.5 us (128 MB), gradient 10.7 (52 and 27
// with one entry at a time and the fences arrive_is_last had); whole runs of 17 to 46 steps, with the runtime's logarithm and
// the former Gram kernels / now, us: 1000 x 1000 3350 / 2800, 700 x 630 2290 / 1820, 300 x 300 (m = 5) 1660 / 1530, 1901 x 333 fp32
// 3900 / 2320, 251 x 997 2190 / 1630.
// Few rows: the workgroups of a group of rows share its columns (split), so that there are up to 512 of them.  Few columns: a row's
// columns take a power of two of lanes and the workgroup as many groups of rows as it has such sets of lanes (SHORT).  Entropy,
// whole runs, us, one workgroup per group of rows and all of its threads along a row / this (the last workgroup's own loop,
// eight to a trip, included): 1 x 500 000 35 100 / 19 000, 5 x 200 000 20 000 / 11 600, 16 x 100 000 12 150 / 8 230, 40 x 20 000 3 880 /
// 3 400, 100 000 x 16 14 650 / 10 560, 100 000 x 40 18 860 / 15 680, 30 000 x 64 6 300 / 5 550, 8000 x 128 3 090 / 3 000; 8000 x 129, where
// a row has the workgroup for itself, the same.
constexpr int kOtRowsMax = 4;
constexpr int kOtShortCols = 128;   // up to this many columns a row takes a part of the workgroup
struct OtShape { int threads, rows, lanes_log2, groups, split; };   // lanes_log2: SHORT, else 0
inline OtShape ot_shape(const Dims& dm) {
    OtShape s{dm.cols > 384 ? 512 : 256, 1, 0, 1, 1};
    if (dm.cols <= kOtShortCols) {
        s.lanes_log2 = 4;
        while ((1 << s.lanes_log2) < dm.cols) ++s.lanes_log2;
    }
    const int sets = s.lanes_log2 ? s.threads >> s.lanes_log2 : 1;   // of rows, side by side in a workgroup
    const int64_t wgs = (dm.rows + sets - 1) / sets;
    s.rows = wgs > 1024 ? 4 : (wgs > 512 ? 2 : 1);
    const int64_t groups = (dm.rows + (int64_t)sets * s.rows - 1) / ((int64_t)sets * s.rows);
    s.groups = (int)(groups > 512 ? 512 : groups);
    const int64_t tiles = (dm.cols + s.threads - 1) / s.threads;
    // (four columns a thread at least: each workgroup of the update is an arrival more; 128 x 2000, 512 workgroups for 128: 11.3 us, not 9.8)
    s.split = (int)(512 / s.groups < (tiles + 3) / 4 ? 512 / s.groups : (tiles + 3) / 4);
    return s;
}
// This thread's first group of rows, the stride to its next one, its first column and the stride to its next one.
template <int NT, int R, bool SHORT>
struct OtPlace {
    int64_t row0, row_step, col0, col_step;
    __device__ __forceinline__ explicit OtPlace(int lanes_log2) {
        if (SHORT) {
            const int sets = NT >> lanes_log2;
            row0 = ((int64_t)blockIdx.x * sets + (threadIdx.x >> lanes_log2)) * R;
            row_step = (int64_t)gridDim.x * sets * R;
            col0 = threadIdx.x & ((1 << lanes_log2) - 1);
            col_step = 1 << lanes_log2;
        } else {
            row0 = (int64_t)blockIdx.x * R;
            row_step = (int64_t)gridDim.x * R;
            col0 = (int64_t)blockIdx.y * NT + threadIdx.x;
            col_step = (int64_t)gridDim.y * NT;
        }
    }
};

// g = M + lambda phi'(x) + K^T (omega . residual); the first workgroup adds up f.
template <int NT, int R, bool SHORT>
__global__ __launch_bounds__(NT) void k_ot_eval_finish(Dims dm, OtArgs a, int loss_parts, int lanes_log2, const double* __restrict__ x,
                                                       const double* __restrict__ res, const double* __restrict__ losspart,
                                                       double* __restrict__ g, Scal* __restrict__ scal) {
    __shared__ double red[NT / 64];
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        const double f = sum_all<NT>(losspart, loss_parts, red);   // (all of earlier launches)
        if (tid == 0) {
            scal->f = f;
            scal->fevals += 1;
            scal->gram_left = 0;
        }
    }
    const OtPlace<NT, R, SHORT> at(lanes_log2);
    for (int64_t r0 = at.row0; r0 < dm.rows; r0 += at.row_step) {
        double ri[R];
        int64_t row[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            row[r] = r0 + r < dm.rows ? r0 + r : dm.rows - 1;
            ri[r] = a.omega ? a.omega[row[r]] * res[row[r]] : 0.0;
        }
        for (int64_t j = at.col0; j < dm.cols; j += at.col_step) {
            double xv[R], mv[R];
#pragma unroll
            for (int r = 0; r < R; ++r) { xv[r] = x[row[r] * dm.cols + j]; mv[r] = m_at(a.M, dm.dtype, row[r] * dm.ld + j); }
            const double cj = a.omega ? a.omega[dm.rows + j] * res[dm.rows + j] : 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r)   // (a row past the end: the last row's entry once more)
                g[row[r] * dm.cols + j] = mv[r] + reg_slope(dm.kind, dm.lambda, xv[r]) + (ri[r] + cj);
        }
    }
}

constexpr int kOtTiles = 4;   // column tiles of a row whose loads the Gaussian update kernel keeps in flight together

// Gaussian regulariser: along p the objective is the quadratic  a <g,p> + a^2/2 (lambda <p,p> + sum omega (K p)^2),
// so the Armijo search is the closed form of the least-squares kinds; the change of the gradient is
// y = a (lambda p + K^T (omega . K p)).
__global__ __launch_bounds__(kBlock) void k_ot_update_gauss(Dims dm, Opts op, OtArgs a, int loss_parts,
                                                            const double* __restrict__ losspart,
                                                            const double* __restrict__ t, const double* __restrict__ p1,
                                                            const double* __restrict__ p2, const double* __restrict__ l,
                                                            const double* __restrict__ u, double* __restrict__ x,
                                                            double* __restrict__ g, double* __restrict__ S,
                                                            double* __restrict__ Y, Scal* __restrict__ scal) {
    __shared__ double red[kWaves];
    __shared__ double ls_alpha;
    __shared__ int ls_ok, ls_bt;
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    const double gp = scal->gp, alpha_ub = scal->alpha_ub, f_old = scal->f;
    const int slot = scal->head;
    const double* p = scal->branch == 1 ? p1 : p2;
    const double tt = sum_all(losspart, loss_parts, red) + dm.lambda * scal->pp;
    if (tid == 0) {
        int ok, bt;
        ls_alpha = armijo_quadratic(gp, tt, alpha_ub, op, ok, bt);
        ls_ok = ok; ls_bt = bt;
    }
    __syncthreads();
    const double alpha = ls_alpha;
    const int ok = ls_ok;
    if (ok) {
        double* Sn = S + (int64_t)slot * dm.n;
        double* Yn = Y + (int64_t)slot * dm.n;
        // kOtTiles column tiles of a row per round, all their loads issued before the first is used (one tile at a
        // time the row is a chain of dependent trips to memory)
        for (int64_t i = blockIdx.x; i < dm.rows; i += gridDim.x) {
            const double ri = a.omega ? a.omega[i] * t[i] : 0.0;
            for (int64_t j0 = 0; j0 < dm.cols; j0 += kOtTiles * kBlock) {
                double pv[kOtTiles], xv[kOtTiles], gv[kOtTiles], cv[kOtTiles], lv[kOtTiles], uv[kOtTiles];
#pragma unroll
                for (int k = 0; k < kOtTiles; ++k) {
                    const int64_t j = j0 + k * kBlock + tid;
                    const bool in = j < dm.cols;
                    const int64_t e = i * dm.cols + (in ? j : 0);
                    pv[k] = p[e]; xv[k] = x[e]; gv[k] = g[e];
                    cv[k] = (a.omega && in) ? a.omega[dm.rows + j] * t[dm.rows + j] : 0.0;
                    lv[k] = op.uniform_bounds ? op.lo : l[e];
                    uv[k] = op.uniform_bounds ? op.hi : u[e];
                }
#pragma unroll
                for (int k = 0; k < kOtTiles; ++k) {
                    const int64_t j = j0 + k * kBlock + tid;
                    if (j < dm.cols) {
                        const int64_t e = i * dm.cols + j;
                        const double y = alpha * fma(dm.lambda, pv[k], ri + cv[k]);
                        const double xn = clampd(fma(alpha, pv[k], xv[k]), lv[k], uv[k]);
                        Sn[e] = xn - xv[k];
                        Yn[e] = y;
                        x[e] = xn;
                        g[e] = gv[k] + y;
                    }
                }
            }
        }
    }
    // as in the least-squares update: no workgroup of this kernel reads the pend_* fields
    if (blockIdx.x == 0 && tid == 0) {
        scal->pend_ok = ok;
        scal->pend_bt = ls_bt;
        scal->pend_alpha = alpha;
        scal->pend_f = f_old + alpha * (gp + 0.5 * alpha * tt);
        scal->pend_valid = 1;
    }
}

// The step lengths are a_0 = min(1, bound), a_k = a_{k-1} backtrack.  From the second iteration of a run on the first is accepted
// nearly always, at a start on the lower bound, where p/x is huge, one after a dozen or more.  So a_0 is tested alone, from a sum
// that the row-sum kernel has formed on the way (where the rows are enough workgroups for a logarithm per entry, else a launch of
// its own), by the first of two further launches; if it is refused, that launch sums the 8 lengths k = kLsCoarse.  The second one
// looks for the first of these that is acceptable and sums what lies between it and the one before: the change of the objective
// along p is convex (the entropy is, and the marginal terms where their weights make a curvature sum omega (K p)^2 >= 0), so every
// length behind an acceptable one is acceptable and none before a refused one.  At most kLsFine lengths at a time; with a negative
// curvature all from the second on.  Only beyond k = 60, the default limit, does the last workgroup go on alone, one at a time.
// 2 10^6 entries, us: row sums 9, the first two lengths 15, the next eight 59, the remaining 51 287, the two launches when not needed
// 7 and 4.6 -> row sums with the first length 17.5, coarse lengths 51, fine 86, not needed 6.5 and 4.6.
constexpr int kLsCoarseCount = 8, kLsFine = 13, kLsAllMax = 54;
__device__ constexpr int kLsCoarse[kLsCoarseCount] = {1, 2, 3, 8, 14, 21, 34, 47};
constexpr int kLsLast = 60;

__device__ __forceinline__ double step_length(double a0, int k, double backtrack) {   // (the same multiplications everywhere)
    for (int j = 0; j < k; ++j) a0 *= backtrack;
    return a0;
}
// Armijo test of step length a, given sum_e x_e h(a p_e / x_e)
__device__ __forceinline__ bool entropy_accepts(double sum, double a, double gp, double tt, double lambda, const Opts& op) {
    const double df = a * (gp + 0.5 * a * tt) + lambda * sum;
    return isfinite(df) && df <= op.c1 * a * gp;
}

// block_sum for workgroups of many waves: thread k adds up the waves' sums of value k (every thread adding all of them
// keeps K NW values in registers).  lds: (NW + 1) K doubles.
template <int K, int NW>
__device__ __forceinline__ void block_sum_by_thread(double (&v)[K], double* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    __syncthreads();   // protect lds against readers of a previous use
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[wave * K + k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < K) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += lds[w * K + threadIdx.x];
        lds[NW * K + threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = lds[NW * K + k];
}

// sum over this workgroup's entries of x h(a_k p / x): GROUP lengths a[0 .. GROUP), or, where BACKTRACK, a[0], a[0] backtrack, ..
// (which are then not kept: the registers hold the sums)
template <int NT, int GROUP, bool BACKTRACK>
__device__ __forceinline__ void entropy_sums(int64_t n, const double* __restrict__ x, const double* __restrict__ p,
                                             const double (&a)[BACKTRACK ? 1 : GROUP], double backtrack, double (&s)[GROUP], double* red) {
#pragma unroll
    for (int k = 0; k < GROUP; ++k) s[k] = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
        const double xe = x[e], ratio = p[e] / xe;
        double ak = a[0];
#pragma unroll
        for (int k = 0; k < GROUP; ++k) {
            s[k] = fma(xe, entropy_h((BACKTRACK ? ak : a[BACKTRACK ? 0 : k]) * ratio), s[k]);
            if constexpr (BACKTRACK) {
                ak *= backtrack;
                asm volatile("" : "+v"(ak));
            }
            // (wide workgroups: one logarithm at a time)
            if constexpr (NT > kBlock) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (NT > kBlock) block_sum_by_thread<GROUP, NT / 64>(s, red);
    else block_sum<GROUP, NT / 64>(s, red);
}

// a_0 in a launch of its own
template <int NT>
__global__ __launch_bounds__(NT) void k_ot_ls_first(int64_t n, const double* __restrict__ x, const double* __restrict__ p1,
                                                    const double* __restrict__ p2, const Scal* __restrict__ scal,
                                                    double* __restrict__ first) {
    __shared__ double red[NT / 64 * 2];
    if (scal->status != LBFGSB_RUNNING) return;
    const double a[1] = {fmin(1.0, scal->alpha_ub)};
    double s[1];
    entropy_sums<NT, 1, false>(n, x, scal->branch == 1 ? p1 : p2, a, 1.0, s, red);
    if (threadIdx.x == 0) first[blockIdx.x] = s[0];
}

template <int NT>
__global__ __launch_bounds__(NT, NT > kBlock ? 4 : 1) void k_ot_ls_coarse(Dims dm, Opts op, int loss_parts, const double* __restrict__ losspart,
                                                     int first_parts, const double* __restrict__ first, const double* __restrict__ x,
                                                     const double* __restrict__ p1, const double* __restrict__ p2,
                                                     Scal* __restrict__ scal, double* __restrict__ coarse) {
    __shared__ double red[(NT / 64 + 1) * kLsCoarseCount];
    if (scal->status != LBFGSB_RUNNING) return;
    const double a0 = fmin(1.0, scal->alpha_ub), gp = scal->gp;
    const double* p = scal->branch == 1 ? p1 : p2;
    const double tt = sum_all<NT>(losspart, loss_parts, red);
    const double s0 = sum_all<NT>(first, first_parts, red);
    const bool ok = entropy_accepts(s0, a0, gp, tt, dm.lambda, op);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal->ls_first = ok;
        if (ok) {
            scal->ls_ok = 1;
            scal->backtracks = 0;
            scal->fevals += 1;
            scal->alpha = a0;
        }
    }
    if (ok) return;
    double a[kLsCoarseCount], s[kLsCoarseCount];
#pragma unroll
    for (int k = 0; k < kLsCoarseCount; ++k) a[k] = step_length(a0, kLsCoarse[k], op.backtrack);
    __syncthreads();   // (red is used again)
    entropy_sums<NT, kLsCoarseCount, false>(dm.n, x, p, a, op.backtrack, s, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kLsCoarseCount; ++k) coarse[(int64_t)blockIdx.x * kLsCoarseCount + k] = s[k];
    }
}

template <int NT>
__global__ __launch_bounds__(NT, NT > kBlock ? 4 : 1) void k_ot_ls_fine(Dims dm, Opts op, int loss_parts, const double* __restrict__ losspart,
                                                   const double* __restrict__ x, const double* __restrict__ p1,
                                                   const double* __restrict__ p2, Scal* __restrict__ scal,
                                                   const double* __restrict__ coarse, double* __restrict__ fine) {
    __shared__ double red[(NT / 64 + 1) * kLsFine];
    __shared__ int flag;
    // (ls_first, not the search's outcome: where the coarse lengths decide, workgroup 0 writes that while others are still to begin,
    // and the waves of a workgroup, each with a load of its own, would not all see the same)
    if (scal->status != LBFGSB_RUNNING || scal->ls_first) return;
    const int tid = threadIdx.x;
    const double a0 = fmin(1.0, scal->alpha_ub), gp = scal->gp;
    const double* p = scal->branch == 1 ? p1 : p2;
    double tc[kLsCoarseCount];
#pragma unroll
    for (int k = 0; k < kLsCoarseCount; ++k) tc[k] = 0.0;
    for (int b = tid; b < (int)gridDim.x; b += NT) {
#pragma unroll
        for (int k = 0; k < kLsCoarseCount; ++k) tc[k] += coarse[(int64_t)b * kLsCoarseCount + k];
    }
    const double tt = sum_all<NT>(losspart, loss_parts, red);
    if constexpr (NT > kBlock) block_sum_by_thread<kLsCoarseCount, NT / 64>(tc, red);
    else block_sum<kLsCoarseCount, NT / 64>(tc, red);
    // (every workgroup the same bits from here to the sums)
    const int most = op.max_backtracks;
    int lo = 1, hi = most < kLsAllMax ? most : kLsAllMax, stop = -1;   // stop: a coarse length known to be acceptable
    if (tt >= 0.0) {
        hi = most < kLsLast ? most : kLsLast;
#pragma unroll
        for (int k = 0; k < kLsCoarseCount; ++k) {
            if (stop < 0 && kLsCoarse[k] <= most) {
                if (entropy_accepts(tc[k], step_length(a0, kLsCoarse[k], op.backtrack), gp, tt, dm.lambda, op)) {
                    stop = kLsCoarse[k];
                    hi = stop - 1;
                } else {
                    lo = kLsCoarse[k] + 1;
                }
            }
        }
    }
    int found = stop;
    if (lo <= hi) {
        const double a_lo = step_length(a0, lo, op.backtrack);
        double a_group = a_lo;
#pragma unroll 1
        for (int k0 = lo; k0 <= hi; k0 += kLsFine) {
            const double a[1] = {a_group};
            double s[kLsFine];
            __syncthreads();
            entropy_sums<NT, kLsFine, true>(dm.n, x, p, a, op.backtrack, s, red);
            a_group = step_length(a_group, kLsFine, op.backtrack);
            if (tid == 0) {
#pragma unroll
                for (int k = 0; k < kLsFine; ++k)
                    if (k0 + k <= hi) publish(fine + (int64_t)blockIdx.x * kLsAllMax + (k0 - lo) + k, s[k]);
            }
        }
        if (!arrive_is_last(&scal->counters[kCntLs], &flag)) return;
        double a = a_lo;
#pragma unroll 1
        for (int k = lo; k <= hi; ++k) {
            double t[1] = {0.0};
            for (int b = tid; b < (int)gridDim.x; b += NT) t[0] += observe(fine + (int64_t)b * kLsAllMax + k - lo);
            block_sum<1, NT / 64>(t, red);
            if (entropy_accepts(t[0], a, gp, tt, dm.lambda, op)) { found = k; break; }
            a *= op.backtrack;
        }
    } else if (blockIdx.x != 0) {
        return;
    }
    // rare: one step length after the other, one workgroup alone (every thread holds the same totals: uniform control flow)
    for (int k = hi + 1; found < 0 && k <= most; ++k) {
        const double a = step_length(a0, k, op.backtrack);
        double sv[1] = {0.0};
        for (int64_t e = tid; e < dm.n; e += NT) sv[0] = fma(x[e], entropy_h(a * (p[e] / x[e])), sv[0]);
        block_sum<1, NT / 64>(sv, red);
        if (entropy_accepts(sv[0], a, gp, tt, dm.lambda, op)) found = k;
    }
    if (tid == 0) {
        // (no workgroup of this launch reads any of these)
        scal->ls_ok = found >= 0;
        scal->backtracks = found >= 0 ? found : most + 1;
        scal->fevals += found >= 0 ? found + 1 : most + 1;
        if (found >= 0) scal->alpha = step_length(a0, found, op.backtrack);
    }
}

// x+ = P(x + a p); g+ = M + lambda (log x+ + 1) + K^T (omega . (res + a K p)); pair; f+ from scratch at x+.
template <int NT, int R, bool SHORT>
__global__ __launch_bounds__(NT) void k_ot_update_entropy(Dims dm, Opts op, OtArgs a, int lanes_log2, double* res,
                                                          const double* __restrict__ t, const double* __restrict__ p1, const double* __restrict__ p2,
                                                          const double* __restrict__ l, const double* __restrict__ u,
                                                          double* __restrict__ x, double* __restrict__ g, double* __restrict__ S,
                                                          double* __restrict__ Y, Scal* __restrict__ scal,
                                                          double* __restrict__ redpart) {
    __shared__ double red[NT / 64];
    __shared__ int flag;
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    const int ok = scal->ls_ok;
    const double alpha = scal->alpha;
    const int slot = scal->head;
    const double* p = scal->branch == 1 ? p1 : p2;
    double fs[1] = {0.0};
    if (ok) {
        double* Sn = S + (int64_t)slot * dm.n;
        double* Yn = Y + (int64_t)slot * dm.n;
        const int64_t bstride = op.uniform_bounds ? 0 : 1;
        const OtPlace<NT, R, SHORT> at(lanes_log2);
        for (int64_t r0 = at.row0; r0 < dm.rows; r0 += at.row_step) {
            double ri[R];
            int64_t row[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                row[r] = r0 + r < dm.rows ? r0 + r : dm.rows - 1;
                ri[r] = a.omega ? a.omega[row[r]] * fma(alpha, t[row[r]], res[row[r]]) : 0.0;
            }
            for (int64_t j = at.col0; j < dm.cols; j += at.col_step) {
                double xv[R], pv[R], gv[R], mv[R], lv[R], uv[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int64_t e = row[r] * dm.cols + j;
                    xv[r] = x[e]; pv[r] = p[e]; gv[r] = g[e];
                    mv[r] = m_at(a.M, dm.dtype, row[r] * dm.ld + j);
                    lv[r] = op.lo; uv[r] = op.hi;
                    if (bstride) { lv[r] = l[e]; uv[r] = u[e]; }
                }
                const double cj = a.omega ? a.omega[dm.rows + j] * fma(alpha, t[dm.rows + j], res[dm.rows + j]) : 0.0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double xn = clampd(fma(alpha, pv[r], xv[r]), lv[r], uv[r]);
                    const double lg = log_d(xn);
                    const double gn = mv[r] + dm.lambda * (lg + 1.0) + (ri[r] + cj);
                    if (r0 + r < dm.rows) {
                        const int64_t e = row[r] * dm.cols + j;
                        Sn[e] = xn - xv[r];
                        Yn[e] = gn - gv[r];
                        x[e] = xn;
                        g[e] = gn;
                        fs[0] = fma(mv[r], xn, fs[0]);
                        if (xn > 0.0) fs[0] = fma(dm.lambda * xn, lg, fs[0]);
                    }
                }
            }
        }
    }
    block_sum<1, NT / 64>(fs, red);
    if (tid == 0) publish(redpart + blockIdx.y * gridDim.x + blockIdx.x, fs[0]);
    if (!arrive_is_last(&scal->counters[kCntUpdate], &flag)) return;
    double tot[1] = {0.0};
    for (int b = tid; b < (int)(gridDim.x * gridDim.y); b += NT) tot[0] += observe(redpart + b);
    if (ok) {
        // the residuals of the marginal terms move to the new point here, res += a K p: every other workgroup has
        // finished reading them (it has arrived)
        // (this workgroup alone: eight to a thread and trip, or the trips to memory of 10^5 of them last longer than the rest)
        const int64_t count = dm.rows + dm.cols;
        for (int64_t k0 = tid; k0 < count; k0 += 8 * NT) {
            double tv[8], rv[8], wv[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t k = k0 + q * NT < count ? k0 + q * NT : k0;
                tv[q] = t[k]; rv[q] = res[k];
                wv[q] = a.omega ? a.omega[k] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (k0 + q * NT < count) {
                    const double rn = fma(alpha, tv[q], rv[q]);
                    res[k0 + q * NT] = rn;
                    if (a.omega) tot[0] = fma(0.5 * wv[q] * rn, rn, tot[0]);
                }
            }
        }
    }
    block_sum<1, NT / 64>(tot, red);
    if (tid == 0) {
        if (ok) {
            scal->f = tot[0];
            scal->head = ring_next(slot, dm.m);
            scal->count = scal->count < dm.m ? scal->count + 1 : dm.m;
            scal->iters += 1;
            record_iteration(scal);
        } else if (scal->count > 0) {
            scal->count = 0;
            scal->memory_resets += 1;
        } else {
            scal->status = LBFGSB_LINESEARCH_FAILED;
        }
    }
}

template <int RPW>
void launch_sums_t(const Dims& dm, const Geometry& ge, const Buffers& bf, const OtArgs& a, int eval, int check_status,
                   hipStream_t st, int dir_blocks, double eps, Scal* scal_next) {
    hipLaunchKernelGGL(k_ot_sums<RPW>, dim3(ge.ot_row_blocks), dim3(kBlock), 0, st, dm, a, eval, check_status,
                       (const double*)bf.x, (const double*)bf.p1, (const double*)bf.p2, bf.scal, eval ? bf.row : bf.t,
                       bf.wpart, bf.losspart, (const double*)bf.redpart, eval ? 0 : dir_blocks, eps, scal_next,
                       !eval && ot_sums_first_length(dm, ge) ? bf.psi : nullptr, !eval && dm.kind == LBFGSB_OBJ_OT_GAUSS ? bf.psi : nullptr);
}

}  // namespace

void launch_ot_sums(const Dims& dm, const Geometry& ge, const Buffers& bf, const OtArgs& a, int eval, int check_status,
                    hipStream_t st, int dir_blocks, double eps, Scal* scal_next) {
    switch (ge.ot_rpw) {
        case 1: launch_sums_t<1>(dm, ge, bf, a, eval, check_status, st, dir_blocks, eps, scal_next); break;
        case 2: launch_sums_t<2>(dm, ge, bf, a, eval, check_status, st, dir_blocks, eps, scal_next); break;
        case 4: launch_sums_t<4>(dm, ge, bf, a, eval, check_status, st, dir_blocks, eps, scal_next); break;
        case 8: launch_sums_t<8>(dm, ge, bf, a, eval, check_status, st, dir_blocks, eps, scal_next); break;
        default: launch_sums_t<kOtRpwMax>(dm, ge, bf, a, eval, check_status, st, dir_blocks, eps, scal_next); break;
    }
    hipLaunchKernelGGL(k_ot_cols, dim3(ge.ot_col_blocks), dim3(kBlock), 0, st, dm, a, eval, check_status, ge.ot_row_blocks,
                       (const double*)bf.wpart, (const Scal*)bf.scal, eval ? bf.row : bf.t, bf.losspart + ge.ot_row_blocks,
                       !eval && dm.kind == LBFGSB_OBJ_OT_GAUSS ? bf.psi : nullptr);
}

// f(workgroup size, rows per group, short rows) for this shape's instantiation
template <class F>
static void with_ot_shape(const OtShape& s, F f) {
    auto rows = [&](auto nt, auto is_short) {
        switch (s.rows) {
            case 1: f(nt, std::integral_constant<int, 1>(), is_short); break;
            case 2: f(nt, std::integral_constant<int, 2>(), is_short); break;
            default: f(nt, std::integral_constant<int, kOtRowsMax>(), is_short); break;
        }
    };
    if (s.lanes_log2) rows(std::integral_constant<int, 256>(), std::true_type());
    else if (s.threads == 512) rows(std::integral_constant<int, 512>(), std::false_type());
    else rows(std::integral_constant<int, 256>(), std::false_type());
}

void launch_ot_eval_finish(const Dims& dm, const Geometry& ge, const Buffers& bf, const OtArgs& a, hipStream_t st) {
    const OtShape s = ot_shape(dm);
    with_ot_shape(s, [&](auto nt, auto rows, auto is_short) {
        hipLaunchKernelGGL((k_ot_eval_finish<nt(), rows(), is_short()>), dim3(s.groups, s.split), dim3(nt()), 0, st, dm, a,
                           ge.ot_row_blocks + ge.ot_col_blocks, s.lanes_log2, (const double*)bf.x, (const double*)bf.row,
                           (const double*)bf.losspart, bf.g, bf.scal);
    });
}

int ot_entry_blocks(const Dims& dm) {
    const OtShape s = ot_shape(dm);
    return s.groups * s.split;
}

void launch_ot_update_gauss(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const OtArgs& a,
                            hipStream_t st) {
    // (no closing arrival in this kernel: one workgroup per row)
    hipLaunchKernelGGL(k_ot_update_gauss, dim3((unsigned)(dm.rows > 2048 ? 2048 : dm.rows)), dim3(kBlock), 0, st, dm, op, a,
                       ge.ot_row_blocks + ge.ot_col_blocks, (const double*)bf.losspart, (const double*)bf.t,
                       (const double*)bf.p1, (const double*)bf.p2, (const double*)bf.l, (const double*)bf.u, bf.x, bf.g,
                       bf.S, bf.Y, bf.scal);
}

template <int NT>
static void launch_search_t(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, hipStream_t st) {
    // (a region of lspart for each launch)
    double* coarse = bf.lspart;
    double* fine = coarse + (size_t)ge.ls_blocks * kLsCoarseCount;
    double* first = fine + (size_t)ge.ls_blocks * kLsAllMax;
    static_assert(kLsCoarseCount + kLsAllMax + 1 <= 64, "lspart holds 64 sums per workgroup");
    const int loss_parts = ge.ot_row_blocks + ge.ot_col_blocks;
    const bool own = !ot_sums_first_length(dm, ge);
    if (own)
        hipLaunchKernelGGL((k_ot_ls_first<NT>), dim3(ge.ls_blocks), dim3(NT), 0, st, dm.n, (const double*)bf.x, (const double*)bf.p1,
                           (const double*)bf.p2, (const Scal*)bf.scal, first);
    hipLaunchKernelGGL((k_ot_ls_coarse<NT>), dim3(ge.ls_blocks), dim3(NT), 0, st, dm, op, loss_parts, (const double*)bf.losspart,
                       own ? ge.ls_blocks : ge.ot_row_blocks, own ? (const double*)first : (const double*)bf.psi, (const double*)bf.x,
                       (const double*)bf.p1, (const double*)bf.p2, bf.scal, coarse);
    hipLaunchKernelGGL((k_ot_ls_fine<NT>), dim3(ge.ls_blocks), dim3(NT), 0, st, dm, op, loss_parts, (const double*)bf.losspart,
                       (const double*)bf.x, (const double*)bf.p1, (const double*)bf.p2, bf.scal, (const double*)coarse, fine);
}
void launch_ot_step_entropy(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const OtArgs& a,
                            hipStream_t st) {
    if (ot_threads(dm) == 1024) launch_search_t<1024>(dm, op, ge, bf, st);
    else launch_search_t<256>(dm, op, ge, bf, st);
    const OtShape s = ot_shape(dm);
    with_ot_shape(s, [&](auto nt, auto rows, auto is_short) {
        hipLaunchKernelGGL((k_ot_update_entropy<nt(), rows(), is_short()>), dim3(s.groups, s.split), dim3(nt()), 0, st, dm, op, a,
                           s.lanes_log2, bf.row, (const double*)bf.t, (const double*)bf.p1, (const double*)bf.p2, (const double*)bf.l,
                           (const double*)bf.u, bf.x, bf.g, bf.S, bf.Y, bf.scal, bf.redpart);
    });
}

}  // namespace lb
