// The O(m*n) part of an iteration of Algorithm 1: free set (Eq. (ws)), the modified two-loop
// recursion (Algorithm 3) in batched form, projectDirection (Algorithm 2), the line search and the
// update of iterate, gradient and pair memory.  Every data-dependent decision is taken on the
// device by the last workgroup of the kernel that produces the numbers it depends on.
// (The free set, the Gram matrix and the recursion of Algorithm 3 are in gram.hip.)
#include "common.h"
#include "gram_close.h"

namespace lb {

__global__ void k_fill_zero(uint64_t* p, size_t words) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}
void launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
    const size_t words = bytes / 8;
    int blocks = (int)((words + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, st, (uint64_t*)p, words);
}

// ---- a new start point ----------------------------------------------------------------------------------
//
// Whether l <= x0 <= u and whether grad f(x0) is finite is found out on the device: the host used to fetch x0, l, u and g
// (32 MB at a million variables: 3 ms of a 7 ms call, 60 of 620 us at a hundred) to look at them itself.  Each kernel is
// one pass over its vectors; only a violation writes anything, a flag in pinned host memory.

__device__ __forceinline__ void fresh_block(Scal* scal, lbfgsb_iter_record* hist, int threads) {
    for (int k = threadIdx.x; k < (int)(sizeof(Scal) / 4); k += threads) reinterpret_cast<int*>(scal)[k] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        scal->status = LBFGSB_RUNNING;
        scal->alpha_ub = 1.0;
        scal->hist = hist;
    }
}
// some x0_i outside its bounds or NaN, among those of this thread
__device__ __forceinline__ bool outside_box(int64_t n, const Opts& op, const double* __restrict__ x0, const double* __restrict__ l,
                                            const double* __restrict__ u, int64_t first, int64_t step) {
    bool bad = false;
    for (int64_t i0 = first; i0 < n; i0 += 4 * step) {
        double v[4], lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + k * step, ic = i < n ? i : n - 1;
            v[k] = x0[ic];
            lo[k] = op.uniform_bounds ? op.lo : l[ic];
            hi[k] = op.uniform_bounds ? op.hi : u[ic];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) bad = bad || !(v[k] >= lo[k]) || !(v[k] <= hi[k]);
    }
    return bad;
}
__global__ __launch_bounds__(kBlock) void k_check_box(int64_t n, Opts op, const double* __restrict__ x0,
                                                      const double* __restrict__ l, const double* __restrict__ u,
                                                      int* __restrict__ host_flag) {
    const bool bad = outside_box(n, op, x0, l, u, (int64_t)blockIdx.x * kBlock + threadIdx.x, (int64_t)gridDim.x * kBlock);
    if (bad) *host_flag = 1;
}
__global__ __launch_bounds__(kBlock) void k_check_bounds(int64_t n, const double* __restrict__ l, const double* __restrict__ u,
                                                         BoundsReport* __restrict__ host) {
    const double l0 = l[0], u0 = u[0];
    bool crossed = false, differ = false, not_positive = false;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < n; i0 += 4 * (int64_t)gridDim.x * kBlock) {
        double lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + k * (int64_t)gridDim.x * kBlock, ic = i < n ? i : n - 1;
            lo[k] = l[ic]; hi[k] = u[ic];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            crossed = crossed || !(lo[k] <= hi[k]);
            differ = differ || lo[k] != l0 || hi[k] != u0;
            not_positive = not_positive || !(lo[k] > 0.0);
        }
    }
    // (one store per wave at most: bounds that differ do so everywhere)
    if (__any(crossed) && (threadIdx.x & 63) == 0) host->flag[0] = 1;
    if (__any(differ) && (threadIdx.x & 63) == 0) host->flag[1] = 1;
    if (__any(not_positive) && (threadIdx.x & 63) == 0) host->flag[2] = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) { host->lo = l0; host->hi = u0; }
}
__global__ __launch_bounds__(kBlock) void k_check_finite(int64_t n, const double* __restrict__ g, int* __restrict__ host_flag) {
    bool bad = false;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < n; i0 += 4 * (int64_t)gridDim.x * kBlock) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + k * (int64_t)gridDim.x * kBlock;
            v[k] = g[i < n ? i : n - 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) bad = bad || !isfinite(v[k]);
    }
    if (bad) host_flag[1] = 1;
}
__global__ __launch_bounds__(kBlock) void k_start(int64_t n, const double* x0, double* x, Scal* scal, lbfgsb_iter_record* hist) {
    if (blockIdx.x == 0) fresh_block(scal, hist, kBlock);
    if (x0 == x) return;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) x[i] = x0[i];
}
// Check and start in one launch, by one workgroup, and the evaluation is enqueued behind it without the host looking in between (a
// trip of ~12 us, and a launch of 4; another went with k_check_finite, whose test k_eval_finish makes).  Beyond kStartOneMax, where one
// compute unit takes ~8 us for the three vectors, the host's trip is under 1 % of what follows.  Whole calls, us: 200 x 100 402 -> 391,
// 3001 x 301 315 -> 302, 20000 x 5000 2750 -> 2737.
constexpr int kCheckStartThreads = 1024;
__global__ __launch_bounds__(kCheckStartThreads) void k_check_start(int64_t n, Opts op, const double* x0, const double* __restrict__ l,
                                                                    const double* __restrict__ u, double* x, Scal* scal,
                                                                    lbfgsb_iter_record* hist, int* __restrict__ host_flag) {
    if (__syncthreads_or(outside_box(n, op, x0, l, u, threadIdx.x, kCheckStartThreads))) {
        if (threadIdx.x == 0) {
            scal->status += kStatusRefused;
            host_flag[0] = 1;
        }
        return;
    }
    fresh_block(scal, hist, kCheckStartThreads);
    if (x0 == x) return;
    for (int64_t i = threadIdx.x; i < n; i += kCheckStartThreads) x[i] = x0[i];
}
__global__ void k_admit(Scal* scal) {
    if (threadIdx.x == 0) scal->status -= kStatusRefused;
}
static int start_blocks(int64_t n) {
    const int64_t b = (n + 4 * kBlock - 1) / (4 * kBlock);
    return (int)(b > 1024 ? 1024 : b);
}
void launch_check_bounds(const Dims& dm, const double* l, const double* u, BoundsReport* host, hipStream_t st) {
    hipLaunchKernelGGL(k_check_bounds, dim3(start_blocks(dm.n)), dim3(kBlock), 0, st, dm.n, l, u, host);
}
void launch_check_box(const Dims& dm, const Opts& op, const Buffers& bf, const double* x0, int* host_flag, hipStream_t st) {
    hipLaunchKernelGGL(k_check_box, dim3(start_blocks(dm.n)), dim3(kBlock), 0, st, dm.n, op, x0, (const double*)bf.l,
                       (const double*)bf.u, host_flag);
}
void launch_start(const Dims& dm, const Buffers& bf, const double* x0, hipStream_t st) {
    hipLaunchKernelGGL(k_start, dim3(start_blocks(dm.n)), dim3(kBlock), 0, st, dm.n, x0, bf.x, bf.scal, bf.hist);
}
void launch_check_start(const Dims& dm, const Opts& op, const Buffers& bf, const double* x0, int* host_flag, hipStream_t st) {
    hipLaunchKernelGGL(k_check_start, dim3(1), dim3(kCheckStartThreads), 0, st, dm.n, op, x0, (const double*)bf.l, (const double*)bf.u,
                       bf.x, bf.scal, bf.hist, host_flag);
}
void launch_admit(const Buffers& bf, hipStream_t st) { hipLaunchKernelGGL(k_admit, dim3(1), dim3(64), 0, st, bf.scal); }
void launch_check_finite(const Dims& dm, const double* g, int* host_flag, hipStream_t st) {
    hipLaunchKernelGGL(k_check_finite, dim3(start_blocks(dm.n)), dim3(kBlock), 0, st, dm.n, g, host_flag);
}

__global__ void k_clear_bail(Scal* scal) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        if (scal->status == kStatusBail) scal->status = LBFGSB_RUNNING;
        scal->bail_skipped = 0;
    }
}
void launch_clear_bail(const Buffers& bf, hipStream_t st) {
    hipLaunchKernelGGL(k_clear_bail, dim3(1), dim3(64), 0, st, bf.scal);
}

// ---- d = -B delta on the free set, then Algorithm 2 ------------------------------------------------------

// Extra dense rows of the objective (at most kFoldMax of them) folded into the direction kernel: their products
// with both candidate directions ride along with the other sums, the last workgroup turns the selected one into the
// coefficient weight_r (e_r . p) of the row's contribution to the gradient change and into the curvature term
// sum weight_r (e_r . p)^2, and the update kernel adds coef_r e_r on the fly.  (A kernel of its own for this, one
// workgroup between the direction kernel and the pass over A, cost 9 us plus a launch gap per iteration.)
struct FoldArgs {
    int n_fold;              // 0: nothing folded
    const double* E;         // n_fold x n, row-major
    const double* weight;    // n_fold entries or NULL (= ones)
    double* coef;            // out: n_fold coefficients
    double* total;           // out: sum weight_r (e_r . p)^2
};

// Partial sums of the direction kernels -> Algorithm 2's choice between the two candidate directions (last workgroup).
__device__ __forceinline__ void dir_finish(double (&s)[6], double ub, double eps, Scal* __restrict__ scal,
                                           double* __restrict__ redpart, double* red, int* flag_p,
                                           double (&sx)[2 * kFoldMax], const FoldArgs& fold, int defer_choice = 0) {
    const int tid = threadIdx.x;
    if (defer_choice) {
        // the consumer of the direction chooses between the candidates from the records: one exchange and one thread an entry
        const int wave = tid >> 6;
        const int lane = tid & 63;
        double eight[8] = {s[0], s[1], s[2], s[3], s[4], s[5], 0.0, 0.0};
        const double sum_of = wave_sums8(eight, lane);
        ub = wave_min(ub);
        if (fold.n_fold > 0) {
#pragma unroll
            for (int k = 0; k < 2 * kFoldMax; ++k) sx[k] = wave_sum(sx[k]);
        }
        if (lane < 7) red[wave * kDirRed + lane] = lane == 6 ? ub : sum_of;
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 2 * kFoldMax; ++k) red[wave * kDirRed + 8 + k] = sx[k];
        }
        __syncthreads();
        if (tid < kDirRed && tid != 7) {
            double sum = 0.0, least = red[tid];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                sum += red[w * kDirRed + tid];
                least = fmin(least, red[w * kDirRed + tid]);
            }
            publish(redpart + (int64_t)blockIdx.x * kDirRed + tid, tid == 6 ? least : sum);
        }
        return;
    }
    block_sum<6, kWaves>(s, red);
    if (fold.n_fold > 0) block_sum<2 * kFoldMax, kWaves>(sx, red);
    double mn = wave_min(ub);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = mn;
    __syncthreads();
    if (tid == 0) {
        mn = red[0];
        for (int w = 1; w < kWaves; ++w) mn = fmin(mn, red[w]);
        double* part = redpart + (int64_t)blockIdx.x * kDirRed;
        for (int k = 0; k < 6; ++k) publish(part + k, s[k]);
        publish(part + 6, mn);
        for (int k = 0; k < 2 * kFoldMax; ++k) publish(part + 8 + k, sx[k]);
    }
    if (!arrive_is_last(&scal->counters[kCntDir], flag_p)) return;
    double tx[2 * kFoldMax];
    {
        // the workgroups' partials, strided over the threads in a fixed order, then the fixed-order reductions
        double t6[6] = {0, 0, 0, 0, 0, 0};
        double tmin = INFINITY;
#pragma unroll
        for (int k = 0; k < 2 * kFoldMax; ++k) tx[k] = 0.0;
        for (int b = tid; b < (int)gridDim.x; b += kBlock) {
#pragma unroll
            for (int k = 0; k < 6; ++k) t6[k] += observe(redpart + (int64_t)b * kDirRed + k);
            tmin = fmin(tmin, observe(redpart + (int64_t)b * kDirRed + 6));
            if (fold.n_fold > 0) {
#pragma unroll
                for (int k = 0; k < 2 * kFoldMax; ++k) tx[k] += observe(redpart + (int64_t)b * kDirRed + 8 + k);
            }
        }
        block_sum<6, kWaves>(t6, red);
        if (fold.n_fold > 0) block_sum<2 * kFoldMax, kWaves>(tx, red);
        tmin = wave_min(tmin);
        __syncthreads();
        if ((tid & 63) == 0) red[tid >> 6] = tmin;
        __syncthreads();
        if (tid == 0) {
            tmin = red[0];
            for (int w = 1; w < kWaves; ++w) tmin = fmin(tmin, red[w]);
        }
        __syncthreads();
        if (tid == 0) {
            for (int k = 0; k < 6; ++k) red[k] = t6[k];
            red[6] = tmin;
        }
    }
    __syncthreads();
    if (tid == 0) {
        const double p1g = red[0], p1p1 = red[1];
        const int branch = (p1g <= -eps * p1p1 && p1p1 >= eps) ? 1 : 2;
        if (branch == 1) {
            scal->branch = 1; scal->gp = p1g; scal->alpha_ub = 1.0; scal->pp = p1p1; scal->xp = red[2];
        } else {
            scal->branch = 2; scal->gp = red[3]; scal->alpha_ub = red[6]; scal->pp = red[4]; scal->xp = red[5];
        }
        if (fold.n_fold > 0) {
            double total = 0.0;
#pragma unroll
            for (int r = 0; r < kFoldMax; ++r) {
                if (r < fold.n_fold) {
                    const double te = branch == 1 ? tx[2 * r] : tx[2 * r + 1];
                    const double wr = fold.weight ? fold.weight[r] : 1.0;
                    fold.coef[r] = wr * te;
                    total += wr * te * te;
                }
            }
            *fold.total = total;
        }
    }
}

// CLOSE: the Gram kernel before this one ended without its closing step.  Every workgroup here then does that step on a
// private copy of the scalar block: adds the records of partial sums in workgroup order, applies the pending update, runs
// Algorithm 3 on coefficients and the stopping test -- the same functions in the same order as the Gram kernel's last
// workgroup, so the same bits -- and takes the coefficients from its copy.  Workgroup 0 leaves its copy in scal_next for the
// pass (nothing in this kernel reads that); the scalar block itself is only read here.  What this saves is the Gram kernel's
// arrival (an atomic, a dependent round of loads) and this kernel's own dependent reads of the status word and the coefficients.
// What bounds it is the chain: 18 000 cycles, of them 6500 for the records, 3000 until the pair memory had been asked for, 3600 for the
// closing step, 2500 for the element and 2500 for the sums, when divisions found the ring's slots, the vectors' addresses went through
// LDS, an element took two quotients and 21 dependent additions, and the sums five barriers.  With comparisons, vectors by slot, one
// quotient, two chains and one exchange, per iteration, us: 4000 x 1500 36.9 -> 35.0, 8000 x 2000 47.5 -> 46.0, 20000 x 5000 1.3 less,
// transport of 200 x 200 1483 -> 1450 a run; from 30 000 variables on no less.  (All 20 slots' vectors asked for behind the records,
// before it is known which hold pairs: 0 to 2 % slower throughout.)
template <bool CLOSE>
__global__ __launch_bounds__(kBlock) void k_dir(int64_t n, int m, Opts op, const double* __restrict__ x,
                                                const double* __restrict__ g, const double* __restrict__ l,
                                                const double* __restrict__ u, const uint8_t* __restrict__ mask,
                                                const double* __restrict__ S, const double* __restrict__ Y,
                                                Scal* __restrict__ scal, double* __restrict__ d,
                                                double* __restrict__ p1, double* __restrict__ p2,
                                                double* __restrict__ redpart, int d_given, int store_d, FoldArgs fold,
                                                int defer_choice, GramRecords records, Scal* __restrict__ scal_next) {
    __shared__ double delta_s[kMaxV + 9];
    __shared__ const double* vecp[kMaxV + 8];
    __shared__ double red[kWaves * kDirRed];
    __shared__ int flag;
    const int tid = threadIdx.x;
    // What depends on nothing the scalar block says is requested together with it: the coefficients (masked by the
    // number of vectors afterwards) and the first element's x, g, l, u and mask -- otherwise three dependent trips.
    const int64_t e_first = (int64_t)blockIdx.x * kBlock + tid;
    const int64_t e_safe = e_first < n ? e_first : n - 1;
    double xn = x[e_safe], gn = g[e_safe], ln = l[e_safe], un = u[e_safe];
    uint8_t mkn = mask[e_safe];
    int c, head;
    // the first element's entries of the pair memory, slot by slot
    constexpr int kPre = CLOSE ? kGramOpenM : 1;
    double vy[kPre], vs[kPre];
#pragma unroll
    for (int k = 0; k < kPre; ++k) vy[k] = vs[k] = 0.0;
    __shared__ double coef_s[2 * kPre];
    const bool more = !CLOSE || (int64_t)gridDim.x * kBlock < n;   // (some thread has a second element)
    if constexpr (CLOSE) {
        __shared__ Scal sc;
        __shared__ double Gs[(2 * kGramOpenM + 2) * (2 * kGramOpenM + 2)];
        __shared__ double tot[gram_entries(kGramOpenM)];
        __shared__ double alpha_s[kMaxM + 1];
        constexpr int kScalWords = (int)(sizeof(Scal) / 4);
        for (int k = tid; k < kScalWords; k += kBlock)
            reinterpret_cast<int*>(&sc)[k] = reinterpret_cast<const int*>(scal)[k];
        int pa, pb;                                                // (worked out while the records are on their way)
        gram_product_slots(tid < gram_products(m) ? tid : 0, m, pa, pb);
        asm volatile("" : "+v"(pa), "+v"(pb));
        gram_sum_entries<kBlock>(records.part, gram_entries(m), records.count, tot);
        __syncthreads();
        if (sc.status != LBFGSB_RUNNING) {
            // (the pass reads its status word from scal_next: it must not find an older one there)
            if (blockIdx.x == 0 && tid == 0) { scal_next->status = sc.status; scal_next->fresh = 0; note_progress(op, sc.status); }
            return;
        }
        head = __builtin_amdgcn_readfirstlane(sc.head); c = __builtin_amdgcn_readfirstlane(sc.count);
        if (__builtin_amdgcn_readfirstlane(sc.pend_valid)) {       // same rule as effective_ring()
            if (__builtin_amdgcn_readfirstlane(sc.pend_ok)) { head = ring_next(head, m); c = c < m ? c + 1 : m; }
            else c = 0;
        }
        const int base_slot = ring_back(head, c, m);
        const double yn_old = prefetch_ynorm2(&sc, c, head, m);
        // the first element's entries are requested now (which slots hold pairs is known), so that their trip to memory runs under the
        // closing step instead of behind it
        if (mkn) {
#pragma unroll
            for (int q = 0; q < kPre; ++q) {
                const int age = q >= base_slot ? q - base_slot : q - base_slot + m;
                if (q >= m || age >= c) continue;                  // (uniform)
                vy[q] = (Y + (int64_t)q * n)[(unsigned)e_safe];
                vs[q] = (S + (int64_t)q * n)[(unsigned)e_safe];
            }
        }
        __syncthreads();                                           // every thread has read the ring before it changes
        gram_finish<kBlock, kGramOpenM, false>(tot, Gs, alpha_s, &sc, m, c, head, base_slot, op, yn_old, 0, 1, blockIdx.x == 0, pa, pb);
        __syncthreads();                                           // the first wave's results are in the copy
        if (blockIdx.x == 0) {
            if (tid == 0) note_progress(op, sc.status);
            for (int k = tid; k < kScalWords; k += kBlock) {
                int v = reinterpret_cast<const int*>(&sc)[k];
                if (k == (int)(offsetof(Scal, fresh) / 4)) v = 1;
                reinterpret_cast<int*>(scal_next)[k] = v;
            }
        }
        if (sc.status != LBFGSB_RUNNING) return;
        c = sc.count; head = sc.head;                              // (as computed above: the update has been applied)
        const int V = 2 * c + 1;
        if (tid < 2 * kPre) {
            // coefficient of slot tid of y, tid - kPre of s
            const int slot = tid < kPre ? tid : tid - kPre, age = slot >= base_slot ? slot - base_slot : slot - base_slot + m;
            coef_s[tid] = slot < m && age < c ? sc.delta[tid < kPre ? c + age : age] : 0.0;
        }
        if (more && tid < kMaxV + 8) {
            vecp[tid] = tid < V ? ring_vec(tid, c, head, m, n, S, Y, g) : g;
            delta_s[tid] = tid < V ? sc.delta[tid] : 0.0;
        }
        if (tid == 0) delta_s[kMaxV + 8] = sc.delta[2 * c];
    } else {
        const int status = scal->status;
        const double delta_raw = tid < kMaxV ? scal->delta[tid] : 0.0;
        if (status != LBFGSB_RUNNING) return;
        c = scal->count; head = scal->head;
        const int V = 2 * c + 1;
        if (tid < kMaxV + 8) {
            vecp[tid] = tid < V ? ring_vec(tid, c, head, m, n, S, Y, g) : g;
            delta_s[tid] = tid < V ? delta_raw : 0.0;
        }
    }
    const int V = 2 * c + 1;
    __syncthreads();
    double s[6] = {0, 0, 0, 0, 0, 0};
    double sx[2 * kFoldMax];
#pragma unroll
    for (int k = 0; k < 2 * kFoldMax; ++k) sx[k] = 0.0;
    double ub = INFINITY;
    for (int64_t e = e_first; e < n; e += (int64_t)gridDim.x * kBlock) {
        const double xe = xn, ge = gn, le = ln, ue = un;
        const uint8_t mk = mkn;
        if (more) {
            // the next element's, one trip ahead
            const int64_t e2 = e + (int64_t)gridDim.x * kBlock;
            const int64_t e2s = e2 < n ? e2 : n - 1;
            xn = x[e2s]; gn = g[e2s]; ln = l[e2s]; un = u[e2s]; mkn = mask[e2s];
        }
        double de;
        if (d_given) {
            de = d[e];
        } else {
            de = 0.0;
            if (mk) {
                double q = 0.0;
                if (CLOSE && e == e_first) {
                    double q1 = 0.0;
                    q = delta_s[kMaxV + 8] * ge;
#pragma unroll
                    for (int k = 0; k < kPre; ++k) {               // (slots that hold no pair: zero times zero)
                        q = fma(coef_s[k], vy[k], q);
                        q1 = fma(coef_s[kPre + k], vs[k], q1);
                    }
                    q += q1;
                } else {
                    for (int j0 = 0; j0 < V; j0 += 8) {
                        double v[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) v[k] = vecp[j0 + k][e];
#pragma unroll
                        for (int k = 0; k < 8; ++k) q = fma(delta_s[j0 + k], v[k], q);
                    }
                }
                de = -q;
            }
            if (store_d) d[e] = de;
        }
        const double a = clampd(xe + de, le, ue) - xe;
        double b = de;
        if (de < 0.0 && xe <= le + op.eps) b = 0.0;
        if (de > 0.0 && xe >= ue - op.eps) b = 0.0;
        p1[e] = a;
        p2[e] = b;
        s[0] = fma(a, ge, s[0]); s[1] = fma(a, a, s[1]); s[2] = fma(xe, a, s[2]);
        s[3] = fma(b, ge, s[3]); s[4] = fma(b, b, s[4]); s[5] = fma(xe, b, s[5]);
        const double room = ((b > 0.0 ? ue : le) - xe) / b;
        if (b != 0.0) ub = fmin(ub, room);
#pragma unroll
        for (int r = 0; r < kFoldMax; ++r) {
            if (r < fold.n_fold) {
                const double ev = fold.E[(int64_t)r * n + e];
                sx[2 * r] = fma(ev, a, sx[2 * r]);
                sx[2 * r + 1] = fma(ev, b, sx[2 * r + 1]);
            }
        }
    }
    dir_finish(s, ub, op.eps, scal, redpart, red, &flag, sx, fold, defer_choice);
}

// The same for long vectors (from 2^17 entries on): two elements per lane through 16-byte accesses; lanes whose elements are
// fixed skip the pair memory.  With odd n a vector of the pair memory may start on any element (the memory pipeline takes
// 16-byte accesses at any multiple of four), and the last pair's second element belongs to whatever follows in the workspace:
// it is read with the first, counts as fixed, and is not written.
typedef double dir_f64x2 __attribute__((ext_vector_type(2)));
typedef dir_f64x2 dir_f64x2_any __attribute__((aligned(8)));

__device__ __forceinline__ void dir_element(double xe, double ge, double le, double ue, double de, double eps, double& a,
                                            double& b, double (&s)[6], double& ub) {
    a = clampd(xe + de, le, ue) - xe;
    b = de;
    if (de < 0.0 && xe <= le + eps) b = 0.0;
    if (de > 0.0 && xe >= ue - eps) b = 0.0;
    s[0] = fma(a, ge, s[0]); s[1] = fma(a, a, s[1]); s[2] = fma(xe, a, s[2]);
    s[3] = fma(b, ge, s[3]); s[4] = fma(b, b, s[4]); s[5] = fma(xe, b, s[5]);
    if (b > 0.0) ub = fmin(ub, (ue - xe) / b);
    else if (b < 0.0) ub = fmin(ub, (le - xe) / b);
}

template <bool CLOSE>
__global__ __launch_bounds__(kBlock) void k_dir_pairs(int64_t n, int m, Opts op, const double* __restrict__ x,
                                                      const double* __restrict__ g, const double* __restrict__ l,
                                                      const double* __restrict__ u, const uint8_t* __restrict__ mask,
                                                      const double* __restrict__ S, const double* __restrict__ Y,
                                                      Scal* __restrict__ scal, double* __restrict__ d,
                                                      double* __restrict__ p1, double* __restrict__ p2,
                                                      double* __restrict__ redpart, int d_given, int store_d,
                                                      int defer_choice, GramRecords records, Scal* __restrict__ scal_next) {
    __shared__ double delta_s[kMaxV + 24];
    __shared__ double red[kWaves * kDirRed];
    __shared__ int flag;
    const int tid = threadIdx.x;
    const int64_t nchunks = (n + 2 * kBlock - 1) / (2 * kBlock);
    // the mask decides which lanes read the pair memory at all, so it (with x, g, l, u) is fetched one chunk ahead
    auto pair_index = [&](int64_t ch, bool& in) -> int64_t {
        const int64_t e = ch * (2 * kBlock) + 2 * tid;
        in = ch < nchunks && e < n;
        return in ? e : 0;
    };
    bool in_next;
    int64_t ec_next = pair_index(blockIdx.x, in_next);
    const bool ub_same = op.uniform_bounds != 0;                 // same bounds everywhere: l and u are not streamed
    dir_f64x2 xn = *reinterpret_cast<const dir_f64x2*>(x + ec_next), gn = *reinterpret_cast<const dir_f64x2*>(g + ec_next);
    dir_f64x2 ln = dir_f64x2{op.lo, op.lo}, un = dir_f64x2{op.hi, op.hi};
    if (!ub_same) { ln = *reinterpret_cast<const dir_f64x2*>(l + ec_next); un = *reinterpret_cast<const dir_f64x2*>(u + ec_next); }
    unsigned short mkn = *reinterpret_cast<const unsigned short*>(mask + ec_next);
    // the free bytes of a pair (an odd vector's last pair has one element)
    auto pair_mask = [&](bool in, int64_t e, unsigned short mk) -> unsigned short {
        return in ? (e + 1 < n ? mk : (unsigned short)(mk & 0xffu)) : (unsigned short)0;
    };
    int c, V;
    // 24 vectors per round: with m <= 11 every load of an element is in flight at once
    constexpr int kRound = 24;
    auto vec = [&](int j, int base_slot) -> const double* {      // (uniform: scalar registers)
        if (j >= 2 * c) return g;
        const int k = base_slot + (j < c ? j : j - c), slot = k < m ? k : k - m;
        return (j < c ? S : Y) + (int64_t)slot * n;
    };
    auto load = [&](int j0, int base_slot, int64_t e, dir_f64x2 (&v)[kRound]) {
#pragma unroll
        for (int k = 0; k < kRound; ++k) {
            v[k] = *reinterpret_cast<const dir_f64x2_any*>(vec(j0 + k, base_slot) + e);   // (past the last: g, its coefficient is zero)
        }
    };
    auto add = [&](int j0, const dir_f64x2 (&v)[kRound], double& q0, double& q1) {
#pragma unroll
        for (int k = 0; k < kRound; ++k) {
            q0 = fma(delta_s[j0 + k], v[k].x, q0);
            q1 = fma(delta_s[j0 + k], v[k].y, q1);
        }
    };
    int base_slot;
    dir_f64x2 first[CLOSE ? kRound : 1];
    if constexpr (CLOSE) {
        // the Gram kernel's closing step on a private copy of the scalar block, as in k_dir<true>; the first chunk's vectors
        // are requested before it and arrive under it
        __shared__ Scal sc;
        __shared__ double Gs[(2 * kGramOpenM + 2) * (2 * kGramOpenM + 2)];
        __shared__ double tot[gram_entries(kGramOpenM)];
        __shared__ double alpha_s[kMaxM + 1];
        static_assert(2 * kGramOpenM + 1 <= kRound, "one round holds every vector");
        constexpr int kScalWords = (int)(sizeof(Scal) / 4);
        for (int k = tid; k < kScalWords; k += kBlock)
            reinterpret_cast<int*>(&sc)[k] = reinterpret_cast<const int*>(scal)[k];
        int pa, pb;
        gram_product_slots(tid < gram_products(m) ? tid : 0, m, pa, pb);
        asm volatile("" : "+v"(pa), "+v"(pb));
        gram_sum_entries<kBlock>(records.part, gram_entries(m), records.count, tot);
        __syncthreads();
        if (sc.status != LBFGSB_RUNNING) {
            // (the kernel behind reads its status word from scal_next: it must not find an older one there)
            if (blockIdx.x == 0 && tid == 0) { scal_next->status = sc.status; scal_next->fresh = 0; note_progress(op, sc.status); }
            return;
        }
        int head = __builtin_amdgcn_readfirstlane(sc.head);
        c = __builtin_amdgcn_readfirstlane(sc.count);
        if (sc.pend_valid) {                                     // same rule as effective_ring()
            if (sc.pend_ok) { head = ring_next(head, m); c = c < m ? c + 1 : m; }
            else c = 0;
        }
        c = __builtin_amdgcn_readfirstlane(c);
        head = __builtin_amdgcn_readfirstlane(head);
        V = 2 * c + 1;
        base_slot = c > 0 ? ring_back(head, c, m) : 0;
        const double yn_old = prefetch_ynorm2(&sc, c, head, m);
        if (pair_mask(in_next, ec_next, mkn) != 0) load(0, base_slot, ec_next, first);
        __syncthreads();                                         // every thread has read the ring before it changes
        gram_finish<kBlock, kGramOpenM, false>(tot, Gs, alpha_s, &sc, m, c, head, base_slot, op, yn_old, 0, 1, blockIdx.x == 0, pa, pb);
        __syncthreads();                                         // the first wave's results are in the copy
        if (blockIdx.x == 0) {
            if (tid == 0) note_progress(op, sc.status);
            for (int k = tid; k < kScalWords; k += kBlock) {
                int v = reinterpret_cast<const int*>(&sc)[k];
                if (k == (int)(offsetof(Scal, fresh) / 4)) v = 1;
                reinterpret_cast<int*>(scal_next)[k] = v;
            }
        }
        if (sc.status != LBFGSB_RUNNING) return;
        if (tid < kMaxV + 24) delta_s[tid] = tid < V ? sc.delta[tid] : 0.0;
    } else {
        if (scal->status != LBFGSB_RUNNING) return;
        c = scal->count;
        V = 2 * c + 1;
        base_slot = c > 0 ? ring_back(scal->head, c, m) : 0;
        if (tid < kMaxV + 24) delta_s[tid] = tid < V ? scal->delta[tid] : 0.0;
    }
    __syncthreads();
    double s[6] = {0, 0, 0, 0, 0, 0};
    double ub = INFINITY;
    auto chunk = [&](int64_t ch, bool have_first) {
        const bool in = in_next;
        const int64_t ec = ec_next, e = ec_next;
        const dir_f64x2 xe = xn, ge = gn, le = ln, ue = un;
        const bool in2 = e + 1 < n;
        const unsigned short mk = pair_mask(in, e, mkn);
        ec_next = pair_index(ch + gridDim.x, in_next);
        xn = *reinterpret_cast<const dir_f64x2*>(x + ec_next); gn = *reinterpret_cast<const dir_f64x2*>(g + ec_next);
        if (!ub_same) { ln = *reinterpret_cast<const dir_f64x2*>(l + ec_next); un = *reinterpret_cast<const dir_f64x2*>(u + ec_next); }
        mkn = *reinterpret_cast<const unsigned short*>(mask + ec_next);
        dir_f64x2 de;
        if (d_given) {
            de = dir_f64x2{d[e], in2 ? d[e + 1] : 0.0};
        } else {
            double q0 = 0.0, q1 = 0.0;
            if (mk != 0) {                                       // lanes whose two elements are both fixed read nothing
                if (CLOSE && have_first) {
                    if constexpr (CLOSE) add(0, first, q0, q1);
                } else {
                    for (int j0 = 0; j0 < V; j0 += kRound) {
                        dir_f64x2 v[kRound];
                        load(j0, base_slot, ec, v);
                        add(j0, v, q0, q1);
                    }
                }
            }
            de.x = (mk & 0xffu) ? -q0 : 0.0;
            de.y = (mk >> 8) ? -q1 : 0.0;
            if (in && store_d) { d[e] = de.x; if (in2) d[e + 1] = de.y; }
        }
        if (in) {
            double a0, b0, a1, b1;
            dir_element(xe.x, ge.x, le.x, ue.x, de.x, op.eps, a0, b0, s, ub);
            if (in2) {
                dir_element(xe.y, ge.y, le.y, ue.y, de.y, op.eps, a1, b1, s, ub);
                *reinterpret_cast<dir_f64x2*>(p1 + e) = dir_f64x2{a0, a1};
                *reinterpret_cast<dir_f64x2*>(p2 + e) = dir_f64x2{b0, b1};
            } else {
                p1[e] = a0;
                p2[e] = b0;
            }
        }
    };
    int64_t ch = blockIdx.x;
    if (CLOSE && ch < nchunks) { chunk(ch, true); ch += gridDim.x; }
    for (; ch < nchunks; ch += gridDim.x) chunk(ch, false);
    double sx[2 * kFoldMax];
#pragma unroll
    for (int k = 0; k < 2 * kFoldMax; ++k) sx[k] = 0.0;
    dir_finish(s, ub, op.eps, scal, redpart, red, &flag, sx, FoldArgs{0, nullptr, nullptr, nullptr, nullptr}, defer_choice);
}

// one or two extra rows ride along with k_dir; k_dir_pairs has no room for them
bool dir_folds_extra_rows(const Dims& dm) {
    return dm.n_extra > 0 && dm.n_extra <= kFoldMax && !(dm.n >= (1 << 17) && dm.n % 2 == 0);
}

void launch_dir(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, int d_given, int store_d,
                hipStream_t st, const double* fold_rows, const double* fold_weight, int defer_choice, int open_gram) {
    FoldArgs fold{0, nullptr, nullptr, nullptr, nullptr};
    if (fold_rows && dir_folds_extra_rows(dm)) fold = FoldArgs{dm.n_extra, fold_rows, fold_weight, bf.wextra, bf.xres + dm.n_extra};
    const GramRecords records = open_gram ? gram_records(dm, ge, bf) : GramRecords{nullptr, 0};
    Scal* next = open_gram ? bf.scal_next : nullptr;
    if (dm.n >= (1 << 17) && !dir_folds_extra_rows(dm))
        hipLaunchKernelGGL(open_gram ? k_dir_pairs<true> : k_dir_pairs<false>, dim3(ge.dir_blocks), dim3(kBlock), 0, st, dm.n, dm.m,
                           op, bf.x, bf.g, bf.l, bf.u, bf.mask, bf.S, bf.Y, bf.scal, bf.d, bf.p1, bf.p2, bf.redpart, d_given,
                           store_d, defer_choice, records, next);
    else
        hipLaunchKernelGGL(open_gram ? k_dir<true> : k_dir<false>, dim3(ge.dir_blocks), dim3(kBlock), 0, st, dm.n, dm.m, op, bf.x,
                           bf.g, bf.l, bf.u, bf.mask, bf.S, bf.Y, bf.scal, bf.d, bf.p1, bf.p2, bf.redpart, d_given, store_d, fold,
                           defer_choice, records, next);
}

// ---- after an evaluation pass: g and f ------------------------------------------------------------------

// f needs x and the pass's loss partials, not the gradient.  Least squares: the first workgroup adds up the partials.  What the
// other kinds take beyond them (the regulariser, the linear term) is shared by the first kRegBlocks workgroups, the last of which
// to finish adds up.  (When every workgroup took a share and arrived, the arrivals at one address made the kernel 15.7 us at 10 000
// columns of a quadratic form and 32 at 20 000 of the L1-split kind; one workgroup for all of it: 53 there.  Now 6.0 and 10.4.)
constexpr int kRegBlocks = 64;
__global__ __launch_bounds__(kBlock) void k_eval_finish(Dims dm, int w_parts, int loss_parts,
                                                        const double* __restrict__ wpart,
                                                        const double* __restrict__ losspart,
                                                        const double* __restrict__ x, double* __restrict__ g,
                                                        Scal* __restrict__ scal, double* __restrict__ redpart,
                                                        const double* __restrict__ lin, const double* __restrict__ sign,
                                                        const double* __restrict__ wextra,
                                                        const double* __restrict__ xres, int reopen, int* __restrict__ host_flag,
                                                        const int* __restrict__ over) {
    __shared__ double lds[kBlock];
    __shared__ double red[kWaves];
    __shared__ int flag;
    if (reopen ? over && *over : scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    const bool shares = dm.kind != LBFGSB_OBJ_LSQ;
    const int nreg = shares ? ((int)gridDim.x < kRegBlocks ? (int)gridDim.x : kRegBlocks) : 1;
    const bool reg_wg = (int)blockIdx.x < nreg;
    double reg[1] = {0.0};
    if (reg_wg && shares) {
        for (int64_t i0 = (int64_t)blockIdx.x * kBlock + tid; i0 < dm.n; i0 += 4 * (int64_t)nreg * kBlock) {
            double xv[4], cv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t i = i0 + k * (int64_t)nreg * kBlock, ic = i < dm.n ? i : i0;
                xv[k] = x[ic];
                cv[k] = dm.kind == LBFGSB_OBJ_QP ? lin[ic] : (dm.kind == LBFGSB_OBJ_LOGISTIC_L2 ? xv[k] : 1.0);
                if (i >= dm.n) cv[k] = 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) reg[0] = fma(cv[k], xv[k], reg[0]);
        }
        block_sum<1, kWaves>(reg, red);
        if (tid == 0) publish(redpart + blockIdx.x, reg[0]);
    }
    for (int64_t c0 = (int64_t)blockIdx.x * kCX; c0 < dm.cols; c0 += (int64_t)gridDim.x * kCX) {
        const int64_t c = c0 + tid % kCX;
        const double w = column_sum(wpart, w_parts, dm.cols, c, lds);
        if (tid < kCX && c < dm.cols) {
            // wextra: the extra rows' contribution E^T (weight * residual), one entry per variable
            double gc;
            if (dm.kind == LBFGSB_OBJ_LSQ) {
                gc = w + (wextra ? wextra[c] : 0.0);
            } else if (dm.kind == LBFGSB_OBJ_LSQ_L1SPLIT) {
                gc = w + dm.lambda + (wextra ? wextra[c] : 0.0);
                const double gm = -w + dm.lambda + (wextra ? wextra[c + dm.cols] : 0.0);
                g[c + dm.cols] = gm;
                if (host_flag && !isfinite(gm)) host_flag[1] = 1;
            } else if (dm.kind == LBFGSB_OBJ_QP) {
                // w = (A (s.x))_c (a single "partial": the row kernel's output); g = s w + b
                gc = (sign ? sign[c] : 1.0) * w + lin[c] + (wextra ? wextra[c] : 0.0);
            } else {
                gc = fma(dm.mu, x[c], w);
            }
            g[c] = gc;
            if (host_flag && !isfinite(gc)) host_flag[1] = 1;
        }
    }
    if (!reg_wg || (shares && !arrive_is_last(&scal->counters[kCntEvalFinish], &flag, (unsigned)nreg))) return;
    const double loss = sum_all(losspart, loss_parts, red);
    if (shares) {
        reg[0] = tid < nreg ? observe(redpart + tid) : 0.0;
        block_sum<1, kWaves>(reg, red);
    }
    if (tid == 0) {
        double f = loss;
        if (dm.kind == LBFGSB_OBJ_LSQ_L1SPLIT) f += dm.lambda * reg[0];
        else if (dm.kind == LBFGSB_OBJ_LOGISTIC_L2) f += 0.5 * dm.mu * reg[0];
        else if (dm.kind == LBFGSB_OBJ_QP) f += reg[0];
        if (xres) f += xres[dm.n_extra];   // 0.5 sum weight * residual^2 of the extra rows
        if (reopen) {
            apply_pending(scal, dm.m);
            if (scal->status == LBFGSB_CONVERGED) scal->status = LBFGSB_RUNNING;
        }
        scal->f = f;
        scal->fevals += 1;
        scal->gram_left = 0;
    }
}

void launch_eval_finish(const Dims& dm, const Geometry& ge, const Buffers& bf, const double* lin, const double* sign,
                        hipStream_t st, bool reopen, int* host_flag, const int* over) {
    const bool qp = dm.kind == LBFGSB_OBJ_QP;
    hipLaunchKernelGGL(k_eval_finish, dim3(ge.fin_blocks), dim3(kBlock), 0, st, dm, qp ? 1 : ge.w_parts, ge.loss_parts,
                       qp ? (const double*)bf.row : (const double*)bf.wpart, bf.losspart, bf.x, bf.g, bf.scal, bf.redpart,
                       lin, sign, dm.n_extra > 0 ? (const double*)bf.wextra : nullptr,
                       dm.n_extra > 0 ? (const double*)bf.xres : nullptr, reopen ? 1 : 0, host_flag, over);
}

// ---- quadratic objectives: closed-form Armijo search, then the update ---------------------------------------
//
// With t = A v_p and w = A^T t from the direction pass:  f(x + a p) - f(x) = a <g,p> + a^2/2 ||t||^2,
// gradient g + a w~ (w~ = w, or [w; -w] for the split form), y = a w~.  The residual is not carried
// along: nothing in the iteration reads it, and an evaluation from x recomputes it.
// The Armijo inequality  a gp + a^2/2 tt <= c1 a gp  is tested after division by a > 0.
__global__ __launch_bounds__(kBlock) void k_update_quadratic(Dims dm, Opts op, int w_parts, int loss_parts,
                                                             const double* __restrict__ wpart,
                                                             const double* __restrict__ losspart,
                                                             const double* __restrict__ p1,
                                                             const double* __restrict__ p2,
                                                             const double* __restrict__ l, const double* __restrict__ u,
                                                             double* __restrict__ x, double* __restrict__ g,
                                                             double* __restrict__ S, double* __restrict__ Y,
                                                             Scal* __restrict__ scal, const double* __restrict__ sign,
                                                             const double* __restrict__ wextra,
                                                             const double* __restrict__ xres, int n_fold,
                                                             const double* __restrict__ fold_rows,
                                                             const double* __restrict__ fold_weight,
                                                             const double* __restrict__ dir_part, int dir_blocks) {
    __shared__ double lds[kBlock];
    __shared__ double red[kWaves];
    __shared__ double ls_alpha;
    __shared__ int ls_ok, ls_bt;
    __shared__ double fold_s[kFoldMax + 1];   // folded rows: coefficients weight_r (e_r . p), then sum weight_r (e_r . p)^2
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    const double gp = scal->gp, alpha_ub = scal->alpha_ub, f_old = scal->f;
    const int slot = scal->head;
    const int branch = scal->branch;
    const double* p = branch == 1 ? p1 : p2;
    const bool own_fold = n_fold > 0 && dir_blocks > 0;
    if (own_fold) {
        // the direction kernel left only its per-workgroup sums: the first wave adds the folded rows' products with
        // the chosen candidate (every workgroup the same bits)
        if (tid < 64) {
            double tx[2 * kFoldMax];
            dir_fold_from_partials(dir_part, dir_blocks, tx);
            if (tid == 0) fold_s[kFoldMax] = fold_coefficients(tx, branch, n_fold, fold_weight, fold_s);
        }
        __syncthreads();
    }
    // curvature along p: ||t||^2 (weighted) from the A pass, plus the extra rows' sum weight (e_r.p)^2
    const double tt = sum_all(losspart, loss_parts, red) + (own_fold ? fold_s[kFoldMax] : (xres ? xres[dm.n_extra] : 0.0));
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
        for (int64_t c0 = (int64_t)blockIdx.x * kCX; c0 < dm.cols; c0 += (int64_t)gridDim.x * kCX) {
            const int64_t c = c0 + tid % kCX;
            const double w = column_sum(wpart, w_parts, dm.cols, c, lds);
            if (tid < kCX && c < dm.cols) {
                const int nvar = dm.kind == LBFGSB_OBJ_LSQ_L1SPLIT ? 2 : 1;
                for (int h = 0; h < nvar; ++h) {
                    const int64_t i = c + h * dm.cols;
                    double wi = h ? -w : w;
                    if (sign) wi *= sign[i];               // QP: the change of the gradient is s.(A (s.p))
                    if (n_fold > 0) {                       // folded extra rows: wextra[0 .. n_fold) holds their coefficients
                        for (int r = 0; r < n_fold; ++r) wi = fma(own_fold ? fold_s[r] : wextra[r], fold_rows[(int64_t)r * dm.n + i], wi);
                    } else if (wextra) {
                        wi += wextra[i];
                    }
                    const double y = alpha * wi;
                    const double xi = x[i];
                    const double xn = clampd(fma(alpha, p[i], xi), l[i], u[i]);
                    Sn[i] = xn - xi;
                    Yn[i] = y;
                    x[i] = xn;
                    g[i] += y;
                }
            }
        }
    }
    // No workgroup of this kernel reads the pend_* fields, so one thread may write them while others
    // are still running; the next Gram kernel (or k_commit) turns them into head/count/iters/f.
    if (blockIdx.x == 0 && tid == 0) {
        scal->pend_ok = ok;
        scal->pend_bt = ls_bt;
        scal->pend_alpha = alpha;
        scal->pend_f = f_old + alpha * (gp + 0.5 * alpha * tt);
        scal->pend_valid = 1;
    }
}

void launch_update_quadratic(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const double* sign,
                             hipStream_t st, const double* fold_rows, const double* fold_weight, int dir_blocks) {
    const int n_fold = fold_rows && dir_folds_extra_rows(dm) ? dm.n_extra : 0;
    const bool qp = dm.kind == LBFGSB_OBJ_QP;   // its "partial columns" are the single vector t = A (s.p)
    hipLaunchKernelGGL(k_update_quadratic, dim3(ge.upd_blocks), dim3(kBlock), 0, st, dm, op, qp ? 1 : ge.w_parts,
                       ge.loss_parts, qp ? (const double*)bf.t : (const double*)bf.wpart, bf.losspart, bf.p1, bf.p2, bf.l,
                       bf.u, bf.x, bf.g, bf.S, bf.Y, bf.scal, qp ? sign : nullptr,
                       dm.n_extra > 0 ? (const double*)bf.wextra : nullptr,
                       dm.n_extra > 0 ? (const double*)bf.xres : nullptr, n_fold, fold_rows, fold_weight,
                       (const double*)bf.redpart, n_fold > 0 ? dir_blocks : 0);
}

// ---- extra dense rows ------------------------------------------------------------------------------------
//
// One workgroup.  z = x (eval) or the direction Algorithm 2 selected.  te_r = e_r . z; coefficient
// c_r = weight_r (te_r - target_r) (eval) or weight_r te_r (direction);
//   wextra[i] = sum_r c_r E[r][i],   xres[r] = te_r - target_r (eval only),
//   xres[n_extra] = 0.5 sum weight_r (te_r - target_r)^2 (eval)  or  sum weight_r te_r^2 (direction).
__global__ __launch_bounds__(kBlock) void k_extra_rows(Dims dm, const double* __restrict__ E,
                                                       const double* __restrict__ target,
                                                       const double* __restrict__ weight, int eval,
                                                       const double* __restrict__ x, const double* __restrict__ p1,
                                                       const double* __restrict__ p2, const Scal* __restrict__ scal,
                                                       double* __restrict__ wextra, double* __restrict__ xres) {
    __shared__ double red[kWaves];
    __shared__ double coef[kMaxExtra];
    if (eval != 1 && scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    const double* z = eval ? x : (scal->branch == 1 ? p1 : p2);
    double total = 0.0;
    for (int r = 0; r < dm.n_extra; ++r) {
        double s[1] = {0.0};
        const double* er = E + (int64_t)r * dm.n;
        for (int64_t i0 = tid; i0 < dm.n; i0 += kBlock * 8) {   // 16 loads in flight per thread: the kernel is latency-bound
            double ev[8], zv[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int64_t i = i0 + (int64_t)k * kBlock;
                ev[k] = i < dm.n ? er[i] : 0.0;
                zv[k] = i < dm.n ? z[i] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) s[0] = fma(ev[k], zv[k], s[0]);
        }
        block_sum<1, kWaves>(s, red);
        const double wr = weight ? weight[r] : 1.0;
        const double res = eval ? s[0] - target[r] : s[0];
        total += (eval ? 0.5 : 1.0) * wr * res * res;
        if (tid == 0) {
            coef[r] = wr * res;
            if (eval) xres[r] = res;
        }
    }
    __syncthreads();
    for (int64_t i0 = tid; i0 < dm.n; i0 += kBlock * 8) {
        double acc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = 0.0;
        for (int r = 0; r < dm.n_extra; ++r) {
            double ev[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int64_t i = i0 + (int64_t)k * kBlock;
                ev[k] = i < dm.n ? E[(int64_t)r * dm.n + i] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] = fma(coef[r], ev[k], acc[k]);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = i0 + (int64_t)k * kBlock;
            if (i < dm.n) wextra[i] = acc[k];
        }
    }
    if (tid == 0) xres[dm.n_extra] = total;
}

void launch_extra_rows(const Dims& dm, const Buffers& bf, const double* rows, const double* target, const double* weight,
                       int eval, hipStream_t st) {
    hipLaunchKernelGGL(k_extra_rows, dim3(1), dim3(kBlock), 0, st, dm, rows, target, weight, eval, bf.x, bf.p1, bf.p2,
                       (const Scal*)bf.scal, bf.wextra, bf.xres);
}

// ---- logistic objective: line search on the margins --------------------------------------------------------
//
// With z = X w (kept in `row`) and t = X p:  f(x + a p) - f(x) = (1/N) sum_r [softplus(-y_r (z_r + a t_r))
// - softplus(-y_r z_r)] + mu (a <x,p> + a^2/2 <p,p>).  The bracket is evaluated in the cancellation-free
// form log(1 + sigmoid(q) expm1(dq)), q = -y z, dq = -y a t (softplus_diff).  Step lengths are evaluated NTRY at a time per sweep
// over the rows: the first launch tries the first one alone (it is accepted in almost every quasi-Newton
// iteration; where the pass over X has formed that sum itself -- first_parts > 0 loss partials -- there is no such launch: the
// short launch sequence has the update kernel decide, see k_update_logistic, the full one this kernel, every workgroup for
// itself), a second launch, which returns at once when the first found the step, tries the next kLsBatch, and
// if none of them is acceptable its last workgroup goes on alone, one length at a time.

// Change of f at the first trial step a, from the loss differences the pass over X has summed (every workgroup the same bits).
// seed: what each thread's sum begins with.
__device__ __forceinline__ double first_step_difference(const Dims& dm, const Scal* scal, const double* __restrict__ losspart,
                                                        int parts, double a, double* lds, double seed = 0.0) {
    const double xp = scal->xp, pp = scal->pp;
    return sum_all(losspart, parts, lds, seed) / (double)dm.rows + dm.mu * a * (xp + 0.5 * a * pp);
}

template <int NTRY>
__global__ __launch_bounds__(kBlock) void k_ls_logistic(Dims dm, Opts op, int first, int last_resort, int spec, int first_parts,
                                                        const double* __restrict__ losspart,
                                                        const double* __restrict__ yl, const double* __restrict__ z,
                                                        const double* __restrict__ t, Scal* __restrict__ scal,
                                                        double* __restrict__ lspart) {
    __shared__ double red[kWaves * NTRY];
    __shared__ int flag;
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x;
    if (first_parts > 0) {
        const double a = fmin(1.0, scal->alpha_ub);
        const double df = first_step_difference(dm, scal, losspart, first_parts, a, red);
        if (isfinite(df) && df <= op.c1 * a * scal->gp) {
            // (the update kernel leaves this step pending, and the trial is counted when that is applied)
            if (blockIdx.x == 0 && tid == 0) {
                scal->ls_ok = 1;
                scal->spec_ok = 1;
                scal->backtracks = 0;
                scal->alpha = a;
            }
            return;
        }
    } else if (first > 0 && scal->ls_ok) {
        return;                                      // an earlier launch of this iteration found the step
    }
    double al[NTRY], s[NTRY];
    {
        double a = fmin(1.0, scal->alpha_ub);
        for (int k = 0; k < first; ++k) a *= op.backtrack;
#pragma unroll
        for (int j = 0; j < NTRY; ++j) { al[j] = a; s[j] = 0.0; a *= op.backtrack; }
    }
    // four rows per trip: the transcendental chains of different rows are independent, and the few waves of this
    // kernel are latency-bound, so interleaving them is what shortens it
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t r0 = (int64_t)blockIdx.x * kBlock + tid; r0 < dm.rows; r0 += 4 * stride) {
        double q[4], sq[4], ty[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t r = r0 + k * stride;
            const bool in = r < dm.rows;
            const double y = in ? yl[r] : 0.0;          // y = 0: q = ty = 0, the row contributes log1p(0.5 * expm1(0)) = 0
            q[k] = -y * (in ? z[r] : 0.0);
            ty[k] = -y * (in ? t[r] : 0.0);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) sq[k] = sigmoid_d(q[k]);
#pragma unroll
        for (int j = 0; j < NTRY; ++j) {
#pragma unroll
            for (int k = 0; k < 4; ++k) s[j] += softplus_diff(q[k], sq[k], al[j] * ty[k]);
        }
    }
    block_sum<NTRY, kWaves>(s, red);
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < NTRY; ++j) publish(lspart + (int64_t)blockIdx.x * NTRY + j, s[j]);
    }
    if (!arrive_is_last(&scal->counters[kCntLs], &flag)) return;
    const double gp = scal->gp, xp = scal->xp, pp = scal->pp;
    const double invn = 1.0 / (double)dm.rows;
    // totals of the batch
    double tot[NTRY];
#pragma unroll
    for (int j = 0; j < NTRY; ++j) tot[j] = 0.0;
    for (int b = tid; b < (int)gridDim.x; b += kBlock) {
#pragma unroll
        for (int j = 0; j < NTRY; ++j) tot[j] += observe(lspart + (int64_t)b * NTRY + j);
    }
    block_sum<NTRY, kWaves>(tot, red);
    int found = -1;
    double a_acc = 0.0;
#pragma unroll
    for (int j = 0; j < NTRY; ++j) {
        const double df = tot[j] * invn + dm.mu * al[j] * (xp + 0.5 * al[j] * pp);
        if (found < 0 && first + j <= op.max_backtracks && isfinite(df) && df <= op.c1 * al[j] * gp) { found = first + j; a_acc = al[j]; }
    }
    // rare: continue one step length at a time (uniform control flow: every thread holds the same totals)
    double a = al[NTRY - 1];
    for (int k = first + NTRY; last_resort && found < 0 && k <= op.max_backtracks; ++k) {
        a *= op.backtrack;
        double sv[1] = {0.0};
        for (int64_t r = tid; r < dm.rows; r += kBlock) {
            const double y = yl[r], q = -y * z[r];
            sv[0] += softplus_diff(q, sigmoid_d(q), -y * a * t[r]);
        }
        block_sum<1, kWaves>(sv, red);
        const double df = sv[0] * invn + dm.mu * a * (xp + 0.5 * a * pp);
        if (isfinite(df) && df <= op.c1 * a * gp) { found = k; a_acc = a; }
    }
    if (tid == 0) {
        scal->ls_ok = found >= 0;
        if (first == 0 || first_parts > 0) scal->spec_ok = spec && found == 0;
        if (found >= 0 || last_resort) {
            scal->backtracks = found >= 0 ? found : op.max_backtracks + 1;
            scal->fevals += found >= 0 ? found + 1 : op.max_backtracks + 1;
        }
        if (found >= 0) scal->alpha = a_acc;
    }
}

void launch_ls_logistic(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const double* labels,
                        int spec, int stages, int first_parts, hipStream_t st) {
    if (stages & 1)
        hipLaunchKernelGGL(k_ls_logistic<1>, dim3(ge.ls_blocks), dim3(kBlock), 0, st, dm, op, 0, 0, spec, 0, (const double*)bf.losspart,
                           labels, (const double*)bf.row, (const double*)bf.t, bf.scal, bf.lspart);
    if (stages & 2)
        hipLaunchKernelGGL(k_ls_logistic<kLsBatch>, dim3(ge.ls_blocks), dim3(kBlock), 0, st, dm, op, 1, 1, spec, first_parts,
                           (const double*)bf.losspart, labels, (const double*)bf.row, (const double*)bf.t, bf.scal, bf.lspart);
}

// z += alpha t; psi = -y sigma(-y z)/N; loss partials of the new point (from the new margins).
// not_first: the update kernel does what is left of this when the first trial step was accepted.
__global__ __launch_bounds__(kBlock) void k_rows_logistic(Dims dm, int not_first, const double* __restrict__ yl,
                                                          const double* __restrict__ t, double* __restrict__ z,
                                                          double* __restrict__ psi, const Scal* __restrict__ scal,
                                                          double* __restrict__ losspart) {
    __shared__ double red[kWaves];
    if (scal->status != LBFGSB_RUNNING || !scal->ls_ok || (not_first && scal->spec_ok)) return;
    const double alpha = scal->alpha;
    const double invn = 1.0 / (double)dm.rows;
    double s[1] = {0.0};
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < dm.rows; r += (int64_t)gridDim.x * kBlock) {
        const double y = yl[r];
        const double zn = fma(alpha, t[r], z[r]);
        const double q = -y * zn;
        z[r] = zn;
        psi[r] = -y * sigmoid_d(q) * invn;
        s[0] += softplus_d(q) * invn;
    }
    block_sum<1, kWaves>(s, red);
    if (threadIdx.x == 0) losspart[blockIdx.x] = s[0];
}

void launch_rows_logistic(const Dims& dm, const Geometry& ge, const Buffers& bf, const double* labels, int not_first,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_rows_logistic, dim3(ge.lrows_blocks), dim3(kBlock), 0, st, dm, not_first, labels, bf.t, bf.row, bf.psi, bf.scal,
                       bf.losspart);
}

// x+ = P(x + alpha p), g+ = X^T psi + mu x+, pair (x+ - x, g+ - g), f+ from the new margins.
// short_seq: the pass over X has left, in its loss partials, the sums over its workgroups' rows of
// softplus(-y (z + a0 t)) - softplus(-y z) for the first trial step a0 = min(1, alpha_ub).  Every workgroup adds
// them in the same order and takes the same Armijo decision; an accepted step is applied here (the margins move
// too), a rejected one parks the solver (kStatusBail) with nothing changed and no arrival counted.
// first_parts > 0 without short_seq: the search kernel has decided from those partials; what it accepted of them is applied
// the same way, with the loss from the same sum, any other step from the recomputed margins.
__global__ __launch_bounds__(kBlock) void k_update_logistic(Dims dm, double c1, int w_parts_two_pass, int w_parts_spec,
                                                            int loss_parts, int first_parts, int short_seq,
                                                            const double* __restrict__ t, double* __restrict__ z, const double* __restrict__ wpart,
                                                            const double* __restrict__ losspart,
                                                            const double* __restrict__ p1, const double* __restrict__ p2,
                                                            const double* __restrict__ l, const double* __restrict__ u,
                                                            double* __restrict__ x, double* __restrict__ g,
                                                            double* __restrict__ S, double* __restrict__ Y,
                                                            Scal* __restrict__ scal, double* __restrict__ redpart) {
    __shared__ double lds[kBlock];
    __shared__ double red[kWaves * 2];
    __shared__ int flag;
    // Short sequence: workgroup 0 may park the solver while another is beginning, whose waves, each with a load of its own, then do
    // not all see the same.  Such a workgroup stays together: a wave that finds the solver stopped makes its sum, and with it every
    // wave's, no number, which is no acceptable step.  (Whole calls, 200000 x 2000: 4074 us before, 4080 so, 4087 with a vote of the workgroup.)
    const bool running = scal->status == LBFGSB_RUNNING;
    if (!running && !(short_seq && blockIdx.x > 0)) return;
    const int tid = threadIdx.x;
    int ok = scal->ls_ok;
    double alpha = scal->alpha;
    const int slot = scal->head;
    const double* p = scal->branch == 1 ? p1 : p2;
    int w_parts = scal->spec_ok ? w_parts_spec : w_parts_two_pass;   // which kernel wrote the partial columns
    double df = 0.0, f_old = 0.0;
    const bool first_step = short_seq || (first_parts > 0 && ok && scal->spec_ok);
    if (first_step) {
        f_old = scal->f;
        alpha = fmin(1.0, scal->alpha_ub);
        df = first_step_difference(dm, scal, losspart, first_parts, alpha, red, running ? 0.0 : NAN);
        ok = !short_seq || (isfinite(df) && df <= c1 * alpha * scal->gp);
        w_parts = w_parts_spec;
        if (!ok) {
            // (a workgroup of which any wave starts after this store changes nothing either)
            if (blockIdx.x == 0 && tid == 0) {
                scal->ls_ok = 0;
                scal->spec_ok = 0;
                scal->status = kStatusBail;
            }
            return;
        }
    }
    double sums[2] = {0.0, 0.0};   // ||y||^2, ||x+||^2
    // first trial step: the first `col_blocks` workgroups take the columns, the others the margins (side by side, not
    // one after the other: a workgroup's trips to memory are dependent and nothing else runs on its compute unit);
    // a grid of one workgroup does both
    int col_first = 0, col_stride = (int)gridDim.x;
    if (ok && first_step) {
        // the margins of the new point (for any other step a kernel before this one, which also recomputes the row weights:
        // the single-read pass already holds X^T psi of this step)
        const int want = (int)((dm.cols + kCX - 1) / kCX);
        const int col_blocks = want < (int)gridDim.x / 2 ? want : (int)gridDim.x / 2;
        int rb = (int)blockIdx.x, nrb = (int)gridDim.x;
        if (col_blocks > 0) {
            col_stride = col_blocks;
            if ((int)blockIdx.x >= col_blocks) col_first = -1;   // this workgroup takes no columns
            rb = (int)blockIdx.x - col_blocks;                   // (negative: no rows)
            nrb = (int)gridDim.x - col_blocks;
        }
        if (rb >= 0) {
            // (four rows per trip with their loads issued together)
            const int64_t stride = (int64_t)nrb * kBlock;
            for (int64_t r0 = (int64_t)rb * kBlock + tid; r0 < dm.rows; r0 += 4 * stride) {
                double tv[4], zv[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t r = r0 + k * stride;
                    tv[k] = r < dm.rows ? t[r] : 0.0;
                    zv[k] = r < dm.rows ? z[r] : 0.0;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t r = r0 + k * stride;
                    if (r < dm.rows) z[r] = fma(alpha, tv[k], zv[k]);
                }
            }
        }
    }
    if (ok && col_first >= 0) {
        double* Sn = S + (int64_t)slot * dm.n;
        double* Yn = Y + (int64_t)slot * dm.n;
        for (int64_t c0 = (int64_t)blockIdx.x * kCX; c0 < dm.cols; c0 += (int64_t)col_stride * kCX) {
            const int64_t c = c0 + tid % kCX;
            const double w = column_sum(wpart, w_parts, dm.cols, c, lds);
            if (tid < kCX && c < dm.cols) {
                const double xi = x[c];
                const double xn = clampd(fma(alpha, p[c], xi), l[c], u[c]);
                const double gn = fma(dm.mu, xn, w);
                const double y = gn - g[c];
                Sn[c] = xn - xi;
                Yn[c] = y;
                x[c] = xn;
                g[c] = gn;
                sums[0] = fma(y, y, sums[0]);
                sums[1] = fma(xn, xn, sums[1]);
            }
        }
    }
    if (first_step) {
        // Nothing is left to add up: f moves by the line search's difference, and the new pair's ||y||^2 comes from
        // the next free-set pass (as for the quadratic kinds).  No workgroup of this kernel reads the pend_* fields,
        // so one thread may write them while others are still running; the next Gram kernel (or k_commit) turns
        // them into head/count/iters/f.  Without an arrival at one address the grid need not stay small.
        if (blockIdx.x == 0 && tid == 0) {
            scal->spec_ok = 1;
            scal->pend_ok = 1;
            scal->pend_bt = 0;
            scal->pend_alpha = alpha;
            scal->pend_f = f_old + df;
            scal->pend_valid = 1;
        }
        return;
    }
    block_sum<2, kWaves>(sums, red);
    if (tid == 0) { publish(redpart + 2 * blockIdx.x, sums[0]); publish(redpart + 2 * blockIdx.x + 1, sums[1]); }
    if (!arrive_is_last(&scal->counters[kCntUpdate], &flag)) return;
    double tot[2] = {0.0, 0.0};
    for (int b = tid; b < (int)gridDim.x; b += kBlock) { tot[0] += observe(redpart + 2 * b); tot[1] += observe(redpart + 2 * b + 1); }
    block_sum<2, kWaves>(tot, red);
    const double loss = ok ? sum_all(losspart, loss_parts, red) : 0.0;
    if (tid == 0) {
        if (ok) {
            // f from the new margins and the new iterate
            scal->f = loss + 0.5 * dm.mu * tot[1];
            scal->ynorm2[slot] = tot[0];
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

void launch_update_logistic(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, int first_parts,
                            int short_seq, hipStream_t st) {
    hipLaunchKernelGGL(k_update_logistic, dim3(first_parts > 0 ? ge.updl_blocks : ge.upd_blocks), dim3(kBlock), 0, st, dm, op.c1,
                       ge.redo_parts, ge.fused_blocks, ge.lrows_blocks, first_parts, short_seq, (const double*)bf.t, bf.row, bf.wpart,
                       bf.losspart, bf.p1, bf.p2, bf.l, bf.u, bf.x, bf.g, bf.S, bf.Y, bf.scal, bf.redpart);
}

}  // namespace lb
