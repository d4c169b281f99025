// Short vectors: free set (Eq. (ws)), masked Gram matrix, Algorithm 3 on coefficients, direction and Algorithm 2's choice
// in ONE workgroup and one launch.
//
// With a few hundred variables the Gram kernel and the direction kernel move 20-150 KB between them and are nothing but
// latency: launches, dependent trips to memory, sums over workgroups.  One workgroup does their work on one compute unit
// in ONE trip: the scalar block, x, g, the bounds and every slot of the pair memory are requested together (which slots
// hold pairs is looked at afterwards).  Thread e owns elements e and e + 512 from the free-set test to the direction and
// keeps all their vectors' entries in registers; masked copies go to LDS, from where the matrix cores take the products
// (v_mfma_f64_16x16x4, lane (i, q) supplies vector i of a block of 16 at one element, as in the Gram kernel).  The vectors are
// ordered y | g | s, so that the blocks of products the recursion does not read -- s with s -- are left out.  The
// recursion runs on an LDS copy of the scalar block, which goes back to memory once, with Algorithm 2's choice in it.
//
// Measured (least squares, iterations of a problem with 1.5 n + 260 rows, us per iteration, Gram + direction kernels /
// this kernel): m = 5: n = 100 26.9 / 18.5, 301 32.4 / 20.4, 1024 32.4 / 26.5; m = 10: 100 28.5 / 20.9, 512 32.4 / 25.3, 832 32.8 / 30.2
// (1000: 33.4 / 33.3, left to the two kernels); m = 20: 100 38.8 / 27.6, 384 41.4 / 32.1.  That was with a branch per slot in the
// statistics and the direction (130 cycles each), 64 elements per wave and turn at the matrix cores and three exchanges between
// the waves where two do; without them 50 steps take 1221 -> 1098 us at n = 301 and 1853 -> 1670 at 801 (m = 10), 1024 -> 902 at 101
// (m = 5), 1723 -> 1533 at 350 (m = 20).
#include <cstddef>

#include "common.h"
#include "recursion.h"

namespace lb {

namespace {

constexpr int kSmallNT = 512, kSmallNW = kSmallNT / 64;
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int small_blocks(int M) { return (2 * M + 1 + 15) / 16; }             // blocks of 16 vectors
// pairs of blocks (a <= b) computed: not the last with itself when it holds s vectors only
constexpr int small_pairs(int M) {
    const int nb = small_blocks(M);
    return nb * (nb + 1) / 2 - (16 * (nb - 1) > M ? 1 : 0);
}
// doubles between two vectors in LDS: even, and an odd multiple of two, so that 16 lanes that read 16 bytes each of 16
// vectors touch every bank once
constexpr int small_stride(int64_t n) { return (int)((n + 15) / 16 * 16 + 2); }
constexpr size_t small_lds_bytes(int M, int64_t n) {
    const size_t vec = (size_t)(2 * M + 1) * small_stride(n), part = (size_t)kSmallNW * small_pairs(M) * 256;
    return (vec > part ? vec : part) * 8;
}

}  // namespace

// M: slots of the pair memory (m <= M); R: rounds of 512 elements that cover n.
template <int M, int R>
__global__ __launch_bounds__(kSmallNT) void k_small_step(Dims dm, Opts op, const double* __restrict__ x,
                                                         const double* __restrict__ g, const double* __restrict__ l,
                                                         const double* __restrict__ u, const double* __restrict__ S,
                                                         const double* __restrict__ Y, uint8_t* __restrict__ mask,
                                                         Scal* __restrict__ scal, double* __restrict__ p1,
                                                         double* __restrict__ p2, int n_fold,
                                                         const double* __restrict__ fold_rows,
                                                         const double* __restrict__ fold_weight,
                                                         double* __restrict__ fold_coef, double* __restrict__ fold_total) {
    constexpr int V0 = 2 * M + 1;                   // static slots: y ring 0..M-1 | g M | s ring M+1..2M
    constexpr int NB = small_blocks(M), NP = small_pairs(M);
    constexpr int GD = 2 * M + 2;
    extern __shared__ __align__(16) double dyn[];   // masked vectors, later the waves' blocks
    __shared__ double G[GD * GD];
    __shared__ Scal sc;
    __shared__ double red[kSmallNW * 8];
    __shared__ double redx[kSmallNW * 2 * kFoldMax];
    __shared__ double alpha_s[kMaxM + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)dm.n, m = dm.m;
    const int ls = small_stride(n);
    double xe[R], ge[R], le[R], ue[R], vy[R][M], vs[R][M];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = tid + r * kSmallNT, ec = e < n ? e : n - 1;
        xe[r] = x[ec]; ge[r] = g[ec]; le[r] = l[ec]; ue[r] = u[ec];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const int slot = k < m ? k : m - 1;     // (slots past m: never used, any valid address)
            vy[r][k] = Y[(int64_t)slot * n + ec];
            vs[r][k] = S[(int64_t)slot * n + ec];
        }
    }
    constexpr int kScalWords = (int)(sizeof(Scal) / 4);
    for (int k = tid; k < kScalWords; k += kSmallNT)
        reinterpret_cast<int*>(&sc)[k] = reinterpret_cast<const int*>(scal)[k];
    __syncthreads();
    if (sc.status != LBFGSB_RUNNING) {
        // a step that finds the solver parked by the short logistic sequence is counted, so that the host can redo it
        if (tid == 0) {
            if (sc.status == kStatusBail) scal->bail_skipped = sc.bail_skipped + 1;
            note_progress(op, sc.status);
        }
        return;
    }
    int head, c;
    bool ls_dead;
    effective_ring(&sc, m, head, c, ls_dead);
    const double yn_old = prefetch_ynorm2(&sc, c, head, m);
    const int V = 2 * c + 1, Vp = V + 1;
    const int base_slot = c > 0 ? ring_back(head, c, m) : 0;   // ring slot of the oldest pair
    const int newest = c > 0 ? ring_back(head, 1, m) : -1;
    // static slot -> place in the recursion's order s^0..s^{c-1}, y^0..y^{c-1}, g (oldest first), -1: holds no pair
    auto logical = [&](int slot) -> int {
        if (slot == M) return 2 * c;
        const int ring = slot < M ? slot : slot - M - 1;
        const int k = ring >= base_slot ? ring - base_slot : ring - base_slot + m;
        return ring >= m || slot >= V0 || k >= c ? -1 : (slot < M ? c + k : k);
    };
    double ysum = 0.0, pginf = 0.0;                  // ||y_new||^2 over the full vector, KKT residual
    int nfix = 0;                                    // #fixed, of this wave
    unsigned freebits = 0;                           // bit r: this thread's element of round r is free
    // (what a slot that holds no pair contains is not looked at)
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const bool holds = logical(k) >= 0;          // (uniform)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            vy[r][k] = holds ? vy[r][k] : 0.0;
            vs[r][k] = holds ? vs[r][k] : 0.0;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = tid + r * kSmallNT;
        const bool in = e < n;
        const bool fr = in && !fixed_at(xe[r], ge[r], le[r], ue[r], op.eps);
        double yn = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) yn = k == newest ? vy[r][k] : yn;
        ysum = in ? fma(yn, yn, ysum) : ysum;
        pginf = in ? fmax(pginf, fabs(xe[r] - clampd(xe[r] - ge[r], le[r], ue[r]))) : pginf;
        freebits |= fr ? 1u << r : 0u;
        nfix += __popcll(__ballot(in && !fr));
        if (in) mask[e] = (uint8_t)fr;
        if (e < ls - 2) {                            // (zeros from n to the end of the last chunk of 16)
            dyn[M * ls + e] = fr ? ge[r] : 0.0;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                dyn[k * ls + e] = fr ? vy[r][k] : 0.0;
                dyn[(M + 1 + k) * ls + e] = fr ? vs[r][k] : 0.0;
            }
        }
    }
    ysum = wave_sum(ysum);
    pginf = wave_max(pginf);
    if (lane == 0) { red[wave] = pginf; red[kSmallNW + wave] = ysum; red[2 * kSmallNW + wave] = (double)nfix; }
    __syncthreads();                                 // (publishes dyn and the waves' statistics)
    if (tid == kSmallNT - 1) apply_pending(&sc, m);  // (every thread has read the ring position out of the copy)

    f64x4 acc[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) acc[k] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int i16 = lane & 15, q = lane >> 4;
    // 16 elements -- four steps of 4 -- per wave and turn, so that the matrix cores of all four SIMDs are busy (a step of one
    // block takes 64 cycles, and at a few hundred elements these are what the phase lasts)
    for (int e0 = 16 * wave; e0 < n; e0 += 16 * kSmallNW) {
        double2 v[NB][2];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = 16 * b + i16;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v[b][h] = *reinterpret_cast<const double2*>(&dyn[(j < V0 ? j : 0) * ls + e0 + 8 * h + 2 * q]);
                if (j >= V0) v[b][h] = double2{0.0, 0.0};
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            int k = 0;
#pragma unroll
            for (int a = 0; a < NB; ++a) {
#pragma unroll
                for (int b = a; b < NB; ++b, ++k)
                    if (k < NP) acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(t & 1 ? v[a][t / 2].y : v[a][t / 2].x, t & 1 ? v[b][t / 2].y : v[b][t / 2].x, acc[k], 0, 0, 0);
            }
        }
    }
    double ynew = red[kSmallNW];
    double nfixed = red[2 * kSmallNW];
    pginf = red[0];
#pragma unroll
    for (int w = 1; w < kSmallNW; ++w) {
        pginf = fmax(pginf, red[w]);
        ynew += red[kSmallNW + w];
        nfixed += red[2 * kSmallNW + w];
    }
    __syncthreads();                                 // (the vectors and the statistics have been read)
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) dyn[(wave * NP + k) * 256 + r * 64 + lane] = acc[k][r];
    __syncthreads();
    // the waves' blocks added in wave order, static slots -> the recursion's order
    for (int idx = tid; idx < NP * 256; idx += kSmallNT) {
        const int pair = idx >> 8, r = (idx >> 6) & 3, ln = idx & 63;
        int a = 0, pb = pair;
        while (pb >= NB - a) { pb -= NB - a; ++a; }      // pair -> blocks (a, a + pb)
        const int ra = 16 * a + (ln >> 4) + 4 * r, cb = 16 * (a + pb) + (ln & 15);
        const int row = logical(ra), col = logical(cb);
        double t = dyn[idx];
#pragma unroll
        for (int w = 1; w < kSmallNW; ++w) t += dyn[w * NP * 256 + idx];
        if (row < 0 || col < 0) continue;
        G[row * Vp + col] = t;
        if (pb != 0) G[col * Vp + row] = t;              // (a block with itself holds both (row, col) and (col, row))
    }
    __syncthreads();
    if (tid == 0 && c > 0) sc.ynorm2[newest] = ynew;
    recursion_on_coefficients<M < 10 ? 10 : M>(G, Vp, c, head, m, op, &sc, G[(2 * c) * Vp + 2 * c], pginf, nfixed, ynew, yn_old, alpha_s, 0, 1);
    __syncthreads();
    if (tid == 0) note_progress(op, sc.status);
    if (sc.status == LBFGSB_RUNNING) {
        // this lane's slot's coefficient, handed round by broadcast (zero where the slot holds no pair)
        const int lg = logical(lane);
        double coef = lg >= 0 ? sc.delta[lg] : 0.0;
        asm volatile("" : "+v"(coef));                   // (here, by all lanes)
        // d = -B delta on the free set, Algorithm 2's two candidates and what the choice between them needs
        double s[6] = {0, 0, 0, 0, 0, 0};
        double sx[2 * kFoldMax];
#pragma unroll
        for (int k = 0; k < 2 * kFoldMax; ++k) sx[k] = 0.0;
        double ub = INFINITY;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = tid + r * kSmallNT;
            // (outside the test: a broadcast from a lane that is switched off would be undefined)
            double q0 = lane_value(coef, M) * ge[r], q1 = 0.0;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                q0 = fma(lane_value(coef, k), vy[r][k], q0);
                q1 = fma(lane_value(coef, M + 1 + k), vs[r][k], q1);
            }
            const double de = (freebits >> r) & 1u ? -(q0 + q1) : 0.0;
            if (e < n) {
                const double a = clampd(xe[r] + de, le[r], ue[r]) - xe[r];
                double b = de;
                if (de < 0.0 && xe[r] <= le[r] + op.eps) b = 0.0;
                if (de > 0.0 && xe[r] >= ue[r] - op.eps) b = 0.0;
                p1[e] = a;
                p2[e] = b;
                s[0] = fma(a, ge[r], s[0]); s[1] = fma(a, a, s[1]); s[2] = fma(xe[r], a, s[2]);
                s[3] = fma(b, ge[r], s[3]); s[4] = fma(b, b, s[4]); s[5] = fma(xe[r], b, s[5]);
                const double room = ((b > 0.0 ? ue[r] : le[r]) - xe[r]) / b;
                if (b != 0.0) ub = fmin(ub, room);
#pragma unroll
                for (int f = 0; f < kFoldMax; ++f) {
                    if (f < n_fold) {
                        const double ev = fold_rows[(int64_t)f * n + e];
                        sx[2 * f] = fma(ev, a, sx[2 * f]);
                        sx[2 * f + 1] = fma(ev, b, sx[2 * f + 1]);
                    }
                }
            }
        }
        // one exchange: the waves' seven results side by side, added by the first wave with the lanes as they lie
        double eight[8] = {s[0], s[1], s[2], s[3], s[4], s[5], 0.0, 0.0};
        const double sum_of = wave_sums8(eight, lane);
        ub = wave_min(ub);
        if (lane < 8) red[wave * 8 + lane] = lane == 6 ? ub : sum_of;
        if (n_fold > 0) {
#pragma unroll
            for (int k = 0; k < 2 * kFoldMax; ++k) sx[k] = wave_sum(sx[k]);
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < 2 * kFoldMax; ++k) redx[wave * 2 * kFoldMax + k] = sx[k];
            }
        }
        __syncthreads();
        if (tid < 64) {
            double tsum = red[lane], tmin = tsum;    // lane = 8 wave + k
#pragma unroll
            for (int dlt = 8; dlt < 64; dlt *= 2) {
                tsum += __shfl_xor(tsum, dlt);
                tmin = fmin(tmin, __shfl_xor(tmin, dlt));
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) s[k] = lane_bcast(tsum, k);
            ub = lane_bcast(tmin, 6);
        }
        if (tid == 0) {
            if (n_fold > 0) {
#pragma unroll
                for (int k = 0; k < 2 * kFoldMax; ++k) {
                    sx[k] = redx[k];
#pragma unroll
                    for (int w = 1; w < kSmallNW; ++w) sx[k] += redx[w * 2 * kFoldMax + k];
                }
            }
            const int branch = (s[0] <= -op.eps * s[1] && s[1] >= op.eps) ? 1 : 2;
            sc.branch = branch;
            if (branch == 1) { sc.gp = s[0]; sc.alpha_ub = 1.0; sc.pp = s[1]; sc.xp = s[2]; }
            else { sc.gp = s[3]; sc.alpha_ub = ub; sc.pp = s[4]; sc.xp = s[5]; }
            if (n_fold > 0) {
                // folded extra rows: the coefficients weight_r (e_r . p) and sum weight_r (e_r . p)^2
                double total = 0.0;
#pragma unroll
                for (int f = 0; f < kFoldMax; ++f) {
                    if (f < n_fold) {
                        const double te = branch == 1 ? sx[2 * f] : sx[2 * f + 1];
                        const double wr = fold_weight ? fold_weight[f] : 1.0;
                        fold_coef[f] = wr * te;
                        total += wr * te * te;
                    }
                }
                *fold_total = total;
            }
        }
        __syncthreads();
    }
    for (int k = tid; k < kScalWords; k += kSmallNT)
        reinterpret_cast<int*>(scal)[k] = reinterpret_cast<const int*>(&sc)[k];
}

namespace {

template <int M, int R>
void launch_t(const Dims& dm, const Opts& op, const Buffers& bf, const double* fold_rows, const double* fold_weight,
              hipStream_t st) {
    const int n_fold = fold_rows && dir_folds_extra_rows(dm) ? dm.n_extra : 0;
    hipLaunchKernelGGL((k_small_step<M, R>), dim3(1), dim3(kSmallNT), small_lds_bytes(M, dm.n), st, dm, op, (const double*)bf.x,
                       (const double*)bf.g, (const double*)bf.l, (const double*)bf.u, (const double*)bf.S,
                       (const double*)bf.Y, bf.mask, bf.scal, bf.p1, bf.p2, n_fold, fold_rows, fold_weight, bf.wextra,
                       bf.xres + dm.n_extra);
}

struct SmallVariant {
    int M;
    int64_t nmax;
    const void* kernel;
    void (*launch)(const Dims&, const Opts&, const Buffers&, const double*, const double*, hipStream_t);
};
// widest n by LDS: (2 M + 1) vectors beside G in 160 KB
#define LB_SMALL(M, R, NMAX) {M, NMAX, (const void*)k_small_step<M, R>, launch_t<M, R>}
const SmallVariant kSmall[] = {LB_SMALL(5, 1, 512), LB_SMALL(5, 2, 1024), LB_SMALL(10, 1, 512), LB_SMALL(10, 2, 832), LB_SMALL(20, 1, 384)};

const SmallVariant* variant_for(const Dims& dm) {
    for (const SmallVariant& v : kSmall)
        if (dm.m <= v.M && dm.n <= v.nmax) return &v;
    return nullptr;
}

}  // namespace

bool small_step_ok(const Dims& dm) { return !is_transport(dm.kind) && variant_for(dm) != nullptr; }

// (the limit is a property of the kernel: raised to the most the variant can ask for)
hipError_t small_step_prepare(const Dims& dm) {
    const SmallVariant* v = variant_for(dm);
    return hipFuncSetAttribute(v->kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)small_lds_bytes(v->M, v->nmax));
}

void launch_small_step(const Dims& dm, const Opts& op, const Buffers& bf, const double* fold_rows, const double* fold_weight,
                       hipStream_t st) {
    variant_for(dm)->launch(dm, op, bf, fold_rows, fold_weight, st);
}

}  // namespace lb
