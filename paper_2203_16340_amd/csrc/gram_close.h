// What the Gram kernel (gram.hip) and the direction kernel (vec.hip) share: the layout of a workgroup's partial sums, their
// addition in workgroup order, and the closing step -- Gram matrix in the recursion's order, pending update, Algorithm 3 on
// coefficients with the stopping test.  The closing step runs either in the Gram kernel's last workgroup on the scalar block
// itself, or in every workgroup of the direction kernel on a private copy of it.
#pragma once

#include "common.h"
#include "recursion.h"

namespace lb {

// The vectors by static slot: y ring 0 .. m-1 | g m | s ring m+1 .. 2m.  Of the products <a, b>, a <= b, the recursion reads
// those with a <= m; <s, s> is never asked for.  Kept row by row: (0,0) (0,1) .. (0,2m) (1,1) ..
constexpr int kGramHdr = 4;             // a workgroup's record: [0] max KKT residual, [1] #fixed, [2] ||y_new||^2, then the products
constexpr int kGramOneLevelMax = 128;   // grids up to this size add their partials in one level
constexpr int kGramOpenM = 10;          // up to this many pairs the direction kernel can do the closing step itself

__host__ __device__ constexpr int gram_products(int m) { return (m + 1) * (2 * m + 1) - m * (m + 1) / 2; }
__host__ __device__ constexpr int gram_entries(int m) { return kGramHdr + gram_products(m); }

__device__ __forceinline__ void gram_product_slots(int idx, int m, int& a, int& b) {
    int len = 2 * m + 1;
    a = 0;
    while (idx >= len) { idx -= len; --len; ++a; }
    b = a + idx;
}

// Adds the records of `nwg` workgroups (NE doubles each; entry 0 is a maximum, the others are sums) in workgroup order into
// tot[0 .. NE): thread idx takes entry idx, BATCH records at a time with every load of a batch issued before the first is used and
// none of them under a test (past the last record: the last one again, not added).
// Called by all NT threads; no barrier inside.  SAME: the records are of this launch (published), else of an earlier one.
template <int NT, bool SAME, int BATCH>
__device__ __forceinline__ void gram_sum_batches(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    for (int idx = threadIdx.x; idx < NE; idx += NT) {
        double sum = 0.0, most = -INFINITY;
        for (int k0 = 0; k0 < nwg; k0 += BATCH) {
            double v[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const double* r = grampart + (int64_t)(k0 + k < nwg ? k0 + k : nwg - 1) * NE + idx;
                v[k] = SAME ? observe(r) : *r;
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                sum += k0 + k < nwg ? v[k] : 0.0;
                most = fmax(most, v[k]);
            }
        }
        tot[idx] = idx == 0 ? most : sum;
    }
}
template <int NT, bool SAME>
__device__ __forceinline__ void gram_sum_partials_flat(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    // (the trips of different batches to memory follow one another: a batch for all where that is not too many loads)
    if (nwg <= 16) gram_sum_batches<NT, SAME, 16>(grampart, NE, nwg, tot);
    else if (nwg <= 32) gram_sum_batches<NT, SAME, 32>(grampart, NE, nwg, tot);
    else gram_sum_batches<NT, SAME, 64>(grampart, NE, nwg, tot);
}

// The closing step from the totals tot[0 .. gram_entries(m)) (LDS, complete: a barrier lies between their last write and this
// call).  c, head: the ring as it will be once the pending update is applied; base_slot: ring slot of the oldest pair.
// Gs: (2 m + 2)^2 doubles, alpha_s: kMaxM + 1 (both LDS).  sc: the scalar block this works on.  mine_a, mine_b (or -1): the
// slots of entry threadIdx.x, when the caller has worked them out while it waited for something.
// MAXK: see recursion_on_coefficients.
template <int NT, int MAXK>
__device__ __forceinline__ void gram_finish(const double* tot, double* Gs, double* alpha_s, Scal* sc, int m,
                                            int c, int head, int base_slot, const Opts& op, double yn_old, int dbg_inputs,
                                            int evaluate_stop, bool record, int mine_a = -1, int mine_b = 0) {
    const int tid = threadIdx.x;
    const int V = 2 * c + 1, Vp = V + 1;
    // The update the previous kernel left pending is applied by the last thread while the others put the matrix
    // together: a chain of two dozen dependent accesses that nothing below the barrier has to wait for twice.  (c and
    // head already are the ring as it will be; the recursion reads the iteration count and the status after the barrier.)
    if (tid == NT - 1) apply_pending(sc, m, record);
    // static slots -> the recursion's order (s oldest..newest, y oldest..newest, g)
    for (int idx = tid; idx < gram_products(m); idx += NT) {
        int a = mine_a, b = mine_b;
        if (mine_a < 0 || idx != tid) gram_product_slots(idx, m, a, b);
        auto logical = [&](int slot) -> int {
            if (slot == m) return 2 * c;
            const int ring = slot < m ? slot : slot - m - 1;
            const int j = ring >= base_slot ? ring - base_slot : ring - base_slot + m;
            if (j >= c) return -1;
            return slot < m ? c + j : j;
        };
        const int row = logical(a), col = logical(b);
        if (row >= 0 && col >= 0) {
            const double t = tot[kGramHdr + idx];
            Gs[row * Vp + col] = t;
            Gs[col * Vp + row] = t;
        }
    }
    __syncthreads();
    const double gg = Gs[(2 * c) * Vp + 2 * c];   // sum over the free set of g^2
    const double ynew = tot[2];                    // ||y_new||^2 over the full vector: kept for later iterations
    if (tid == 0 && c > 0 && !dbg_inputs) sc->ynorm2[(head - 1 + m) % m] = ynew;
    recursion_on_coefficients<MAXK>(Gs, Vp, c, head, m, op, sc, gg, tot[0], tot[1], ynew, yn_old, alpha_s, dbg_inputs, evaluate_stop);
}

}  // namespace lb
